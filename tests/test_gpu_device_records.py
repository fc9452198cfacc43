"""Where a registration of device buffers leaves its records: a buffer of the device at
each alignment gets them (by kernel where records can be stored, else by a copy), one of a
call that finds no candidate or refuses its inputs keeps what it held."""
import numpy as np
import pytest

from paper_2502_00115_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2502_00115_amd import dses  # noqa: E402

NBYTES = dses.RECORD_DTYPE.itemsize


def _problem(k):
    rng = np.random.default_rng(5)
    tgt = rng.uniform(-0.6, 0.6, (90, 3)).astype(np.float32)
    rot = synth.random_rotations(rng, k).reshape(-1, 9).astype(np.float32)
    return tgt[:40], tgt, rot


def _into(monkeypatch, raw, offset):
    monkeypatch.setattr(dses, "_records_buffer",
                        lambda args, k: (raw, raw.data_ptr() + offset))
    monkeypatch.setattr(dses, "_records_out", lambda buf, dtype=None: buf)


@pytest.mark.parametrize("k", [1, 7, 1000])
@pytest.mark.parametrize("offset", [0, 4, 2])
def test_device_records(monkeypatch, k, offset):
    src, tgt, rot = _problem(k)
    want = dses.register(src, tgt, rot, 0.05, records=True).records.tobytes()
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (src, tgt, rot)]
    raw = torch.full((k * NBYTES + 16,), 0xA5, dtype=torch.uint8, device="cuda")
    _into(monkeypatch, raw, offset)
    dses.register(*dev, 0.05, records=True)
    got = raw.cpu().numpy()
    assert got[offset:offset + k * NBYTES].tobytes() == want
    assert (got[:offset] == 0xA5).all() and (got[offset + k * NBYTES:] == 0xA5).all()


@pytest.mark.parametrize("bad", ["no candidate", "not finite"])
def test_failed_call_leaves_the_records(monkeypatch, bad):
    src, tgt, rot = _problem(64)
    src = src.copy()
    src[:] = src + 40.0 if bad == "no candidate" else src
    if bad == "not finite":
        src[7, 1] = np.nan
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (src, tgt, rot)]
    raw = torch.full((64 * NBYTES,), 0xA5, dtype=torch.uint8, device="cuda")
    _into(monkeypatch, raw, 0)
    with pytest.raises(dses.DsesError,
                       match="E_NOCANDIDATE" if bad == "no candidate" else "E_INVAL"):
        dses.register(*dev, 0.05, records=True)
    assert bool((raw == 0xA5).all())
