"""Long sweeps put the points of each lane group into the order of their LDS banks; the
records have to be those of the x order.  Each test shows that the long call does so and the
short ones it is compared with do not (routes.py)."""
import numpy as np
import pytest

from paper_2502_00115_amd import synth
from routes import clouds, route

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2502_00115_amd import dses  # noqa: E402

# groups of 64 points under 16- and 32-bit counters and of 32 under 32-bit ones, with whole
# groups only, a last group of one point and of most of one (which keep their order)
CASES = [(1100, 2500, 0.03, 4608, 64, 16), (1100, 2560, 0.03, 4608, 64, 16),
         (2600, 4097, 0.03, 1152, 32, 32), (2600, 4095, 0.03, 1152, 32, 32),
         (2600, 8200, 0.03, 576, 64, 32)]


def _long(n, m, k):
    src, tgt, _ = clouds(n, m, 9)
    rot = synth.random_rotations(np.random.default_rng(1), k).reshape(-1, 9).astype(np.float32)
    return src, tgt, rot


@pytest.mark.parametrize("n,m,eps,k,lg,bits", CASES)
def test_bank_order_keeps_every_record(n, m, eps, k, lg, bits):
    src, tgt, rot = _long(n, m, k)
    r = route(n, tgt, k, eps, lane_group=lg)
    assert r.arrange and r.gref == lg and r.bits == bits
    assert not route(n, tgt, 32, eps, lane_group=lg).arrange
    got = dses.register(src, tgt, rot, eps, records=True, lane_group=lg)
    for lo in range(0, k, k // 8):
        part = dses.register(src, tgt, rot[lo:lo + 32], eps, records=True, lane_group=lg)
        assert part.records.tobytes() == got.records[lo:lo + 32].tobytes()


# few rotations in bank order, in parts and whole, against a batch of eight, which stay in the
# order by x
@pytest.mark.parametrize("n,m,eps,k,lg,parts", [(5520, 3103, 0.0523, 40, 64, 2),
                                                (5520, 3103, 0.0523, 300, 32, 2),
                                                (3001, 3000, 0.05, 200, 64, 1),
                                                (2600, 8200, 0.03, 100, 32, 5)])
def test_bank_order_of_few_rotations(n, m, eps, k, lg, parts):
    src, tgt, rot = _long(n, m, k)
    r = route(n, tgt, k, eps, lane_group=lg)
    assert r.arrange and r.gref == lg and r.bits == 32 and r.parts == parts
    got = dses.register(src, tgt, rot, eps, records=True, lane_group=lg)
    few = 8
    assert not route(n, tgt, few, eps, lane_group=lg, batched=True).arrange
    some, _ = dses.register_batch([dict(src=src, tgt=tgt, rotations=rot[:few], eps=eps)],
                                  records=True)
    assert some[0].records.tobytes() == got.records[:few].tobytes()


def test_bank_order_in_batches_and_served():
    """The batched staging orders the groups of its long problems only; a served reference is
    always in bank order."""
    probs, want = [], []
    for n, m, eps, k, lg, bits in CASES[::2]:
        src, tgt, rot = _long(n, m, k)
        assert route(n, tgt, k, eps).arrange
        for some in (rot, rot[:40]):
            probs.append(dict(src=src, tgt=tgt, rotations=some, eps=eps))
        short = dses.register(src, tgt, rot[:40], eps, records=True)
        want.append(short.records.tobytes())
    for graph in (False, True):
        got, _ = dses.register_batch(probs, records=True, use_graph=graph)
        for i, w in enumerate(want):
            assert got[2 * i].records[:40].tobytes() == w
            assert got[2 * i + 1].records.tobytes() == w
    srv = dses.Server()
    kept = [(dses.Target(p["tgt"]), dses.RotationSet(p["rotations"])) for p in probs[1::2]]
    ids = [srv.submit(*tr, p["src"], p["eps"], records=True) for tr, p in zip(kept, probs[1::2])]
    got = [srv.wait(i, timeout_ms=60000) for i in ids]
    srv.close()
    assert [g.records.tobytes() for g in got] == want
