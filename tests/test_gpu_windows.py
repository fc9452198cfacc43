"""The windowed vote at the sizes where its pieces end: lane groups of 32 and 64
reference points (partial last groups), source windows with and without whole blocks
and tails, one and many slabs, both counter widths, one and many chunks of 64 groups;
against the oracle, and both group sizes bit for bit against each other."""
import numpy as np
import pytest

import oracle
from paper_2502_00115_amd import synth
from parity import check_selection, compare_records

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2502_00115_amd import dses  # noqa: E402


def _clouds(n, m, seed):
    rng = np.random.default_rng(seed)
    shape = synth.multi_primitive_shape(rng)
    tgt = synth.sample_surface(rng, shape, m)
    R, t = synth.random_transform(rng)
    src = synth.jitter(rng, synth.sample_surface(rng, shape, n), 0.01) @ R.T + t
    rot = synth.random_rotations(rng, 5).reshape(-1, 9)
    f = lambda a: np.ascontiguousarray(a, np.float32)
    return f(src), f(tgt), f(rot)


# n: below, at and past a tail step (4), a block (16) and two; m: the same for groups
# of 32 and 64 and for a chunk of 64 groups (4,096 points of 64, 2,048 of 32)
@pytest.mark.parametrize("n,m,eps", [
    (1, 1, 0.05), (3, 31, 0.05), (4, 32, 0.05), (5, 33, 0.05), (15, 63, 0.04),
    (16, 64, 0.04), (17, 65, 0.04), (31, 127, 0.03), (33, 128, 0.03), (64, 129, 0.03),
    (130, 2047, 0.03), (200, 2049, 0.05), (97, 4095, 0.02), (129, 4097, 0.02),
    (1500, 4500, 0.06),
])
def test_windows_match_the_oracle(n, m, eps):
    src, tgt, rot = _clouds(n, m, 100 + n + m)
    ref = oracle.records(src, tgt, rot, eps)
    if not np.any(ref["valid"]):                 # no pair's translation lies in the box
        with pytest.raises(dses.DsesError, match="E_NOCANDIDATE"):
            dses.register(src, tgt, rot, eps)
        return
    got = {}
    for lg in (0, 16, 32, 64):
        got[lg] = dses.register(src, tgt, rot, eps, records=True, lane_group=lg)
        rep = compare_records(got[lg].records, ref, n, label=f"{n}x{m} lane_group={lg}")
        check_selection(got[lg], rep, eps, label=f"{n}x{m} lane_group={lg}")
    for lg in (16, 32, 64):
        assert got[lg].records.tobytes() == got[0].records.tobytes()


@pytest.mark.parametrize("eps,box", [(0.015, 1.0), (0.0625, 0.0625), (0.02, 0.9)])
def test_box_shapes(eps, box):
    """Planes too wide for the windowed vote's strides (135 x 135 bins: the general
    path), a box of three bins per axis, and slabs with a shorter last one."""
    src, tgt, rot = _clouds(150, 700, 7)
    ref = oracle.records(src, tgt, rot, eps, t_min=-box, t_max=box)
    got = dses.register(src, tgt, rot, eps, records=True, t_min=-box, t_max=box)
    compare_records(got.records, ref, 150, label=f"eps={eps} box={box}")


def test_batch_mixes_the_general_path_with_the_windowed_one():
    """A batch whose problems need both (a fine lattice beside coarse ones) returns what
    each problem returns alone, with and without a graph."""
    probs = []
    for i, eps in enumerate((0.05, 0.015, 0.03, 0.015)):
        src, tgt, rot = _clouds(60 + 40 * i, 300 + 50 * i, 40 + i)
        probs.append(dict(src=src, tgt=tgt, rotations=rot, eps=eps))
    alone = [dses.register(p["src"], p["tgt"], p["rotations"], p["eps"], records=True)
             for p in probs]
    for graph in (True, False, True):
        got, st = dses.register_batch(probs, records=True, use_graph=graph)
        assert st == [0] * len(probs)
        for a, b in zip(alone, got):
            assert a.records.tobytes() == b.records.tobytes()
    got, st = dses.register_batch(probs[::2], records=True)       # windowed problems only
    assert st == [0, 0]
    for a, b in zip(alone[::2], got):
        assert a.records.tobytes() == b.records.tobytes()


@pytest.mark.parametrize("n,m,eps,k,lg", [(1100, 2500, 0.03, 2304, 64), (2600, 4097, 0.03, 640, 32),
                                          (2600, 8200, 0.03, 320, 64)])
def test_bank_order_does_not_change_records(n, m, eps, k, lg):
    """Calls long enough for the staging to order each lane group's points by LDS bank
    (a last group that is not full keeps its order): every record equals that of a
    call of few rotations, which keeps the points in x order."""
    src, tgt, _ = _clouds(n, m, 9)
    rot = synth.random_rotations(np.random.default_rng(1), k).reshape(-1, 9).astype(np.float32)
    got = dses.register(src, tgt, rot, eps, records=True, lane_group=lg)
    for lo in range(0, k, k // 4):
        part = dses.register(src, tgt, rot[lo:lo + 16], eps, records=True, lane_group=lg)
        assert part.records.tobytes() == got.records[lo:lo + 16].tobytes()


@pytest.mark.parametrize("m", [511, 512, 513, 3000])
def test_equal_and_signed_x(m):
    """Reference points that share their x (both zeros among them), on both sides of the
    size from which the order by x is made by counting."""
    src, tgt, rot = _clouds(120, m, 21)
    tgt[:, 0] = np.float32(0.037) * np.round(tgt[:, 0] / np.float32(0.037))
    tgt[::2, 0] *= np.where(tgt[::2, 0] == 0, np.float32(-1), np.float32(1))
    ref = oracle.records(src, tgt, rot, 0.04)
    got = dses.register(src, tgt, rot, 0.04, records=True)
    compare_records(got.records, ref, 120, label=f"m={m}")


@pytest.mark.parametrize("n,m,eps,scorer,metric", [
    (300, 8192, 0.03, "grid", "trunc_l2"), (300, 8192, 0.03, "df", "trunc_l2"),
    (1000, 2500, 0.05, "brute", "trunc_l1"), (2600, 4097, 0.03, "grid", "votes"),
    (500, 3000, 0.13, "grid", "tls"), (400, 3000, 0.01, "grid", "inliers"),
])
def test_slabs_in_parts(n, m, eps, scorer, metric):
    """Calls of few rotations, whose slabs may go to several workgroups (two slabs at the
    coarsest lattice, a box of one plane per slab at the finest), give the records of the
    same rotations inside a list that fills the device for whole rounds."""
    src, tgt, _ = _clouds(n, m, 33)
    rot = synth.random_rotations(np.random.default_rng(2), 2048).reshape(-1, 9).astype(np.float32)
    target = dses.Target(tgt, df_trunc=eps if scorer == "df" else 0.0)
    box = dict(t_min=-0.6, t_max=0.6) if eps < 0.02 else {}
    run = lambda r: dses.register_resident(target, dses.RotationSet(r), src, eps, metric,
                                           scorer=scorer, records=True, **box).records
    want = run(rot)
    for k in (1, 3, 100, 257, 300, 576):
        assert run(rot[:k]).tobytes() == want[:k].tobytes(), k
