"""The general vote path, for x planes wider than the windowed vote's 16-bit strides (more
than 65,535 bytes of counters), for sources too many to be sorted and where it is the faster:
both counter widths, every lane-group size, alone, in batches and served, at the sizes where
its pieces end.  Each test shows that its calls take the path (routes.py)."""
import numpy as np
import pytest

import oracle
from paper_2502_00115_amd import synth
from parity import check_selection, compare_records
from routes import clouds, route

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2502_00115_amd import dses  # noqa: E402


# n: below, at and past a tail step and a block (8, 16 and 32 sources with groups of 64, 32
# and 16); m: the same for the groups; 420 reference points in one bin: 32-bit counters
@pytest.mark.parametrize("n,m,eps,clustered", [
    (3, 15, 0.01, 0), (4, 16, 0.01, 0), (5, 17, 0.01, 0), (7, 31, 0.01, 0), (9, 33, 0.01, 0),
    (16, 63, 0.01, 0), (17, 65, 0.01, 0), (31, 129, 0.01, 0), (33, 200, 0.01, 0),
    (150, 700, 0.01, 0), (1500, 300, 0.01, 0), (160, 600, 0.0125, 420), (157, 1025, 0.0125, 420),
])
def test_wide_planes_match_the_oracle(n, m, eps, clustered):
    src, tgt, rot = clouds(n, m, 100 + n + m, clustered)
    r = route(n, tgt, len(rot), eps)
    assert r.wide and r.sorted and r.gref == 0 and r.bits == (32 if clustered else 16)
    ref = oracle.records(src, tgt, rot, eps)
    assert np.any(ref["valid"])
    got = {}
    for lg in (0, 16, 32, 64):
        got[lg] = dses.register(src, tgt, rot, eps, records=True, lane_group=lg)
        rep = compare_records(got[lg].records, ref, n, label=f"{n}x{m} lane_group={lg}")
        check_selection(got[lg], rep, eps, label=f"{n}x{m} lane_group={lg}")
    for lg in (16, 32, 64):
        assert got[lg].records.tobytes() == got[0].records.tobytes()


@pytest.mark.parametrize("m,eps,clustered,bits,wide", [
    (3, 0.05, 0, 16, 0), (40, 0.05, 30, 32, 0), (3, 0.01, 0, 16, 1), (41, 0.0125, 30, 32, 1),
])
def test_unsorted_sources_match_the_oracle(m, eps, clustered, bits, wide):
    n = 16385
    src, tgt, rot = clouds(n, m, 7, clustered)
    r = route(n, tgt, 3, eps)
    assert (r.sorted, r.gref, r.bits, r.wide) == (0, 0, bits, wide)
    ref = oracle.records(src, tgt, rot[:3], eps)
    got = dses.register(src, tgt, rot[:3], eps, records=True)
    compare_records(got.records, ref, n, label=f"m={m} eps={eps}")


# groups of 16 points and of 64, whole and partial, one and many slabs, both counter widths
@pytest.mark.parametrize("n,m,eps,clustered,group,bits", [
    (12000, 100, 0.0118, 0, 16, 16), (3000, 17, 0.02, 0, 16, 16), (4000, 1001, 0.0118, 0, 16, 16),
    (1000, 853, 0.0461, 285, 16, 32), (717, 1025, 0.03, 500, 16, 32),
    (100, 5001, 0.0118, 0, 64, 16), (10, 8192, 0.03, 0, 64, 16),
])
def test_faster_general_path_equals_the_windowed_vote(n, m, eps, clustered, group, bits):
    src, tgt, rot = clouds(n, m, 60 + m, clustered)
    r = route(n, tgt, 2304, eps)
    assert (r.wide, r.gref, r.group, r.bits) == (0, 0, group, bits)
    more = synth.random_rotations(np.random.default_rng(m), 2304).reshape(-1, 9)
    rot = np.concatenate([rot, more[len(rot):]]).astype(np.float32)
    got = dses.register(src, tgt, rot, eps, records=True)
    for lg in (16, 32, 64):
        assert lg == 16 or route(n, tgt, 2304, eps, lane_group=lg).gref == lg
        want = dses.register(src, tgt, rot, eps, records=True, lane_group=lg)
        assert got.records.tobytes() == want.records.tobytes()
    compare_records(got.records[:5], oracle.records(src, tgt, rot[:5], eps), n, label=f"{n}x{m}")


def _problems():
    """Problems of both paths, the general ones with 16- and 32-bit counters and unsorted."""
    out = []
    for i, (n, m, eps, clustered) in enumerate([
            (60, 300, 0.05, 0), (100, 350, 0.01, 0), (140, 400, 0.03, 0), (180, 450, 0.0125, 420),
            (16385, 5, 0.05, 0), (717, 1024, 0.01, 0), (200, 500, 0.05, 0),
            (6000, 100, 0.0118, 0)]):
        src, tgt, rot = clouds(n, m, 40 + i, clustered)
        r = route(n, tgt, len(rot), eps, batched=True)
        assert (r.gref == 0) == (i in (1, 3, 4, 5, 7)) and r.bits == (32 if clustered else r.bits)
        out.append(dict(src=src, tgt=tgt, rotations=rot, eps=eps))
    return out


def _alone(p):
    return dses.register(p["src"], p["tgt"], p["rotations"], p["eps"], records=True)


def test_batch_mixes_both_paths():
    """Every problem of a mixed batch returns what it returns alone, eagerly and by graph
    replays, with windowed-only and general-only batches in between; any split of the windows."""
    probs = _problems()
    alone = [_alone(p).records.tobytes() for p in probs]
    general = [1, 3, 4, 5, 7]
    windowed = [0, 2, 6]
    every = list(range(len(probs)))
    for which, graph in ((every, True), (every, False), (every, True), (windowed, True),
                         (general, True), (every, True), (general, False)):
        got, st = dses.register_batch([probs[i] for i in which], records=True, use_graph=graph)
        assert st == [0] * len(which)
        assert [g.records.tobytes() for g in got] == [alone[i] for i in which]
    # problems that would gain: all of them together, or not for their own sake
    for which in ([7, 7], [7, 0], [0, 7, 6]):
        got, _ = dses.register_batch([probs[i] for i in which], records=True)
        assert [g.records.tobytes() for g in got] == [alone[i] for i in which]
    for parts in (1, 3, 16):
        got, _ = dses.register_batch(probs, records=True, vote_parts=parts)
        assert [g.records.tobytes() for g in got] == alone
    got, _ = dses.register_batch(probs, records=True, autotune=True)
    assert [g.records.tobytes() for g in got] == alone


def test_server_mixes_both_paths():
    """Served requests of both paths, all outstanding at once, equal their lone calls."""
    _, tgt, _ = clouds(10, 900, 5)
    rot = synth.random_rotations(np.random.default_rng(6), 300).reshape(-1, 9).astype(np.float32)
    target, rotset = dses.Target(tgt), dses.RotationSet(rot)
    reqs = []
    for i in range(12):
        n, eps = 70 + 45 * i, (0.01, 0.03, 0.0125)[i % 3]
        src = clouds(n, 900, 5)[0]
        assert (route(n, tgt, len(rot), eps, batched=True).gref == 0) == (i % 3 == 0)
        reqs.append((src, eps))
    with_records = [i % 2 == 0 for i in range(12)]
    want = [dses.register(src, tgt, rot, eps, records=True) for src, eps in reqs]
    srv = dses.Server()
    got = []
    for _ in range(2):
        ids = [srv.submit(target, rotset, src, eps, records=rec)
               for (src, eps), rec in zip(reqs, with_records)]
        got += [srv.wait(i, timeout_ms=60000) for i in ids]
    srv.close()
    for g, w, rec in zip(got, 2 * want, 2 * with_records):
        assert (g.rot_index, g.error, g.inliers, g.votes) == (w.rot_index, w.error, w.inliers,
                                                              w.votes)
        if rec:
            assert g.records.tobytes() == w.records.tobytes()
