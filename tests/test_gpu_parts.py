"""Calls of few rotations, whose slabs go to several workgroups: two and three slabs, the
narrowest (two planes) and most parts, both counter widths, every scorer's kernel.  Each
case shows its slabs and how many parts its calls take (routes.py)."""
import numpy as np
import pytest

from paper_2502_00115_amd import synth
from routes import clouds, route

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2502_00115_amd import dses  # noqa: E402


@pytest.mark.parametrize("n,m,eps,clustered,bits,nslabs,pps,parts,scorer,metric", [
    (500, 3000, 0.04, 0, 16, 2, 26, (2, 2, 2, 1), "grid", "tls"),
    (500, 3000, 0.035, 0, 16, 3, 19, (3, 3, 2, 3), "df", "trunc_l2"),
    (1500, 3000, 0.05, 0, 32, 2, 21, (2, 2, 2, 2), "brute", "trunc_l1"),
    (400, 3000, 0.0115, 0, 16, 87, 2, (16, 16, 5, 5), "grid", "trunc_lp"),
    (300, 1200, 0.0165, 450, 32, 61, 2, (16, 16, 5, 5), "df", "inliers"),
    (2600, 4097, 0.03, 0, 32, 8, 9, (8, 7, 5, 5), "grid", "votes"),
])
def test_parts_keep_every_record(n, m, eps, clustered, bits, nslabs, pps, parts, scorer, metric):
    src, tgt, _ = clouds(n, m, 33, clustered)
    r = route(n, tgt, 2304, eps)
    assert (r.bits, r.nslabs, r.pps, r.parts) == (bits, nslabs, pps, 1) and r.gref
    rot = synth.random_rotations(np.random.default_rng(2), 2304).reshape(-1, 9).astype(np.float32)
    target = dses.Target(tgt, df_trunc=eps if scorer == "df" else 0.0)

    def run(rotations):
        return dses.register_resident(target, dses.RotationSet(rotations), src, eps, metric,
                                      scorer=scorer, records=True).records

    want = run(rot)
    for k, p in zip((1, 3, 100, 300), parts):
        assert route(n, tgt, k, eps).parts == p
        assert run(rot[:k]).tobytes() == want[:k].tobytes(), k
