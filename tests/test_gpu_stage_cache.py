"""The staged copies of a served reference are bounded: requests whose translation boxes
differ in their upper ends alone share a few of them, and return what lone calls return."""
import numpy as np
import pytest

from paper_2502_00115_amd import synth
from routes import clouds, route

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2502_00115_amd import dses  # noqa: E402

M = 1 << 18
COPY = 2 * (4 << 20)     # two arrays of 12 to 13 bytes a point, each in whole 2 MiB pages


@pytest.mark.parametrize("eps,gref,orders", [(0.05, True, 4), (0.01, False, 1)])
def test_boxes_of_one_origin_share_staged_copies(eps, gref, orders):
    src, tgt, _ = clouds(40, M, 3)
    assert (route(40, tgt, 8, eps).gref != 0) == gref
    rot = synth.random_rotations(np.random.default_rng(4), 8).reshape(-1, 9).astype(np.float32)
    target, rotset = dses.Target(tgt), dses.RotationSet(rot)
    uppers = [1.0 - eps * i for i in range(12)]
    want = [dses.register_resident(target, rotset, src, eps, t_min=-1.0, t_max=u) for u in uppers]
    srv = dses.Server()

    def serve(u):
        return srv.wait(srv.submit(target, rotset, src, eps, t_min=-1.0, t_max=u),
                        timeout_ms=60000)

    # the runtime allocates 32 to 64 MiB on the first use of each of the server's streams
    for _ in range(4):
        got = [serve(uppers[0])]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    got += [serve(u) for u in uppers[1:]]
    used = free - torch.cuda.mem_get_info()[0]
    got += [serve(u) for u in uppers]
    again = free - torch.cuda.mem_get_info()[0]
    srv.close()
    assert used <= orders * COPY and again == used
    for g, w in zip(got, 2 * want):
        assert (g.rot_index, g.error, g.inliers, g.votes) == (w.rot_index, w.error, w.inliers,
                                                              w.votes)
        assert np.array_equal(g.t, w.t)
