"""The host rules that pick the vote's layout (CPU only)."""
import pytest

from routes import clouds, route


# planes of 201 x 201 bins: small sources gain from small groups, whose windows carry less
# slack; large ones from large groups, which need fewer work units
@pytest.mark.parametrize("n,m,group", [(64, 256, 64), (717, 1024, 16), (1200, 2048, 32),
                                       (2000, 4096, 32), (4096, 16384, 64)])
def test_group_of_wide_planes(n, m, group):
    _, tgt, _ = clouds(n, m, 1)
    r = route(n, tgt, 1000, 0.01)
    assert r.wide and r.sorted and r.gref == 0 and r.group == group
    for asked in (16, 32, 64):
        assert route(n, tgt, 1000, 0.01, lane_group=asked).group == asked
