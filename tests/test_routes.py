"""The host rules that pick the vote's layout (CPU only)."""
import pytest

from routes import clouds, parts_and_sort_us, route


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


# (lane group, parts of its windows) of the windowed vote; 0 and the general path's group
# where that is faster; the same in a batch, whose 32-bit kernels hold groups of 64 only and
# where the general path has to gain clearly
@pytest.mark.parametrize("n,m,eps,clustered,plain,batched", [
    (717, 1024, 0.03, 0, (32, 2, 0), (32, 2, 0)),           # windows of 110 sources
    (2000, 8192, 0.03, 0, (64, 1, 0), (64, 1, 0)),
    (5298, 853, 0.0461, 0, (32, 4, 0), (64, 8, 0)),        # of 400: up to 128 units
    (400, 1000, 0.0118, 0, (32, 1, 0), (32, 1, 0)),         # of 8: not split
    (100, 3000, 0.0118, 0, (64, 1, 0), (64, 1, 0)),         # of 1: few units
    (200, 17555, 0.0118, 0, (0, 0, 64), (64, 1, 0)),
    (12000, 100, 0.0118, 0, (0, 0, 16), (0, 0, 16)),        # 32 points span 39 bins
    (4000, 1000, 0.0118, 0, (0, 0, 16), (32, 2, 0)),
    (5298, 853, 0.0461, 285, (0, 0, 16), (0, 0, 16)),       # a third in one cell
])
def test_layout(n, m, eps, clustered, plain, batched):
    _, tgt, _ = clouds(n, m, 1, clustered)
    for want, b in ((plain, False), (batched, True)):
        r = route(n, tgt, 2304, eps, batched=b)
        assert (r.gref, r.windows, r.group) == want
    for asked in (32, 64):
        assert route(n, tgt, 2304, eps, lane_group=asked).gref == asked
    r = route(n, tgt, 2304, eps, lane_group=16)       # 32, or 16 where that is faster
    assert (r.gref, r.group) == ((0, 16) if plain[2] == 16 else (32, 0))


# slabs of few rotations: parts taken at 1, 100, 257, 576 and 2,304 rotations
@pytest.mark.parametrize("n,m,eps,parts", [
    (500, 3000, 0.04, (2, 2, 1, 1, 1)), (500, 3000, 0.035, (3, 2, 3, 1, 1)),
    (300, 8192, 0.03, (4, 2, 4, 4, 1)), (400, 3000, 0.0115, (16, 5, 9, 4, 1)),
    (2600, 4097, 0.03, (8, 5, 7, 4, 1)), (900, 3000, 0.06, (1, 1, 1, 1, 1)),
])
def test_parts(n, m, eps, parts):
    _, tgt, _ = clouds(n, m, 33)
    assert tuple(route(n, tgt, k, eps).parts for k in (1, 100, 257, 576, 2304)) == parts


# 32-bit counters gain from bank order from few rotations on, which count as whole rounds of
# the card's 256 workgroups; a batch's problems share theirs
@pytest.mark.parametrize("n,m,eps,k,plain,batched", [
    (5520, 3103, 0.0523, 300, 1, 1), (5520, 3103, 0.0523, 16, 1, 0), (1500, 3000, 0.05, 300, 1, 1),
    (2600, 8200, 0.03, 100, 1, 1), (2600, 4097, 0.03, 60, 0, 0), (1000, 2500, 0.05, 100, 0, 0),
    (1100, 2500, 0.03, 1000, 0, 0), (3000, 600, 0.03, 2000, 0, 0), (1100, 2500, 0.03, 4608, 1, 1),
])
def test_bank_order(n, m, eps, k, plain, batched):
    _, tgt, _ = clouds(n, m, 1)
    for lg in (64,) if n == 1100 or n == 3000 else (0, 64):
        assert route(n, tgt, k, eps, lane_group=lg).arrange == plain
        assert route(n, tgt, k, eps, lane_group=lg, batched=True).arrange == batched


def test_choosing_parts_is_short():
    """Every call of up to 2,048 rotations over several slabs pays for the choice before its
    first launch: less than half of what it pays to order 8,192 points (once as much)."""
    _, tgt, _ = clouds(10, 8192, 1)
    parts, sort = parts_and_sort_us(tgt, 84, 1000)
    assert parts < 0.5 * sort
