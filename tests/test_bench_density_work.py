"""bench.py prices the kernels that run: behind the matrix-core support test the vector ALU forms the
distances of the pairs, not of every window candidate, and the counters' source hash covers that kernel."""
import bench
from paper_1908_01682_amd import inputs as I


def _box(n, cells, **kw):
    prob = I.dusty_box(n_side=8, cells_per_axis=4, regions_per_axis=1)
    prob.params = prob.params.replace(n_cells=(cells,) * 3, h=kw.pop("h", 1.0 / (2 * cells)), **kw)
    prob.gas = type("Gas", (), dict(n=n))()
    return prob


def test_density_kernel_and_its_vector_flops():
    one_round = 64 * 7 * 4 * 256
    assert bench.density_work(_box(128 ** 3, 64), 1000, 100) == ("k_density_tiles", 21 * 100)
    assert bench.density_work(_box(64 ** 3, 32), 1000, 100) == ("k_density", 8 * 1000 + 13 * 100)
    assert bench.density_work(_box(one_round, 40), 1, 1)[0] == "k_density"
    assert bench.density_work(_box(one_round + 1, 40), 1, 1)[0] == "k_density_tiles"
    # two cells of window, cells beyond 4 h, crowded and sparse pairs of rows, one and two dimensions
    ok = dict(least=8 * 64 ** 3, most=8 * 64 ** 3)
    assert bench.takes_tiles(_box(1, 64), **ok)
    assert not bench.takes_tiles(_box(1, 64, h=1.0 / 64), **ok)
    assert not bench.takes_tiles(_box(1, 64, h=1.0 / 260), **ok)
    assert bench.takes_tiles(_box(1, 6), 38 * 36, 55 * 36)
    assert not bench.takes_tiles(_box(1, 6), 38 * 36, 55 * 36 + 1)
    assert not bench.takes_tiles(_box(1, 6), 38 * 36 - 1, 55 * 36)
    assert not bench.takes_tiles(I.wave_2d(n_side=16), 2048, 2048)


def test_counters_belong_to_the_tile_kernel_too():
    assert "tiles.hpp" in bench.COUNTER_SOURCES
