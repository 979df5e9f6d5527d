"""Calls that tiles must not make slower than the kernels before them, as times of the
same process.

Storing uneven rows with a plan of tiles pays for itself in one short run: H stored by
the library's choice and 16 time steps of four vectors take no longer than with the CSR
named, which has no plan (about 9 ms against 12;
22 while the tiles were grown by one thread and every depth was tried on all of them)."""
import time

import pytest

from tb_inputs.lattices import cell_by_name, supercell

pytestmark = pytest.mark.gpu


def test_one_short_run_on_a_fresh_h():
    from paper_2509_26309_amd import tbpm as T
    lat = supercell(cell_by_name("graphene"), 640, 480, vacancy_p=0.2, seed=3)
    with T.Context(0) as ctx:
        p, _ = T.make_params(9.0, 16, 4, block=4, seed=1)

        def once(fmt):
            t = time.perf_counter()
            ham = ctx.build(lat, fmt=fmt)
            T.tbpm_propagate_dos(ctx.handle, ham, p)
            took = time.perf_counter() - t
            planned = T.tbpm_ham_tiles(ham, 4)["products"] > 0
            T.tbpm_ham_destroy(ham)
            return took, planned

        runs = [(once(T.TBPM_FMT_AUTO), once(T.TBPM_FMT_CSR)) for _ in range(6)]
    assert all(auto[1] and not named[1] for auto, named in runs)
    assert min(auto[0] for auto, _ in runs) <= min(named[0] for _, named in runs)


def test_wide_blocks_of_a_small_sample():
    """Local correlations of a block of 64 vectors on 512 rows by tiles: starting a block and
    gathering the sites is a launch each for the whole block, so the tiles take no longer than
    the term kernels (launched with kernel timing on)."""
    from paper_2509_26309_amd import tbpm as T
    from tb_inputs import graphene, sample_sites
    lat = graphene(16, disorder_w=1.0, seed=1)
    with T.Context(0) as ctx:
        ham = ctx.build(lat)
        p, keep = T.make_params(9.0, 32, 64, block=64, seed=1, sites=sample_sites(lat.n, 50, 3))
        took = {}
        for timing in (False, True):
            T.tbpm_ctx_set_profiling(ctx.handle, timing)
            runs = []
            for _ in range(8):
                t = time.perf_counter()
                T.tbpm_propagate_dos(ctx.handle, ham, p)
                runs.append(time.perf_counter() - t)
            took[timing] = min(runs)
        assert T.tbpm_ham_tiles(ham, 64)["products"] > 0
        T.tbpm_ham_destroy(ham)
    assert took[False] <= took[True], took


@pytest.mark.parametrize("cells", [512, 1024])
def test_moments_by_the_faster_kernels(cells):
    """Moments of the clean bilayer in complex128 (the tiles' kernel spills registers for its
    sums there): no slower than by pairs of products, which kernel timing asks for."""
    from paper_2509_26309_amd import tbpm as T
    from tb_inputs import bilayer
    lat = bilayer(cells)
    with T.Context(0) as ctx:
        ham = ctx.build(lat)
        p, _ = T.make_params(9.0, 0, 1, seed=1)
        took = {}
        for timing in (False, True):
            T.tbpm_ctx_set_profiling(ctx.handle, timing)
            runs = []
            for _ in range(8):
                t = time.perf_counter()
                T.tbpm_chebyshev_moments(ctx.handle, ham, p, 300)
                runs.append(time.perf_counter() - t)
            took[timing] = min(runs)
        assert T.tbpm_ham_tiles(ham, 1)["tiles"] > 0
        T.tbpm_ham_destroy(ham)
    assert took[False] <= 1.1 * took[True], took


def test_rows_per_tile_of_a_sample_with_gaps():
    """What growing tiles in ranges leaves over shares tiles: at most 1.4 times as many as
    full ones (1.6 while only pieces under an eighth of a tile did)."""
    from paper_2509_26309_amd import tbpm as T
    lat = supercell(cell_by_name("graphene"), 772, 462, vacancy_p=0.3, seed=3)
    with T.Context(0) as ctx:
        ham = ctx.build(lat, dtype=T.TBPM_C64)
        tiles = T.tbpm_ham_tiles(ham, 1)["tiles"]
        T.tbpm_ham_destroy(ham)
    assert 0 < tiles <= 1.4 * lat.n / 1024
