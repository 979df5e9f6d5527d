"""Several products per launch at the edges of its tiles: a lane has two rows of a tile
(512 lanes, tiles of at most 1024 rows), so samples of 511 to 1025 rows, of one and two
tiles, and ELL and CSR samples whose tiles pass 512 rows (more than 131,072 rows); with
a table of values and without, real and complex, for every row length.  The plan itself
is asserted, so that no case compares the term kernels with themselves.

Against the oracle; tolerances as in test_gpu_parity: 1e-10 (complex128), 1e-5
(complex64) on C(t_k), norms and moments.
"""
import copy

import numpy as np
import pytest

from tb_inputs.lattices import cell_by_name, supercell
from tb_inputs import bilayer, graphene, square

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2509_26309_amd import tbpm
    return tbpm


@pytest.fixture(scope="module")
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


def _gauge(lat, phases, seed=3):
    """The same spectrum with complex hoppings of a few values: H_ij exp(i(a_i - a_j))."""
    lat = copy.copy(lat)
    a = np.random.default_rng(seed).integers(0, phases, lat.n) * (2 * np.pi / phases)
    row = np.repeat(np.arange(lat.n), np.diff(lat.row_ptr))
    lat.val = lat.val * np.exp(1j * (a[row] - a[lat.col]))
    return lat


def _check(T, ctx, orc, lat, rho, fmt, stored, dtype, R, block, tiles, flags=0, table=None, nt=4, num=61):
    """tiles(plan) says whether the plan is the one that the case is about."""
    ham = ctx.build(lat, dtype=dtype, fmt=fmt, flags=flags)
    try:
        assert T.tbpm_ham_info(ham)["format"] == stored
        plan = T.tbpm_ham_tiles(ham, block)
        assert plan["products"] > 0 and tiles(plan), plan
        if table is not None:
            assert (T.tbpm_ham_value_table(ham)["entries"] > 0) == table
        p, _ = T.make_params(rho, nt, R, block=block, seed=3)
        got = T.tbpm_propagate_dos(ctx.handle, ham, p)
        p, _ = T.make_params(rho, 0, R, block=block, seed=3)
        mu = T.tbpm_chebyshev_moments(ctx.handle, ham, p, num)
    finally:
        T.tbpm_ham_destroy(ham)
    tol = 1e-10 if dtype == 0 else 1e-5
    _, per, norms, _ = orc.corr_dos(lat, rescale=rho, num_steps=nt, num_vectors=R, seed=3)
    assert np.abs(got["corr"] - per).max() <= tol
    assert np.abs(got["norms"] - norms).max() <= tol
    ref = np.stack([orc.moments(lat, orc.random_state(lat.n, 3, r), rescale=rho, num_moments=num) for r in range(R)])
    assert np.abs(mu - ref).max() <= tol


EDGES = {
    # rows of one patch: a lane's second row begins at 512, the tile ends at 1024
    "w8_511": (lambda: square(7, 73), 4.5, 511),
    "w4_512": (lambda: graphene(16, 16, disorder_w=1.0, seed=5), 9.0, 512),
    "w8_513": (lambda: square(19, 27), 4.5, 513),
    "w5_516": (lambda: bilayer(3, 43, disorder_w=1.0, seed=6), 9.5, 516),
    "w8_1023": (lambda: square(33, 31), 4.5, 1023),
    "w4_1024": (lambda: graphene(32, 16, disorder_w=1.0, seed=5), 9.0, 1024),
    "w3_1024": (lambda: graphene(16, 32), 8.2, 1024),
}


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("R,block", [(1, 1), (3, 2)])
@pytest.mark.parametrize("name", list(EDGES))
def test_one_tile(T, ctx, orc, name, R, block, dtype):
    make, rho, n = EDGES[name]
    lat = make()
    assert lat.n == n
    _check(T, ctx, orc, lat, rho, T.TBPM_FMT_PATCH, T.TBPM_FMT_PATCH, dtype, R, block,
           lambda plan: plan["tiles"] == 1 and plan["tile_rows"] == n)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("name,make,rho", [("w8_1025", lambda: square(41, 25), 4.5),
                                           ("w4_1026", lambda: graphene(27, 19, disorder_w=1.0, seed=5), 9.0)],
                         ids=["w8_1025", "w4_1026"])
def test_two_tiles(T, ctx, orc, name, make, rho, dtype):
    _check(T, ctx, orc, make(), rho, T.TBPM_FMT_PATCH, T.TBPM_FMT_PATCH, dtype, 2, 2,
           lambda plan: plan["tiles"] >= 2)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("kind", ["ell", "csr"])
def test_tiles_of_more_than_a_row_per_lane(T, ctx, orc, kind, dtype):
    """ELL and CSR tiles hold a 256th of the rows: past 131,072 rows a lane has two."""
    if kind == "ell":
        lat = graphene(270, 250, disorder_w=1.0, seed=4)
        fmt = stored = T.TBPM_FMT_ELL
    else:
        lat = supercell(cell_by_name("graphene"), 310, 290, vacancy_p=0.2, seed=4)
        fmt, stored = T.TBPM_FMT_AUTO, T.TBPM_FMT_CSR
    assert lat.n > 131072
    _check(T, ctx, orc, lat, 9.0, fmt, stored, dtype, 2, 2, lambda plan: plan["tile_rows"] > 512, nt=2, num=21)


TABLES = {
    "w3": (lambda: graphene(41, 25), 8.2),
    "w4": (lambda: graphene(41, 25, disorder_w=1.0, seed=6), 9.0),
    "w4_complex": (lambda: _gauge(graphene(41, 25, disorder_w=1.0, seed=6), 4), 9.0),
    "w5": (lambda: bilayer(21, 19, disorder_w=1.0, seed=7), 9.5),
    "w5_complex": (lambda: _gauge(bilayer(21, 19, disorder_w=1.0, seed=7), 4), 9.5),
    "w8": (lambda: square(45, 37), 4.5),
    "w8_complex": (lambda: _gauge(square(45, 37), 4), 4.5),
}


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("table", [True, False])
@pytest.mark.parametrize("name", list(TABLES))
def test_value_table(T, ctx, orc, name, table, dtype):
    """A table of the hoppings' values exists on patch-reordered H, unless switched off."""
    make, rho = TABLES[name]
    _check(T, ctx, orc, make(), rho, T.TBPM_FMT_PATCH, T.TBPM_FMT_PATCH, dtype, 3, 2, lambda plan: plan["tiles"] >= 2,
           flags=0 if table else T.TBPM_BUILD_NO_VALUE_TABLE, table=table)


def test_query_arguments(T, ctx):
    lat = graphene(16, 16)
    ham = ctx.build(lat, fmt=T.TBPM_FMT_CSR)
    try:
        assert T.tbpm_ham_tiles(ham, 1) == {"products": 0, "tiles": 0, "tile_rows": 0}
        for block in (0, 65):
            with pytest.raises(T.TBPMError):
                T.tbpm_ham_tiles(ham, block)
    finally:
        T.tbpm_ham_destroy(ham)


@pytest.mark.parametrize("kind", ["ell", "csr"])
def test_h_given_in_device_memory(T, ctx, kind):
    """The plan of an H given in device memory is that of the same H given in host memory."""
    import torch
    if kind == "ell":
        lat, fmt = graphene(61, 47, disorder_w=1.0, seed=4), T.TBPM_FMT_ELL
    else:
        lat, fmt = supercell(cell_by_name("graphene"), 61, 47, vacancy_p=0.2, seed=3), T.TBPM_FMT_AUTO
    dev = [torch.as_tensor(x, device="cuda") for x in (np.asarray(lat.row_ptr, dtype=np.int64),
                                                       np.asarray(lat.col, dtype=np.int32),
                                                       np.asarray(lat.val, dtype=np.complex128))]
    torch.cuda.synchronize()
    got = []
    for ham in (ctx.build(lat, fmt=fmt),
                T.tbpm_build_csr_device(ctx.handle, lat.n, lat.nnz, *(x.data_ptr() for x in dev), 0, fmt)):
        try:
            p, _ = T.make_params(9.0, 5, 2, block=2, seed=3)
            got.append((T.tbpm_ham_tiles(ham, 2), T.tbpm_propagate_dos(ctx.handle, ham, p)["corr"]))
        finally:
            T.tbpm_ham_destroy(ham)
    assert got[0][0] == got[1][0] and got[0][0]["products"] > 0
    assert np.array_equal(got[0][1], got[1][1])
