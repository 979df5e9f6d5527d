"""Several Chebyshev products per launch: tiles of rows with their neighbourhoods
(the time evolution, moments and the response's series on ELL and patch formats).

Checked against the oracle, and the option's own term kernels (which run while
kernel timing is on).  Sizes lie at a tile's edges (1024 rows) and where the
neighbourhood does not fit so that tiles are cut and a series takes several
launches; rows of 3, 4, 5, 8 and 12 slots with real and complex values, with and
without a table of values, single vectors and blocks.

Tolerances as in test_gpu_parity: 1e-10 (complex128) and 1e-5 (complex64) on
C(t_k) and norms; states of the two kernels differ by rounding alone: each of a
step's M products rounds by 2^-53 (2^-24) of the largest element and the
recurrence passes that on at most M times, on either side, nt steps long.
"""
import copy
import time

import numpy as np
import pytest

from tb_inputs.lattices import cell_by_name, supercell
from tb_inputs import graphene, bilayer, honeycomb3, square, sample_sites, current_operator

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
    """The same spectrum with complex hoppings: H_ij exp(i(a_i - a_j)), a from `phases` values."""
    lat = copy.copy(lat)
    a = np.random.default_rng(seed).integers(0, phases, lat.n) * (2 * np.pi / phases)
    row = np.repeat(np.arange(lat.n), np.diff(lat.row_ptr))
    lat.val = lat.val * np.exp(1j * (a[row] - a[lat.col]))
    return lat


def _tol(dtype):
    return 1e-10 if dtype == 0 else 1e-5


LATTICES = {
    # one tile: everything on chip in one launch; 1024 and 1026 rows: one and two tiles
    "w3_286": (lambda: graphene(13, 11), 8.2),
    "w4_1024": (lambda: graphene(32, 16, disorder_w=1.0, seed=5), 9.0),
    "w4_1026": (lambda: graphene(27, 19, disorder_w=1.0, seed=5), 9.0),
    "w3_2050": (lambda: graphene(41, 25), 8.2),
    "w4_10150": (lambda: graphene(175, 29, disorder_w=1.0, seed=6), 9.0),
    "w5_bilayer": (lambda: bilayer(37, 31, disorder_w=1.0, seed=7), 9.5),
    "w8_square": (lambda: square(61, 53), 4.5),
    "w12_honeycomb3": (lambda: honeycomb3(43, 37, vacancy_p=0.01, seed=9), 10.0),
    "w4_complex_table": (lambda: _gauge(graphene(47, 33, disorder_w=0.0), 4), 8.2),
    "w4_complex": (lambda: _gauge(graphene(47, 33, disorder_w=1.0, seed=8), 10 ** 6), 9.0),
    "w5_complex": (lambda: _gauge(bilayer(21, 19, disorder_w=1.0, seed=8), 10 ** 6), 9.5),
    "w8_complex": (lambda: _gauge(square(35, 33), 10 ** 6), 4.5),
    # cut in strips: neighbourhoods with long sides
    "w4_strip": (lambda: graphene(5, 900, disorder_w=1.0, seed=4), 9.0),
}


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("R,block", [(1, 1), (5, 4), (16, 16)])
@pytest.mark.parametrize("name", list(LATTICES))
def test_propagation(T, ctx, orc, name, R, block, dtype):
    make, rho = LATTICES[name]
    lat = make()
    nt = 4
    ham = ctx.build(lat, dtype=dtype, fmt=T.TBPM_FMT_ELL,
                    flags=T.TBPM_BUILD_NO_VALUE_TABLE if (R, block) == (5, 4) else 0)
    try:
        p, _ = T.make_params(rho, nt, R, block=block, seed=3)
        got = T.tbpm_propagate_dos(ctx.handle, ham, p)
        again = T.tbpm_propagate_dos(ctx.handle, ham, p)
    finally:
        T.tbpm_ham_destroy(ham)
    _, per, norms, _ = orc.corr_dos(lat, rescale=rho, num_steps=nt, num_vectors=R, seed=3)
    assert np.array_equal(got["corr"], again["corr"])           # no dependence on the order of workgroups
    assert np.abs(got["corr"] - per).max() <= _tol(dtype)
    assert np.abs(got["norms"] - norms).max() <= _tol(dtype)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("name,fmt,R,block", [
    ("w3_2050", 1, 3, 2), ("w4_10150", 1, 8, 8), ("w5_bilayer", 1, 17, 16), ("w12_honeycomb3", 1, 5, 4),
    ("w4_complex", 1, 1, 1), ("w4_10150", 3, 1, 1), ("w5_bilayer", 3, 8, 8)])
def test_states_and_sites_equal_the_term_kernels(T, ctx, name, fmt, R, block, dtype):
    """Given initial states in, final states out (blocks are laid out another way
    inside), local correlations, and more time steps than a reduction holds."""
    make, rho = LATTICES[name]
    lat = make()
    nt = 15
    rng = np.random.default_rng(1)
    psi = rng.standard_normal((R, lat.n)) + 1j * rng.standard_normal((R, lat.n))
    psi /= np.linalg.norm(psi, axis=1)[:, None]
    sites = sample_sites(lat.n, 19, 2)
    res = []
    ham = ctx.build(lat, dtype=dtype, fmt=fmt)
    try:
        M = T.tbpm_coefficients(np.pi).size
        for profiling in (False, True):
            T.tbpm_ctx_set_profiling(ctx.handle, profiling)
            p, _ = T.make_params(rho, nt, R, block=block, seed=3)
            st = T.tbpm_propagate_states(ctx.handle, ham, p, psi, keep_final=True)
            q, keep = T.make_params(rho, nt, R, block=block, seed=3, sites=sites)
            res.append((st, T.tbpm_propagate_dos(ctx.handle, ham, q)))
    finally:
        T.tbpm_ctx_set_profiling(ctx.handle, False)
        T.tbpm_ham_destroy(ham)
    bound = 2 * nt * M ** 2 * 2.0 ** (-53 if dtype == 0 else -24) * np.abs(psi).max()
    (s0, d0), (s1, d1) = res
    assert np.abs(s0["psi_final"] - s1["psi_final"]).max() <= bound
    assert np.abs(s0["corr"] - s1["corr"]).max() <= _tol(dtype)
    for key in d0:
        if isinstance(d0[key], np.ndarray):
            assert np.abs(d0[key] - d1[key]).max() <= _tol(dtype), key


UNEVEN = {
    # rows of uneven length (CSR, with a padded copy for the tiles): one tile, two,
    # pieces that vacancies cut off (isolated orbitals among them), wide rows
    "graphene_one_tile": (lambda: supercell(cell_by_name("graphene"), 13, 11, vacancy_p=0.2, seed=2), 8.2),
    "graphene": (lambda: supercell(cell_by_name("graphene"), 61, 47, vacancy_p=0.2, seed=3), 8.2),
    "graphene_clusters": (lambda: supercell(cell_by_name("graphene"), 60, 50, vacancy_p=0.5, seed=4), 8.2),
    "graphene_complex": (lambda: _gauge(supercell(cell_by_name("graphene"), 60, 50, vacancy_p=0.2, seed=4), 10 ** 6), 8.2),
    "honeycomb3": (lambda: honeycomb3(41, 37, vacancy_p=0.3, seed=5), 10.0),
    "square": (lambda: supercell(cell_by_name("square_nnn"), 51, 47, vacancy_p=0.3, seed=6), 4.5),
}


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("R,block", [(1, 1), (5, 4)])
@pytest.mark.parametrize("name", list(UNEVEN))
def test_uneven_rows(T, ctx, orc, name, R, block, dtype):
    make, rho = UNEVEN[name]
    lat = make()
    nt, num = 14, 90
    ham = ctx.build(lat, dtype=dtype)
    try:
        assert T.tbpm_ham_info(ham)["format"] == T.TBPM_FMT_CSR
        p, _ = T.make_params(rho, nt, R, block=block, seed=3)
        got = T.tbpm_propagate_dos(ctx.handle, ham, p)
        p, _ = T.make_params(rho, 0, R, block=block, seed=3)
        mu = T.tbpm_chebyshev_moments(ctx.handle, ham, p, num)
    finally:
        T.tbpm_ham_destroy(ham)
    _, per, norms, _ = orc.corr_dos(lat, rescale=rho, num_steps=nt, num_vectors=R, seed=3)
    assert np.abs(got["corr"] - per).max() <= _tol(dtype)
    assert np.abs(got["norms"] - norms).max() <= _tol(dtype)
    ref = np.stack([orc.moments(lat, orc.random_state(lat.n, 3, r), rescale=rho, num_moments=num) for r in range(R)])
    assert np.abs(mu - ref).max() <= _tol(dtype)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("num", [2, 37, 38, 39, 40, 41, 290])
@pytest.mark.parametrize("name,R,block", [("w4_1026", 1, 1), ("w4_10150", 3, 2), ("w8_complex", 1, 1)])
def test_moments(T, ctx, orc, name, R, block, num, dtype):
    """Two moments a product: launches' remainders, and more products than a reduction holds."""
    make, rho = LATTICES[name]
    lat = make()
    ham = ctx.build(lat, dtype=dtype, fmt=T.TBPM_FMT_ELL)
    try:
        p, _ = T.make_params(rho, 0, R, block=block, seed=4)
        mu = T.tbpm_chebyshev_moments(ctx.handle, ham, p, num)
    finally:
        T.tbpm_ham_destroy(ham)
    ref = np.stack([orc.moments(lat, orc.random_state(lat.n, 4, r), rescale=rho, num_moments=num) for r in range(R)])
    assert np.abs(mu - ref).max() <= _tol(dtype)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("kT", [0.02, 0.3])
def test_response(T, ctx, orc, kT, dtype):
    """The Fermi operator's series (hundreds of terms: many launches) and the time steps."""
    lat = graphene(29, 31, disorder_w=1.0, seed=5)
    A = current_operator(lat, (1, 0))
    ham = ctx.build(lat, dtype=dtype, fmt=T.TBPM_FMT_ELL)
    op = ctx.operator(ham, A)
    try:
        p, _ = T.make_params(9.0, 6, 1, seed=2)
        got = T.tbpm_response_corr(ctx.handle, ham, op, op, p, 0.1, kT)
    finally:
        T.tbpm_ham_destroy(op)
        T.tbpm_ham_destroy(ham)
    ref = orc.response_corr(lat, orc.random_state(lat.n, 2, 0), A, A, rescale=9.0, num_steps=6, mu=0.1, kT=kT)
    assert np.abs(got - ref).max() <= 0.2 * _tol(dtype)


def test_server_takes_what_fits_the_term_kernels(T, ctx, orc):
    """A request whose vectors fit the budget only without the extra ones of
    several launches per series is accepted, and gives the same rows."""
    lat = honeycomb3(70, 60, vacancy_p=0.01, seed=5)
    ham = ctx.build(lat, dtype=T.TBPM_C128, fmt=T.TBPM_FMT_ELL)
    p, _ = T.make_params(10.0, 12, 2, block=1, seed=6)
    T.tbpm_ctx_set_profiling(ctx.handle, True)
    least = T.tbpm_footprint(ham, p)
    T.tbpm_ctx_set_profiling(ctx.handle, False)
    most = T.tbpm_footprint(ham, p)
    srv = T.tbpm_server_create(ctx.handle, least, 2)
    try:
        ticket = T.tbpm_submit(srv, ham, p)
        end = time.time() + 60
        while (res := T.tbpm_poll(srv, ticket, 2, 12))[0] == T.TBPM_PENDING and time.time() < end:
            time.sleep(0.002)
    finally:
        T.tbpm_server_destroy(srv)
        T.tbpm_ham_destroy(ham)
    assert most > least
    assert res[0] == T.TBPM_OK
    per = orc.corr_dos(lat, rescale=10.0, num_steps=12, num_vectors=2, seed=6)[1]
    assert np.abs(res[1] - per).max() <= 1e-10
