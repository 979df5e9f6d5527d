"""The kernels of one and two Chebyshev terms per launch, which tiles (several
products per launch) have taken most of the small samples from: they run where H has
no plan of tiles, where the tiles take longer, where memory is short, and while kernel
timing is on.  These tests switch the timing on (or take an H without a plan) and
assert from the launches counted which kernels ran.

A launch holds the newest terms of its rows, so the series is brought up to date only
where the next launch could no longer do it; every length M is another pattern.
Checked against the oracle's one update per term; tolerances as in test_gpu_parity:
1e-10 (complex128) and 1e-5 (complex64) on C(t_k), few steps.
"""
import numpy as np
import pytest
from scipy.special import jv

from tb_inputs import PrimCell, bilayer, graphene, honeycomb3, supercell

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


def _eps(orc, M):
    eps = 1.0001 * abs(jv(M, np.pi))
    assert orc.coefficients(np.pi, eps).size == M
    return eps


def _launches(M, nt, route):
    """Launches of nt steps of a block: terms one by one, in pairs, or in pairs that
    straddle the steps (M even and at least 6: every other step ends with the next's
    first term)."""
    if route == "single" or M < 4:
        return nt * (M - 1)
    if route == "pair" or M % 2 or M < 6:
        return nt * (1 + (M - 2) % 2 + (M - 2) // 2)
    return nt // 2 * (M // 2 + (M - 2) // 2) + nt % 2 * (1 + (M - 2) // 2)


def _timed(T, ctx, ham, rho, nt, R, block, seed, eps):
    T.tbpm_ctx_set_profiling(ctx.handle, True)
    try:
        p, _ = T.make_params(rho, nt, R, block=block, seed=seed, bessel_eps=eps)
        out = T.tbpm_propagate_dos(ctx.handle, ham, p)
        return out, sum(T.tbpm_ctx_kernel_time(ctx.handle, k)[1] for k in range(3))
    finally:
        T.tbpm_ctx_set_profiling(ctx.handle, False)


CASES = [
    # (name, lattice maker, rho, dtype, format, block, launches)
    ("csr_c128", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 9.0, 0, 0, 1, "single"),
    ("csr_c64_block4", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 9.0, 1, 0, 4, "single"),
    ("ell_c128", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 9.0, 0, 1, 1, "single"),
    ("ell_c128_block4", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 9.0, 0, 1, 4, "single"),
    ("ell_c64_block2", lambda: graphene(17, 12, disorder_w=1.0, seed=6), 9.0, 1, 1, 2, "single"),
    ("ell_c64_block16", lambda: graphene(17, 12, disorder_w=1.0, seed=6), 9.0, 1, 1, 16, "single"),
    ("patch_c128", lambda: graphene(41, 37, disorder_w=1.0, seed=7), 9.0, 0, 3, 1, "cross"),
    ("patch_c64", lambda: graphene(41, 37, disorder_w=1.0, seed=7), 9.0, 1, 3, 1, "cross"),
    ("patch_c128_w8", lambda: supercell(PrimCell("sq", 1, [(1, 0, 0, 0, -1.0), (0, 1, 0, 0, -1.0), (1, 1, 0, 0, 0.1),
                                                           (1, -1, 0, 0, 0.1)], (0.0,)), 45, 37), 4.5, 0, 3, 1,
     "cross"),
    ("pairs_w5_block8", lambda: bilayer(23, 21, disorder_w=1.0, seed=8), 9.0, 1, 3, 8, "pair"),
    ("pairs_w5_block16", lambda: bilayer(23, 21, disorder_w=1.0, seed=8), 9.0, 1, 3, 16, "pair"),
    ("pairs_w4_block8", lambda: graphene(41, 37, disorder_w=1.0, seed=7), 9.0, 1, 3, 8, "pair"),
    ("pairs_w4_block16", lambda: graphene(41, 37, disorder_w=1.0, seed=7), 9.0, 1, 3, 16, "pair"),
    ("pairs_one_patch_block8", lambda: bilayer(16, disorder_w=1.0, seed=16), 9.0, 1, 3, 8, "pair"),
    ("pairs_ragged_patch_block16", lambda: bilayer(15, disorder_w=1.0, seed=15), 9.0, 1, 3, 16, "pair"),
    ("staged_block16", lambda: honeycomb3(33, 31, vacancy_p=0.01, seed=9), 10.0, 1, 3, 16, "single"),
]


@pytest.mark.parametrize("M", [4, 5, 6, 7, 8, 9, 10, 12, 15, 18, 20])
@pytest.mark.parametrize("name,make,rho,dtype,fmt,block,route", CASES, ids=[c[0] for c in CASES])
def test_every_series_length(T, ctx, orc, name, make, rho, dtype, fmt, block, route, M):
    eps = _eps(orc, M)
    lat, nt = make(), 5
    ham = ctx.build(lat, dtype=dtype, fmt=fmt)
    try:
        assert T.tbpm_ham_info(ham)["format"] == fmt
        if fmt == 3:
            assert T.tbpm_ham_fused_pairs(ham, block) == (route != "single")
        out, launches = _timed(T, ctx, ham, rho, nt, block, block, 3, eps)
    finally:
        T.tbpm_ham_destroy(ham)
    assert launches == _launches(M, nt, route)
    _, per, norms, _ = orc.corr_dos(lat, rescale=rho, num_steps=nt, num_vectors=block, seed=3, eps=eps)
    tol = 1e-10 if dtype == 0 else 1e-5
    assert np.abs(out["corr"] - per).max() <= tol
    assert np.abs(out["norms"] - norms).max() <= tol


def _ring(hops, w):
    """A chain with `hops` neighbours on either side: rows of 2 hops (+ 1 with disorder) entries."""
    cell = PrimCell("ring", 1, [(0, d, 0, 0, -1.0 / d) for d in range(1, hops + 1)], (0.0,))
    return supercell(cell, 1, 997, disorder_w=w, seed=hops)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("block", [1, 4])
@pytest.mark.parametrize("hops,w,width", [(1, 0.0, 2), (3, 0.0, 6), (3, 1.0, 7), (4, 1.0, 9), (5, 0.0, 10),
                                          (5, 1.0, 11), (8, 0.0, 16)])
def test_rows_without_tiles(T, ctx, orc, hops, w, width, block, dtype):
    """ELL rows of a width that the tiles' kernel is not compiled for: terms one by one, timed or not."""
    lat, nt, rho = _ring(hops, w), 6, 7.0
    assert int(np.diff(lat.row_ptr).max()) == width
    ham = ctx.build(lat, dtype=dtype, fmt=T.TBPM_FMT_ELL)
    try:
        assert T.tbpm_ham_tiles(ham, block) == {"products": 0, "tiles": 0, "tile_rows": 0}
        p, _ = T.make_params(rho, nt, block, block=block, seed=2)
        got = T.tbpm_propagate_dos(ctx.handle, ham, p)
        timed, launches = _timed(T, ctx, ham, rho, nt, block, block, 2, 0.0)
    finally:
        T.tbpm_ham_destroy(ham)
    assert launches == nt * (T.tbpm_coefficients(np.pi).size - 1)
    assert np.array_equal(got["corr"], timed["corr"])
    per = orc.corr_dos(lat, rescale=rho, num_steps=nt, num_vectors=block, seed=2)[1]
    assert np.abs(got["corr"] - per).max() <= (1e-10 if dtype == 0 else 1e-5)


GRAPHS = [
    ("ell_c128", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 0, 1, 1, 20),
    ("ell_c64_block16", lambda: bilayer(9, disorder_w=1.0, seed=3), 1, 1, 16, 20),
    ("patch_pairs", lambda: graphene(41, 37, disorder_w=1.0, seed=2), 0, 3, 1, 20),
    ("patch_pairs_another_cycle", lambda: graphene(41, 37, disorder_w=1.0, seed=2), 0, 3, 1, 18),
    ("block_pairs", lambda: bilayer(23, disorder_w=1.0, seed=3), 1, 3, 8, 20),
]


@pytest.mark.parametrize("name,make,dtype,fmt,block,M", GRAPHS, ids=[c[0] for c in GRAPHS])
def test_replayed_steps_are_bitwise_eager(T, ctx, orc, name, make, dtype, fmt, block, M):
    """Steps replayed from graphs (several replays, eager work between them) against
    the launches one by one, on the term and pair kernels."""
    eps = _eps(orc, M)
    lat, nt = make(), 25
    ham = ctx.build(lat, dtype=dtype, fmt=fmt)

    def run(mode):
        T.tbpm_ctx_set_graphs(ctx.handle, mode)
        before = T.tbpm_ctx_graph_replays(ctx.handle)
        out, launches = _timed(T, ctx, ham, 9.0, nt, block, block, 4, eps)
        assert launches >= nt * (M - 2) // 2 and launches <= nt * (M - 1)
        return out, T.tbpm_ctx_graph_replays(ctx.handle) - before

    try:
        eager, n0 = run(0)
        assert n0 == 0
        for _ in range(3):
            graph, n1 = run(2)
            assert n1 == nt // 6
            assert np.array_equal(graph["corr"], eager["corr"])
            assert np.array_equal(graph["norms"], eager["norms"])
            p, _ = T.make_params(9.0, 7, 1, seed=9)
            T.tbpm_propagate_dos(ctx.handle, ham, p)
    finally:
        T.tbpm_ctx_set_graphs(ctx.handle, 1)
        T.tbpm_ham_destroy(ham)
    per = orc.corr_dos(lat, rescale=9.0, num_steps=nt, num_vectors=block, seed=4, eps=eps)[1]
    assert np.abs(eager["corr"] - per).max() <= (1e-10 if dtype == 0 else 1e-5)
