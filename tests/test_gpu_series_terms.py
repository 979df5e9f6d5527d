"""When the series takes its terms: a launch holds the newest terms of its rows,
so out is brought up to date only where the next launch could no longer do it.
Every length M of the series is another pattern of such launches; each is
checked against the oracle's one update per term.

Tolerances as in test_gpu_parity: 1e-10 (complex128) and 1e-5 (complex64) on
C(t_k); the number of steps is small, so the bounds on rounding that they were
derived from hold with room to spare.
"""
import numpy as np
import pytest
from scipy.special import jv

from tb_inputs import graphene, honeycomb3, bilayer

pytestmark = pytest.mark.gpu

CASES = [
    # (name, lattice maker, rho, dtype, format, R, block)
    ("csr_c128", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 9.0, 0, 0, 1, 1),
    ("ell_c128_block4", lambda: graphene(13, 11, disorder_w=1.0, seed=5), 9.0, 0, 1, 4, 4),
    ("ell_c64_block2", lambda: graphene(17, 12, disorder_w=1.0, seed=6), 9.0, 1, 1, 2, 2),
    ("patch_c128", lambda: graphene(41, 37, disorder_w=1.0, seed=7), 9.0, 0, 3, 1, 1),
    ("patch_c64_pairs_block8", lambda: bilayer(23, 21, disorder_w=1.0, seed=8), 9.0, 1, 3, 8, 8),
    ("patch_c64_staged_block16", lambda: honeycomb3(33, 31, vacancy_p=0.01, seed=9), 10.0, 1, 3, 16, 16),
]


@pytest.fixture(scope="module")
def T():
    from paper_2509_26309_amd import tbpm
    return tbpm


@pytest.fixture(scope="module")
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("M", [4, 5, 6, 7, 8, 9, 10, 12, 15, 18, 20])
@pytest.mark.parametrize("name,make,rho,dtype,fmt,R,block", CASES, ids=[c[0] for c in CASES])
def test_every_series_length(T, ctx, orc, name, make, rho, dtype, fmt, R, block, M):
    eps = 1.0001 * abs(jv(M, np.pi))
    assert orc.coefficients(np.pi, eps).size == M
    lat = make()
    nt = 5
    ham = ctx.build(lat, dtype=dtype, fmt=fmt)
    try:
        assert T.tbpm_ham_info(ham)["format"] == fmt
        p, _ = T.make_params(rho, nt, R, block=block, seed=3, bessel_eps=eps)
        out = T.tbpm_propagate_dos(ctx.handle, ham, p)
    finally:
        T.tbpm_ham_destroy(ham)
    _, per, norms, _ = orc.corr_dos(lat, rescale=rho, num_steps=nt, num_vectors=R, seed=3, eps=eps)
    tol = 1e-10 if dtype == 0 else 1e-5
    assert np.abs(out["corr"] - per).max() <= tol
    assert np.abs(out["norms"] - norms).max() <= tol
