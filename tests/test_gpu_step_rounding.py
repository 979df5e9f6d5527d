"""Complex64 vectors by tiles in several launches a time step: the series is stored
between them, and what a later launch adds must not lie below its last place as a whole.

H's values are exact in 32 bits and the rescale a power of two, the initial states are
rounded beforehand, so only the steps' own rounding counts, which is random from row to
row: C(t) averaged over the vectors.  Tolerance: a launch's 2^-25 of unit modulus at most,
20 terms and launches a step at most, 8 steps, n rows and R vectors at random:
2^-25 sqrt(20 * 8 / (n R)) = 1.9e-9 as a standard deviation's bound, five times that, and
the terms that 7 + 7 products leave to the last launch, at most 1.3e-9 a step."""
import numpy as np
import pytest
from scipy.special import jv

from tb_inputs.lattices import honeycomb3_cell, supercell

pytestmark = pytest.mark.gpu


def test_last_launch_is_not_rounded_away(orc):
    from paper_2509_26309_amd import tbpm as T
    lat = supercell(honeycomb3_cell(-2.75, -0.25, -0.1875), 50, 51)
    rho, nt, R = 16.0, 8, 8
    psi = np.stack([orc.random_state(lat.n, 1, r) for r in range(R)]).astype(np.complex64).astype(np.complex128)
    with T.Context(0) as ctx:
        ham = ctx.build(lat, dtype=T.TBPM_C64, fmt=T.TBPM_FMT_ELL)
        try:
            plan = T.tbpm_ham_tiles(ham, 1)
            p, _ = T.make_params(rho, nt, R, block=1)
            got = T.tbpm_propagate_states(ctx.handle, ham, p, psi)["corr"]
        finally:
            T.tbpm_ham_destroy(ham)
    assert plan["products"] == 7                         # three launches for 19 products
    ref = np.stack([orc.propagate(lat, psi[r], rescale=rho, num_steps=nt).corr for r in range(R)])
    err = np.abs((got - ref).mean(axis=0))
    lost = sum(2 * abs(jv(m, np.pi)) for m in range(15, 20))
    k = np.arange(nt + 1)
    assert np.all(err <= 5 * 2.0 ** -25 * np.sqrt(20 * nt / (lat.n * R)) + k * lost), err
