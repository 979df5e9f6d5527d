"""The autotuner times what a call runs: its microseconds per vector and term are those
of the call with that block width, whichever kernels it takes."""
import time

import numpy as np
import pytest

from tb_inputs import graphene
from tb_inputs.lattices import cell_by_name, supercell

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


CASES = [
    # several products per launch take 0.7 us a term and vector of 8,192 rows, terms one by one 2.9
    ("ell_tiles", lambda: graphene(64), 2, 0, 1),
    ("ell_tiles_blocks", lambda: graphene(64), 2, 1, 4),
    ("csr_tiles", lambda: supercell(cell_by_name("graphene"), 61, 47, vacancy_p=0.2, seed=3), 2, 0, 1),
    ("csr_terms", lambda: graphene(64), 0, 0, 4),
    ("patch_tiles", lambda: graphene(192, disorder_w=1.0, seed=2), 2, 0, 1),
]


@pytest.mark.parametrize("name,make,fmt,dtype,max_block", CASES, ids=[c[0] for c in CASES])
def test_times_are_a_calls(T, ctx, name, make, fmt, dtype, max_block):
    lat, nt = make(), 600
    ham = ctx.build(lat, dtype=dtype, fmt=fmt)
    try:
        r = T.tbpm_autotune(ctx.handle, ham, max_block)
        p, _ = T.make_params(9.0, nt, r["block"], block=r["block"], seed=3)
        T.tbpm_propagate_dos(ctx.handle, ham, p)
        took = []
        for _ in range(3):
            t = time.perf_counter()
            T.tbpm_propagate_dos(ctx.handle, ham, p)
            took.append(time.perf_counter() - t)
    finally:
        T.tbpm_ham_destroy(ham)
    call = min(took) * 1e6 / (nt * (T.tbpm_coefficients(np.pi).size - 1) * r["block"])
    # the call has its ends besides, the autotuner a few steps only: a factor of two either way
    assert 0.5 * call <= r["us_per_vector_term"] <= 2.0 * call


def test_tuning_leaves_results_and_memory(T, ctx):
    """Nothing stays allocated, and results are those without tuning up to rounding."""
    lat = graphene(24, 20, disorder_w=1.0, seed=12)
    p, _ = T.make_params(9.0, 20, 5, seed=3)
    for fmt in (0, 1, 3):
        ham = ctx.build(lat, fmt=fmt)
        try:
            before = T.tbpm_propagate_dos(ctx.handle, ham, p)["corr"]
            live = ctx.allocator.live_bytes
            r = T.tbpm_autotune(ctx.handle, ham, 64)
            assert ctx.allocator.live_bytes == live
            assert r["block"] in (1, 2, 4, 8, 16, 32, 64)
            after = T.tbpm_propagate_dos(ctx.handle, ham, p)["corr"]
        finally:
            T.tbpm_ham_destroy(ham)
        assert np.abs(after - before).max() <= 1e-10
