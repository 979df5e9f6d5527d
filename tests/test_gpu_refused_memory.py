"""Device memory that is refused: a call that can do with less goes on and gives the
same results, one that cannot says so, and neither leaves an error behind for the
next call.

The contexts take their memory from an allocator that refuses chosen requests the
way a full device does: by a hipMalloc that fails, whose error the runtime keeps
until somebody reads it.
"""
import ctypes

import numpy as np
import pytest

from tb_inputs.lattices import cell_by_name, supercell
from tb_inputs import graphene, honeycomb3

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2509_26309_amd import tbpm
    return tbpm


class Refusing:
    """hipMalloc / hipFree behind the caller's allocator; `refuse(nbytes, live)` decides,
    `live` being the sizes that are held at the moment."""

    def __init__(self, T):
        hip = T.load()                           # symbols of the runtime that the library is linked to
        self.refuse = None
        self.live, self.requests, self.refused = {}, 0, 0

        def _alloc(nbytes, user):
            self.requests += 1
            no = self.refuse is not None and self.refuse(int(nbytes), list(self.live.values()))
            p = ctypes.c_void_p()
            rc = hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60 if no else int(nbytes)))
            assert (rc != 0) == no
            if no:
                self.refused += 1
                return None
            self.live[p.value] = int(nbytes)
            return p.value

        def _free(ptr, user):
            if ptr:
                self.live.pop(int(ptr))
                hip.hipFree(ctypes.c_void_p(int(ptr)))

        self._keep = (T.ALLOC_FN(_alloc), T.FREE_FN(_free))
        self.struct = T.tbpm_allocator(*self._keep, None)


@pytest.fixture
def env(T):
    a = Refusing(T)
    h = T.tbpm_ctx_create(0, a)
    yield h, a
    a.refuse = None
    T.tbpm_ctx_destroy(h)
    assert not a.live


def _build(T, h, lat, fmt, dtype=0):
    return T.tbpm_build_csr(h, lat.n, lat.row_ptr, lat.col, lat.val, dtype, fmt, 0)


def test_propagation_goes_on_with_the_vectors_of_the_term_kernels(T, env):
    """Several products per launch take five or six vectors here, single terms four."""
    h, a = env
    lat = honeycomb3(70, 60, vacancy_p=0.01, seed=5)
    ham = _build(T, h, lat, T.TBPM_FMT_ELL)
    try:
        p, _ = T.make_params(10.0, 13, 2, block=1, seed=6)
        T.tbpm_ctx_set_profiling(h, True)
        terms = T.tbpm_propagate_dos(h, ham, p)
        T.tbpm_ctx_set_profiling(h, False)
        a.refuse = lambda nbytes, live: nbytes == 16 * lat.n and live.count(nbytes) >= 4
        got = T.tbpm_propagate_dos(h, ham, p)
    finally:
        T.tbpm_ham_destroy(ham)
    assert a.refused == 1
    assert np.array_equal(got["corr"], terms["corr"]) and np.array_equal(got["norms"], terms["norms"])


@pytest.mark.parametrize("live", [0, 1, 2, 3])
def test_propagation_without_enough_memory_fails_alone(T, env, live):
    h, a = env
    lat = graphene(40, disorder_w=1.0, seed=1)
    ham = _build(T, h, lat, T.TBPM_FMT_ELL)
    try:
        p, _ = T.make_params(9.0, 13, 1, block=1, seed=6)
        ref = T.tbpm_propagate_dos(h, ham, p)
        a.refuse = lambda nbytes, held: nbytes == 16 * lat.n and held.count(nbytes) >= live
        with pytest.raises(T.TBPMError) as e:
            T.tbpm_propagate_dos(h, ham, p)
        assert e.value.status == T.TBPM_ERR_OOM
        a.refuse = None
        assert np.array_equal(T.tbpm_propagate_dos(h, ham, p)["corr"], ref["corr"])
    finally:
        T.tbpm_ham_destroy(ham)


def test_moments_go_on_with_the_vectors_of_the_product_kernels(T, env, orc):
    """Several products per launch take four vectors, single products two."""
    h, a = env
    lat = graphene(175, 29, disorder_w=1.0, seed=6)
    ham = _build(T, h, lat, T.TBPM_FMT_ELL)
    try:
        p, _ = T.make_params(9.0, 0, 1, seed=4)
        a.refuse = lambda nbytes, live: nbytes == 16 * lat.n and live.count(nbytes) >= 2
        mu = T.tbpm_chebyshev_moments(h, ham, p, 60)
    finally:
        T.tbpm_ham_destroy(ham)
    assert a.refused > 0
    ref = orc.moments(lat, orc.random_state(lat.n, 4, 0), rescale=9.0, num_moments=60)
    assert np.abs(mu[0] - ref).max() <= 1e-10


STORED = {
    "uneven_csr": (lambda: supercell(cell_by_name("graphene"), 61, 47, vacancy_p=0.2, seed=3), 2),
    "ell": (lambda: graphene(47, 33, disorder_w=1.0, seed=8), 1),
    "patch": (lambda: graphene(47, 33, disorder_w=1.0, seed=8), 3),
}


@pytest.mark.parametrize("name", list(STORED))
def test_every_refusal_while_h_is_stored(T, env, orc, name):
    """One allocation after the other is refused: H is stored without what is optional
    (the plan of tiles, a padded copy) and serves, or the call fails with nothing held."""
    h, a = env
    make, fmt = STORED[name]
    lat = make()
    p, _ = T.make_params(9.0, 4, 1, seed=3)
    per = orc.corr_dos(lat, rescale=9.0, num_steps=4, num_vectors=1, seed=3)[1]
    a.requests = 0
    T.tbpm_ham_destroy(_build(T, h, lat, fmt))
    total, optional = a.requests, 0
    for k in range(total):
        a.requests = a.refused = 0
        a.refuse = lambda nbytes, live: a.requests == k + 1
        try:
            ham = _build(T, h, lat, fmt)
        except T.TBPMError as e:
            assert e.status in (T.TBPM_ERR_OOM, T.TBPM_ERR_HIP), (k, e)
            assert "memory" in str(e) or e.status == T.TBPM_ERR_OOM, (k, e)
            a.refuse = None
            assert not a.live, k
            continue
        a.refuse = None
        assert a.refused == 1
        optional += 1
        try:
            got = T.tbpm_propagate_dos(h, ham, p)
        finally:
            T.tbpm_ham_destroy(ham)
        assert np.abs(got["corr"] - per).max() <= 1e-10, k
    assert optional >= 4                        # the plan's arrays, at least
