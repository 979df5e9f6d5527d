"""What a served request runs and holds is settled by the server: kernel timing, which
is for the synchronous calls, changes nothing about it, and a series mode that is
switched while the request waits is read at its start without the request taking more
than the budget holds."""
import time

import numpy as np
import pytest

from tb_inputs import graphene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2509_26309_amd import tbpm
    return tbpm


@pytest.fixture
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


def _wait(T, srv, ticket, R, nt, timeout=60.0):
    end = time.time() + timeout
    while (res := T.tbpm_poll(srv, ticket, R, nt))[0] == T.TBPM_PENDING:
        if time.time() > end:
            raise TimeoutError
        time.sleep(0.002)
    return res


def _queued_behind_another(T, ctx, budget, fmt, while_waiting):
    """One request that waits for a longer one on a single slot; `while_waiting` runs in between."""
    small, lat = graphene(10), graphene(96, disorder_w=1.0, seed=3)
    hs, ham = ctx.build(small), ctx.build(lat, fmt=fmt)
    p0, _ = T.make_params(9.0, 20000, 1, seed=1)
    p, _ = T.make_params(9.0, 25, 1, seed=2)
    srv = T.tbpm_server_create(ctx.handle, budget(ham, p), 1)
    try:
        first = T.tbpm_submit(srv, hs, p0)
        ticket = T.tbpm_submit(srv, ham, p)
        while_waiting()
        assert T.tbpm_poll(srv, first, 1, 20000)[0] == T.TBPM_PENDING     # it did wait
        try:
            return _wait(T, srv, ticket, 1, 25), ham, p
        finally:
            assert _wait(T, srv, first, 1, 20000)[0] == T.TBPM_OK
    finally:
        T.tbpm_server_destroy(srv)


@pytest.mark.parametrize("fmt", [1, 3])
def test_kernel_timing_is_not_for_served_requests(T, ctx, fmt):
    (st, corr, _, _), ham, p = _queued_behind_another(T, ctx, lambda h, q: 1 << 28, fmt,
                                                      lambda: T.tbpm_ctx_set_profiling(ctx.handle, True))
    T.tbpm_ctx_set_profiling(ctx.handle, False)
    assert st == T.TBPM_OK
    assert T.tbpm_ham_tiles(ham)["products"] > 0
    assert np.array_equal(corr, T.tbpm_propagate_dos(ctx.handle, ham, p)["corr"])


def _clenshaw_footprint(T, ctx, ham, p):
    T.tbpm_ctx_set_series(ctx.handle, T.TBPM_SERIES_CLENSHAW)
    try:
        return T.tbpm_footprint(ham, p)
    finally:
        T.tbpm_ctx_set_series(ctx.handle, T.TBPM_SERIES_FORWARD)


def test_series_mode_switched_while_waiting(T, ctx):
    """Clenshaw's pairs take more vectors here than the tiles that were admitted: with
    room for them the request runs them, as a lone call would."""
    (st, corr, _, _), ham, p = _queued_behind_another(
        T, ctx, lambda h, q: _clenshaw_footprint(T, ctx, h, q), 3,
        lambda: T.tbpm_ctx_set_series(ctx.handle, T.TBPM_SERIES_CLENSHAW))
    assert st == T.TBPM_OK
    assert np.array_equal(corr, T.tbpm_propagate_dos(ctx.handle, ham, p)["corr"])


def test_never_more_than_the_budget(T, ctx):
    """The same with a budget that holds the tiles' vectors alone: refused, not overdrawn."""
    seen = []

    def budget(h, q):
        seen.extend([T.tbpm_footprint(h, q), _clenshaw_footprint(T, ctx, h, q)])
        return seen[0]

    with pytest.raises(T.TBPMError) as e:
        _queued_behind_another(T, ctx, budget, 3, lambda: T.tbpm_ctx_set_series(ctx.handle, T.TBPM_SERIES_CLENSHAW))
    assert seen[1] > seen[0]
    assert e.value.status == T.TBPM_ERR_TOO_LARGE and "poll" in str(e.value)       # accepted, refused at its start


@pytest.mark.parametrize("cells,R,replays", [(12, 1, True), (512, 8, False)])
def test_chunks_are_whole_graphs_only_where_one_fits(T, ctx, cells, R, replays):
    """A chunk is about 300 us of device time, or one step: steps of a few microseconds
    are replayed in whole graphs, slow ones (eight vectors of 524,288 orbitals: more than
    150 us) are launched one by one, also where graphs are asked for at any size."""
    lat = graphene(cells, disorder_w=1.0, seed=3)
    ham = ctx.build(lat)
    p, _ = T.make_params(9.0, 24, R, block=R, seed=2)
    T.tbpm_ctx_set_graphs(ctx.handle, 2)
    before = T.tbpm_ctx_graph_replays(ctx.handle)
    srv = T.tbpm_server_create(ctx.handle, 8 << 30, 1)
    try:
        st, corr, _, _ = _wait(T, srv, T.tbpm_submit(srv, ham, p), R, 24)
    finally:
        T.tbpm_server_destroy(srv)
    assert st == T.TBPM_OK
    assert (T.tbpm_ctx_graph_replays(ctx.handle) > before) == replays
    assert np.array_equal(corr, T.tbpm_propagate_dos(ctx.handle, ham, p)["corr"])
