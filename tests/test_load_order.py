"""The order in which inputs are loaded when GPU memory does not prescribe one, on the CPU (the fake GPU of test_dispatch): a grid of products
whose serial order wants the first rows, every column and then the other rows."""
import pytest

from paper_2405_16283_amd import binding as B

from test_dispatch import Session, fake  # noqa: F401  (fixture)

N, ROWS, COLS = 512, 8, 8


def _grid(fake, cap):
    """ROWS x COLS products of fp32 tiles; (session, vertices of the row tiles, of the column tiles)."""
    tg = B.tn_taskgraph_create()
    x = [B.tn_taskgraph_add_input(tg, B.TN_F32, N, N, B.TN_HOST) for _ in range(ROWS)]
    w = [B.tn_taskgraph_add_input(tg, B.TN_F32, N, N, B.TN_HOST) for _ in range(COLS)]
    for i in range(ROWS):
        for j in range(COLS):
            v = B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, B.tn_op_params(nk=1, trans_b=1), [x[i], w[j]], B.TN_F32, N, N)
            B.tn_taskgraph_mark_output(tg, v)
    return Session(fake, tg, cap), x, w


def _loaded(s):
    """Input vertices in the order of their loads."""
    out = []
    for m in B.tn_executor_last_order(s.ex, s.stats.n_vertices):
        v = B.tn_memgraph_vertex(s.mg, m)
        if v.kind == B.TN_MG_LOAD:
            out.append(v.src)
    return out


@pytest.mark.parametrize("seed", [0, 1])
def test_rows_and_columns_take_turns_where_there_is_room(fake, seed):  # noqa: F811
    s, x, w = _grid(fake, 160 * N * N * 4)
    try:
        want, _, _ = s.run(policy=B.TN_POLICY_IN_ORDER, max_batch=1, max_transfers=1)
        assert _loaded(s) == [x[0]] + w + x[1:]
        got, _, _ = s.run(seed, policy=B.TN_POLICY_BY_ORDER, max_transfers=1)
        order = _loaded(s)
        assert got == want and sorted(order) == sorted(x + w)
        for k in range(2, ROWS + COLS):  # neither side is more than two ahead until one has arrived
            here = set(order[:k])
            a, b = len(here & set(x)), len(here & set(w))
            assert abs(a - b) <= 2 or a == ROWS or b == COLS
    finally:
        s.close()


def test_the_serial_order_stays_where_loads_wait_for_memory(fake):  # noqa: F811
    s, x, w = _grid(fake, 14 * N * N * 4)
    try:
        want, _, _ = s.run(policy=B.TN_POLICY_IN_ORDER, max_batch=1, max_transfers=1)
        serial = _loaded(s)
        assert len(serial) >= ROWS + COLS
        got, _, _ = s.run(1, policy=B.TN_POLICY_BY_ORDER, max_transfers=1)
        assert got == want and _loaded(s)[:8] == serial[:8]
    finally:
        s.close()
