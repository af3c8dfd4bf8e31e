"""Which kernel a bf16 product goes to, by its shape alone, on the CPU (the fake GPU of test_dispatch).  Its bits depend on it, so the size
of a launch does not."""
import pytest

from paper_2405_16283_amd import binding as B

from test_dispatch import KERNEL, Session, fake  # noqa: F401  (fixture)

SMALL, TILES_128 = 1, 3  # LaunchClass


def _class(fake, m, n, k, mode, copies):  # noqa: F811
    tg = B.tn_taskgraph_create()
    shapes = [(m, k), (n, k)] + [(m, n)] * (mode == 1) + [(n, k)] * (mode == 2)
    ins = [B.tn_taskgraph_add_input(tg, B.TN_BF16, r, c, B.TN_DEVICE) for r, c in shapes]
    for _ in range(copies):
        B.tn_taskgraph_mark_output(tg, B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, B.tn_op_params(nk=1, trans_b=1, mode=mode), ins, B.TN_BF16, m, n))
    s = Session(fake, tg, sum(r * c * 2 + 512 for r, c in shapes) + copies * (m * n * 2 + 512))
    try:
        _, _, log = s.run(max_batch=copies)
        return set(int(x) for x in log[log.kind == KERNEL].detail)
    finally:
        s.close()


@pytest.mark.parametrize("m,n,k,mode,small", [
    (33, 512, 4096, 1, True), (63, 1024, 512, 1, True), (64, 512, 4096, 1, False), (63, 1032, 512, 1, False),
    (48, 512, 4096, 0, False), (48, 512, 4096, 2, False),
    (64, 512, 4104, 1, True), (127, 1024, 504, 1, True), (128, 512, 4104, 1, False), (96, 512, 4104, 0, False), (96, 512, 4104, 2, False),
    (32, 512, 4096, 0, True), (64, 128, 4096, 2, True), (64, 136, 4096, 0, False), (512, 32, 64, 1, True),
])
def test_small_products(fake, m, n, k, mode, small):  # noqa: F811
    for copies in (1, 3):
        got = _class(fake, m, n, k, mode, copies)
        assert got == ({SMALL} if small else {TILES_128})
