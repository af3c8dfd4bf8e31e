"""The room in LDS that launches of small products ask for: as many pieces along K as a wavefront of their deepest vertex takes, at most
four, on the CPU (the fake GPU of test_dispatch).  More than that keeps other workgroups off the compute unit."""
import ctypes as C

import pytest

from paper_2405_16283_amd import binding as B

from test_dispatch import Session, fake  # noqa: F401  (fixture)


def _launch(fake, vertices):  # noqa: F811
    """Stages of the one launch of products (dtype, m, n, depths, trans_a, trans_b)."""
    tg = B.tn_taskgraph_create()
    size = 0
    for dtype, m, n, ks, ta, tb in vertices:
        shapes = [(k, m) if ta else (m, k) for k in ks] + [(n, k) if tb else (k, n) for k in ks]
        ins = [B.tn_taskgraph_add_input(tg, dtype, r, c, B.TN_DEVICE) for r, c in shapes]
        B.tn_taskgraph_mark_output(tg, B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, B.tn_op_params(nk=len(ks), trans_a=ta, trans_b=tb), ins, dtype, m, n))
        size += sum(r * c * 4 + 512 for r, c in shapes + [(m, n)])
    s = Session(fake, tg, size)
    try:
        s.run()
        out = (C.c_int32 * 16)()
        assert fake.fake_stages(out, C.c_int64(16)) == 1
        return out[0]
    finally:
        s.close()


F, H = B.TN_F32, B.TN_BF16


@pytest.mark.parametrize("vertices,want", [
    ([(F, 64, 64, [32], 0, 1)], 1), ([(F, 64, 64, [128], 0, 1)], 1), ([(F, 64, 64, [132], 0, 1)], 1), ([(F, 64, 64, [160], 0, 1)], 2),
    ([(F, 64, 64, [64, 36, 384], 0, 1)], 4), ([(F, 64, 64, [4096], 0, 1)], 4),
    ([(F, 64, 64, [28], 0, 1)], 0),                                           # no whole piece
    ([(F, 64, 64, [1022], 0, 1)], 0),                                         # rows not aligned to four elements
    ([(F, 64, 64, [64], 0, 0)], 1), ([(F, 64, 64, [1024], 1, 0)], 4), ([(F, 64, 64, [1022], 1, 0)], 4), ([(F, 64, 64, [1022], 0, 0)], 0),
    ([(H, 64, 64, [256], 0, 1)], 1), ([(H, 64, 64, [512], 0, 1)], 2), ([(H, 64, 64, [8], 0, 1)], 0), ([(H, 64, 64, [4096], 0, 1)], 4),
    ([(H, 64, 64, [4096], 1, 1)], 0),                                         # bf16 storage, fp32 products: through registers
    ([(F, 1, 64, [256], 0, 1)], 2), ([(H, 1, 64, [256], 0, 1)], 1), ([(H, 1, 64, [64] * 64, 0, 1)], 4), ([(H, 1, 64, [64] * 65, 0, 1)], 0),
    ([(F, 64, 64, [32], 0, 1), (F, 32, 64, [288], 0, 1), (F, 64, 32, [1022], 0, 1)], 3),  # a launch takes its largest
])
def test_stages_follow_the_deepest_vertex(fake, vertices, want):  # noqa: F811
    fake.fake_stages.restype = C.c_int64
    assert _launch(fake, vertices) == want
