"""Tensors around 4 GiB: copies inside GPU memory whose byte offsets come close to what 32 bits hold."""
import numpy as np
import pytest
import torch

from paper_2405_16283_amd import binding as B

pytestmark = pytest.mark.gpu

COLS = 32768


def _row_statistics(rows):
    """rows x 32768 fp32, loaded from a buffer in GPU memory, row i holding i + 1 throughout: its RMSNorm statistic is
    1 / (i + 1) if every piece of the row arrived."""
    tg = B.tn_taskgraph_create()
    x = B.tn_taskgraph_add_input(tg, B.TN_F32, rows, COLS, B.TN_HOST)
    stat = B.tn_taskgraph_add_op(tg, B.TN_OP_RMS_STAT, B.tn_op_params(d=COLS, eps=0.0), [x], B.TN_F32, rows, 1)
    B.tn_taskgraph_mark_output(tg, stat)
    cap = rows * COLS * 4 + (1 << 20)
    mg = B.tn_compile(tg, None, cap, None)
    dev = torch.full((cap,), 0xFF, dtype=torch.uint8, device="cuda:0")  # what does not arrive is NaN
    src = torch.arange(1, rows + 1, dtype=torch.float32, device="cuda:0").repeat_interleave(COLS)
    out = torch.zeros(rows, dtype=torch.float32).pin_memory()
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(3)]
    ex = B.tn_executor_create(mg, dev.data_ptr(), cap, 0, 0, [st[0].cuda_stream], st[1].cuda_stream, st[2].cuda_stream)
    try:
        B.tn_execute(ex, [src.data_ptr(), 0], [out.data_ptr()], None)
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(tg)
    return out.numpy()


@pytest.mark.parametrize("rows", [32768 - 128])
def test_a_tensor_near_4_gib_is_copied_whole(rows):
    """16 MiB below 4 GiB, where a workgroup's last step along the tensor leads past 4 GiB."""
    print(f"[case] copy inside GPU memory of {rows} x {COLS} fp32", flush=True)
    got = _row_statistics(rows)
    # sums of 32768 equal squares in fp32, a division and a square root
    assert np.allclose(got, 1.0 / np.arange(1, rows + 1), rtol=1e-5, atol=0)
