"""Tensors around and beyond 4 GiB, where byte offsets come close to what 32 bits hold: copies inside GPU memory, and products."""
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


@pytest.mark.parametrize("rows", [32768 - 128, 32768 + 128])
def test_a_tensor_near_4_gib_is_copied_whole(rows):
    """16 MiB below 4 GiB, where a workgroup's last step along the tensor leads past 4 GiB, and 16 MiB above."""
    print(f"[case] copy inside GPU memory of {rows} x {COLS} fp32", flush=True)
    got = _row_statistics(rows)
    # sums of 32768 equal squares in fp32, a division and a square root
    assert np.allclose(got, 1.0 / np.arange(1, rows + 1), rtol=1e-5, atol=0)


PRODUCTS = [
    # dtype, m, n, k, trans_a, trans_b: which operand passes 4 GiB, or 32 bits of bytes from one element to another
    ("f32", 33000, 16, 32768, 0, 1),      # A
    ("f32", 16, 33000, 32768, 0, 0),      # B, stored [K, n]
    ("bf16", 66000, 16, 32768, 0, 1),     # A, bf16 products
    ("bf16", 66000, 128, 32768, 0, 1),    # A, tiles of 128x128
    ("bf16", 128, 66000, 32768, 0, 1),    # B
    ("bf16", 66000, 256, 32776, 0, 1),    # A, K no multiple of the chunks along it
    ("bf16", 66000, 520, 32768, 0, 1),    # A, tiles of 256x256
    ("bf16", 257, 256, (1 << 23) - 8, 0, 1),  # 257 rows along K, the deepest that these kernels take
    ("bf16", 72, 128, (1 << 23) + 8, 0, 1),   # deeper
    ("f32", 1, 33000, 32768, 0, 1),       # B of a single row
    ("bf16", 1, 66000, 32768, 0, 1),
    ("f32", 33, 1, (1 << 25) + 64, 0, 1),  # 32 rows along K
    ("f32", 84 << 20, 1, 32, 1, 1),        # rows of A stored [K, m]
]


@pytest.mark.parametrize("dtype,m,n,k,ta,tb", PRODUCTS)
def test_products_of_operands_beyond_4_gib(dtype, m, n, k, ta, tb):
    """Operands that lie in GPU memory; the first and last rows and columns of the result against float64."""
    print(f"[case] gemm {dtype} {m}x{n} K {k} trans {ta}{tb}", flush=True)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    code = B.TN_F32 if dtype == "f32" else B.TN_BF16
    gen = torch.Generator(device="cuda:0").manual_seed(m + n)
    shapes = [(k, m) if ta else (m, k), (n, k) if tb else (k, n)]
    a, b = (torch.empty(s, dtype=kind, device="cuda:0").normal_(generator=gen) for s in shapes)
    tg = B.tn_taskgraph_create()
    ins = [B.tn_taskgraph_add_input(tg, code, r, c, B.TN_DEVICE) for r, c in shapes]
    v = B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, B.tn_op_params(nk=1, trans_a=ta, trans_b=tb), ins, code, m, n)
    B.tn_taskgraph_mark_output(tg, v)
    cap = (a.numel() + b.numel() + m * n) * a.element_size() + (1 << 20)
    mg = B.tn_compile(tg, None, cap, None)
    dev = torch.empty(cap, dtype=torch.uint8, device="cuda:0")
    out = torch.zeros((m, n), dtype=kind, device="cuda:0")
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(3)]
    ex = B.tn_executor_create(mg, dev.data_ptr(), cap, 0, 0, [st[0].cuda_stream], st[1].cuda_stream, st[2].cuda_stream)
    try:
        B.tn_executor_place_inputs(ex, [a.data_ptr(), b.data_ptr(), 0])
        B.tn_execute(ex, [0, 0, 0], [out.data_ptr()], B.tn_exec_opts(small_gemm_tiles=-1 if k >> 22 else 0))  # (-1: 256 rows to a workgroup)
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(tg)
    del dev
    pick = lambda n: torch.tensor(sorted(set(range(min(n, 8))) | set(range(max(0, n - 40), n))), device="cuda:0")
    rows, cols = pick(m), pick(n)
    x = (a[:, rows].T if ta else a[rows]).double().contiguous()
    y = (b[cols].T if tb else b[:, cols]).double().contiguous()
    ref = x @ y
    got = out[rows][:, cols].double()
    err = ((got - ref).norm() / ref.norm()).item()
    # a sum of k products in fp32 is off by less than k 2^-24 of the sum of their magnitudes, and for random signs by
    # far less than that of the result (sqrt(k) of its terms); a bf16 result adds half a unit of 2^-8
    bound = min(k * 2.0 ** -24, 1e-3) + (2.0 ** -8 if dtype == "bf16" else 0.0)
    print(f"  rel err {err:.2e} (bound {bound:.1e})", flush=True)
    del a, b, x, y, out
    torch.cuda.empty_cache()
    assert err < bound
