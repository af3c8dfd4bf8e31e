"""Tile products of the kernels made for small tiles, at the edges of their 32x32 workgroups, of their pieces
along K and of the shares of their four wavefronts, over every layout of the GEMM vertex, against float64.
Tolerance: products summed in fp32 differ from float64 by less than K 2^-24 of the sum of their magnitudes, and for
random operands by far less than K 2^-24 of the result in the 2-norm; a bf16 result adds half a unit of 2^-8."""
import numpy as np
import pytest
import torch

from oracle import llama_ref as R
from oracle import tiled as T
from paper_2405_16283_amd import binding as B

from test_gpu_backward_ops import Graph

pytestmark = pytest.mark.gpu


def _product(dtype, m, n, ks, ta=0, tb=1, tc=0, mode=0):
    print(f"[case] gemm {dtype} {m}x{n} K {ks} trans {ta}{tb}{tc} mode {mode}", flush=True)
    rng = np.random.default_rng(m * 1000 + n + sum(ks))
    g = Graph(dtype)
    scale = 1.0 / np.sqrt(sum(ks))
    a = [g.inp(rng.standard_normal((k, m) if ta else (m, k))) for k in ks]
    b = [[g.inp(rng.standard_normal((n, k) if tb else (k, n)) * scale) for k in ks] for _ in range(2 if mode == 2 else 1)]
    extra = [g.inp(rng.standard_normal((m, n)))] if mode == 1 else []
    ins = a + sum(b, []) + extra
    p = dict(nk=len(ks), trans_a=ta, trans_b=tb, trans_c=tc, mode=mode)
    v = g.op(B.TN_OP_GEMM, [i[0] for i in ins], n if tc else m, m if tc else n, **p)
    (got,) = g.run([v])
    wide = [i[1].T if ta and q < len(ks) else i[1] for q, i in enumerate(ins)]  # the oracle holds A plain
    ref = T._eval_vertex("gemm", p, wide)
    err = R.rel_err(got, ref)
    bound = sum(ks) * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    print(f"  rel err {err:.2e} (bound {bound:.1e})", flush=True)
    assert np.isfinite(got).all() and err < bound


F32 = [
    ((1, 1, [1]), {}), ((32, 32, [32]), {}), ((33, 31, [36, 4]), {}), ((64, 64, [64, 64, 64, 64]), {}),
    ((40, 72, [96, 128, 20]), {}), ((31, 65, [35, 7]), {}),         # rows along K not aligned to four elements
    ((256, 192, [256, 256]), {}), ((70, 45, [672]), {}),            # 21 pieces: five and six per wavefront
    ((16, 64, [33, 64]), dict(ta=1)), ((50, 34, [64, 40]), dict(ta=1, tb=0)), ((35, 66, [70]), dict(tb=0)),
    ((64, 37, [64, 32]), dict(tc=1)), ((37, 64, [416]), dict(ta=1, tb=0, tc=1)),
    ((33, 40, [64, 16]), dict(mode=1)), ((40, 33, [224]), dict(mode=2)),
    # single rows stored as columns
    ((1, 100, [64, 40]), dict(ta=1)), ((1, 36, [512]), dict(tc=1)), ((1, 65, [96, 8]), dict(ta=1, tc=1)), ((1, 33, [30]), dict(ta=1)),
]


@pytest.mark.parametrize("shape,kw", F32)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_any_layout_with_fp32_products(dtype, shape, kw):
    """(bf16 with both operands along K, in multiples of eight, goes to the kernels with bf16 products.)"""
    _product(dtype, *shape, **kw)


BF16 = [
    ((16, 512, [512, 512]), {}), ((512, 16, [256, 8]), {}), ((33, 31, [64, 24]), {}), ((64, 128, [200]), {}),
    ((20, 300, [1344]), {}), ((70, 30, [64, 64]), dict(tc=1)), ((65, 64, [136]), dict(mode=1)), ((40, 100, [72]), dict(mode=2)),
]


@pytest.mark.parametrize("shape,kw", BF16)
def test_small_and_thin_bf16_products(shape, kw):
    _product("bf16", *shape, **kw)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,n,ks,mode", [(1, 64, [64], 0), (33, 100, [512, 512, 40], 0), (32, 34, [64] * 9, 1),
                                            (70, 48, [128, 8], 2), (5, 256, [1024, 1024], 0)])
def test_single_rows_formed_together(dtype, rows, n, ks, mode):
    """`rows` single-row vertices, all but the last against one set of B tiles (70: three groups), the last against its own."""
    print(f"[case] rows {dtype} {rows} n {n} K {ks} mode {mode}", flush=True)
    rng = np.random.default_rng(rows + n)
    g = Graph(dtype)
    sets = 2 if mode == 2 else 1
    b = [[g.inp(rng.standard_normal((n, k)) / np.sqrt(sum(ks))) for _ in range(sets) for k in ks] for _ in range(2)]
    p = dict(nk=len(ks), trans_b=1, mode=mode)
    outs, refs = [], []
    for r in range(rows):
        own = b[1 if r + 1 == rows and rows > 1 else 0]
        ins = [g.inp(rng.standard_normal((1, k))) for k in ks] + own + ([g.inp(rng.standard_normal((1, n)))] if mode == 1 else [])
        outs.append(g.op(B.TN_OP_GEMM, [i[0] for i in ins], 1, n, **p))
        refs.append(T._eval_vertex("gemm", p, [i[1] for i in ins]))
    got = np.concatenate(g.run(outs))
    err = R.rel_err(got, np.concatenate(refs))
    bound = sum(ks) * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    print(f"  rel err {err:.2e} (bound {bound:.1e})", flush=True)
    assert np.isfinite(got).all() and err < bound


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_more_single_rows_than_one_launch_names(dtype):
    """1200 vertices against 801 sets of B, all ready at once: starts of groups and vertices together pass what a launch holds (1920).
    Sums of eight products: the bound of the other tests."""
    print(f"[case] 1200 rows, 801 sets of B, {dtype}", flush=True)
    n_b, n_rows, k, n = 801, 1200, 8, 12
    kind, code = (torch.float32, B.TN_F32) if dtype == "f32" else (torch.bfloat16, B.TN_BF16)
    gen = torch.Generator().manual_seed(5)
    a, b = torch.randn((16, k), generator=gen).to(kind), torch.randn((n_b, n, k), generator=gen).to(kind)
    tg = B.tn_taskgraph_create()
    va = [B.tn_taskgraph_add_input(tg, code, 1, k, B.TN_DEVICE) for _ in range(len(a))]
    vb = [B.tn_taskgraph_add_input(tg, code, n, k, B.TN_DEVICE) for _ in range(n_b)]
    of = [r if r < n_b else r % 7 * 100 for r in range(n_rows)]  # groups of one row and of fifty and more
    for r in range(n_rows):
        v = B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, B.tn_op_params(nk=1, trans_b=1), [va[r % 16], vb[of[r]]], code, 1, n)
        B.tn_taskgraph_mark_output(tg, v)
    cap = 4 << 20
    mg = B.tn_compile(tg, None, cap, None)
    dev = torch.empty(cap, dtype=torch.uint8, device="cuda:0")
    da, db = a.cuda(), b.cuda()
    out = torch.zeros((n_rows, 64), dtype=kind).pin_memory()
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(3)]
    ex = B.tn_executor_create(mg, dev.data_ptr(), cap, 0, 0, [st[0].cuda_stream], st[1].cuda_stream, st[2].cuda_stream)
    try:
        ins = [0] * B.tn_taskgraph_num_vertices(tg)
        for v, t in list(zip(va, da)) + list(zip(vb, db)):
            ins[v] = t.data_ptr()
        B.tn_executor_place_inputs(ex, ins)
        rep = B.tn_execute(ex, ins, [o.data_ptr() for o in out], B.tn_exec_opts(policy=B.TN_POLICY_RANDOM, max_batch=1920))
        assert rep.n_kernel_launches == 1  # one group, more than one launch
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(tg)
    ref = torch.stack([b[of[r]].double() @ a[r % 16].double() for r in range(n_rows)]).numpy()
    err = R.rel_err(out[:, :n].double().numpy(), ref)
    print(f"  rel err {err:.2e}", flush=True)
    assert err < k * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
