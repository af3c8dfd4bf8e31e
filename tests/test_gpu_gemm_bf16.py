"""Tile products with bf16 operands in all forms in which they are launched (256x256 per workgroup, 128x128 with one or two
workgroups per CU), at the edges of their tiles, of their chunks of 64 along K and of their rings of chunks, against float64.
Tolerance: products summed in fp32 differ from float64 by less than K 2^-24 of the sum of their magnitudes, and for random operands by
far less than K 2^-24 of the result in the 2-norm; a bf16 result adds half a unit of 2^-8.  The forms agree bit for bit."""
import numpy as np
import pytest
import torch

from oracle import llama_ref as R
from oracle import tiled as T
from paper_2405_16283_amd import binding as B

from test_gpu_backward_ops import Graph

pytestmark = pytest.mark.gpu


def _run_forms(g, outs, forms):
    """[results as bf16 bits, one array per output] for every value of the option small_gemm_tiles."""
    shapes = []
    for v in outs:
        B.tn_taskgraph_mark_output(g.tg, v)
        x = B.tn_taskgraph_vertex(g.tg, v)
        shapes.append((x.desc.rows, x.desc.cols))
    n = B.tn_taskgraph_num_vertices(g.tg)
    cap = 256 << 20
    mg = B.tn_compile(g.tg, None, cap, None)
    dev = torch.empty(cap, dtype=torch.uint8, device="cuda:0")
    st = [torch.cuda.Stream() for _ in range(3)]
    bufs = [torch.zeros(r * c, dtype=torch.int16).pin_memory() for r, c in shapes]
    ex = B.tn_executor_create(mg, dev.data_ptr(), cap, 0, 0, [st[0].cuda_stream], st[1].cuda_stream, st[2].cuda_stream)
    res = []
    try:
        ptrs = [g.host[v].data_ptr() if v in g.host else 0 for v in range(n)]
        for f in forms:
            for b in bufs:
                b.zero_()
            B.tn_execute(ex, ptrs, [b.data_ptr() for b in bufs], B.tn_exec_opts(policy=B.TN_POLICY_FIFO, small_gemm_tiles=f))
            res.append([b.numpy().view(np.uint16).reshape(s).copy() for b, s in zip(bufs, shapes)])
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(g.tg)
    return res


def _wide(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


# rows, columns of the product, K of its tiles, parameters
CASES = [
    ((256, 256, [64]), {}), ((256, 256, [128, 128]), {}),             # one chunk (and one of zeros), two
    ((256, 256, [64] * 7), {}), ((256, 256, [64] * 16), {}),          # rings filled once, three pairs of chunks
    ((257, 300, [72, 8]), {}), ((511, 513, [40]), {}), ((300, 520, [512, 512, 40]), {}), ((260, 260, [8]), {}),
    ((384, 288, [384, 384, 384, 288]), {}), ((290, 270, [520, 72, 520]), {}),
    ((256, 384, [192, 96]), dict(tc=1)), ((300, 259, [136]), dict(tc=1)),
    ((300, 271, [264]), dict(mode=1)), ((257, 512, [512, 64]), dict(mode=1)),
    ((270, 260, [200]), dict(mode=2)), ((512, 384, [512, 32]), dict(mode=2)),
    ((128, 128, [64, 64]), {}), ((129, 127, [1000]), {}), ((347, 128, [512, 136]), {}), ((100, 130, [24]), dict(mode=2)),
    ((100, 90, [72]), dict(mode=1)), ((255, 700, [88]), dict(tc=1)),  # less than 256 one way: 128x128 always
    ((2100, 2200, [136]), {}),                                        # 306 workgroups of 128x128: two per CU
]


@pytest.mark.parametrize("shape,kw", CASES)
def test_forms_agree_with_float64_and_each_other(shape, kw):
    m, n, ks = shape
    tc, mode = kw.get("tc", 0), kw.get("mode", 0)
    print(f"[case] gemm bf16 {m}x{n} K {ks} transposed {tc} mode {mode}", flush=True)
    rng = np.random.default_rng(m * 1000 + n + sum(ks))
    g = Graph("bf16")
    a = [g.inp(rng.standard_normal((m, k))) for k in ks]
    b = [[g.inp(rng.standard_normal((n, k)) / np.sqrt(sum(ks))) for k in ks] for _ in range(2 if mode == 2 else 1)]
    extra = [g.inp(rng.standard_normal((m, n)))] if mode == 1 else []
    ins = a + sum(b, []) + extra
    p = dict(nk=len(ks), trans_b=1, trans_c=tc, mode=mode)
    v = g.op(B.TN_OP_GEMM, [i[0] for i in ins], n if tc else m, m if tc else n, **p)
    forms = _run_forms(g, [v], (0, -1, 1 << 20))
    ref = T._eval_vertex("gemm", dict(p, trans_a=0), [i[1] for i in ins])
    err = R.rel_err(_wide(forms[0][0]), ref)
    bound = sum(ks) * 2.0 ** -24 + 2.0 ** -8
    print(f"  rel err {err:.2e} (bound {bound:.1e})", flush=True)
    assert np.isfinite(_wide(forms[0][0])).all() and err < bound
    for other in forms[1:]:
        assert np.array_equal(forms[0][0], other[0])


@pytest.mark.parametrize("form", [0, -1, 1 << 20])
def test_what_lies_behind_the_end_of_a_row_is_not_multiplied(form):
    """K of 40 and 72 in chunks of 64: the elements behind a row's end are the next row's, here infinite, and those of another tensor."""
    print(f"[case] infinite rows, small_gemm_tiles {form}", flush=True)
    rng = np.random.default_rng(7)
    ks, m, n = [40, 72], 300, 280
    g = Graph("bf16")
    full = [rng.standard_normal((m, k)) for k in ks]
    for x in full:
        x[1::3] = np.inf
    ins = [g.inp(x) for x in full] + [g.inp(rng.standard_normal((n, k))) for k in ks]
    v = g.op(B.TN_OP_GEMM, [i[0] for i in ins], m, n, nk=len(ks), trans_b=1)
    got = _wide(_run_forms(g, [v], (form,))[0][0])
    keep = np.ones(m, bool)
    keep[1::3] = False
    ref = sum(ins[q][1][keep] @ ins[q + len(ks)][1].T for q in range(len(ks)))
    assert R.rel_err(got[keep], ref) < sum(ks) * 2.0 ** -24 + 2.0 ** -8
    assert not np.isfinite(got[1::3]).any()


def test_products_of_different_shapes_share_a_launch():
    """Ragged vertices of one launch take fewer workgroups than its largest."""
    print("[case] six shapes in one launch", flush=True)
    rng = np.random.default_rng(9)
    g = Graph("bf16")
    k, outs, refs = 192, [], []
    for m, n in [(256, 256), (700, 300), (259, 520), (512, 256), (300, 300), (256, 1000)]:
        a, b = g.inp(rng.standard_normal((m, k))), g.inp(rng.standard_normal((n, k)) / np.sqrt(k))
        outs.append(g.op(B.TN_OP_GEMM, [a[0], b[0]], m, n, nk=1, trans_b=1))
        refs.append(a[1] @ b[1].T)
    for res in _run_forms(g, outs, (0, -1, 1 << 20)):
        for got, ref in zip(res, refs):
            assert R.rel_err(_wide(got), ref) < k * 2.0 ** -24 + 2.0 ** -8
