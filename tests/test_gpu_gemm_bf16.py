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


def _run_forms(g, outs, forms, one_launch=False):
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
            rep = B.tn_execute(ex, ptrs, [b.data_ptr() for b in bufs],
                               B.tn_exec_opts(policy=B.TN_POLICY_FIFO, small_gemm_tiles=f, max_batch=1920))
            assert rep.gemm_launches == 1 or not one_launch
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


# The same in launches of more than 256 workgroups of 128x128, two to a CU: chunks of one or two and of many, rings filled once and several
# times, K that changes inside the ring, every way to store.
PAIRED = [
    ((128, 128, [8]), {}), ((128, 128, [72]), {}), ((129, 130, [64] * 9), {}), ((256, 256, [64, 8, 72, 200, 24]), {}), ((100, 97, [1000, 16]), {}),
    ((130, 300, [512, 136]), dict(tc=1)), ((347, 128, [192, 96]), dict(tc=1)), ((256, 257, [520]), dict(tc=1)),
    ((200, 136, [264, 264]), dict(mode=1)), ((260, 300, [576]), dict(mode=1)), ((66, 131, [40, 88]), dict(mode=1)),
    ((128, 192, [640]), dict(mode=2)), ((300, 260, [72, 512]), dict(mode=2)), ((65, 133, [8]), dict(mode=2)),
]


@pytest.mark.parametrize("shape,kw", PAIRED)
def test_two_workgroups_to_a_cu_agree_with_one(shape, kw):
    """One vertex in a launch of its own, and so many on the same operands that they fill 256 workgroups and more."""
    m, n, ks = shape
    tc, mode = kw.get("tc", 0), kw.get("mode", 0)
    wide = 64 if mode == 2 else 128
    blocks = -(-m // 128) * -(-n // wide)
    copies = 1 + 256 // blocks
    print(f"[case] gemm bf16 {m}x{n} K {ks} transposed {tc} mode {mode}, 1 and {copies}", flush=True)
    ref, res = None, []
    for c in (1, copies):
        rng = np.random.default_rng(m * 1000 + n + sum(ks))
        g = Graph("bf16")
        a = [g.inp(rng.standard_normal((m, k))) for k in ks]
        b = [[g.inp(rng.standard_normal((n, k)) / np.sqrt(sum(ks))) for k in ks] for _ in range(2 if mode == 2 else 1)]
        ins = a + sum(b, []) + ([g.inp(rng.standard_normal((m, n)))] if mode == 1 else [])
        p = dict(nk=len(ks), trans_b=1, trans_c=tc, mode=mode)
        outs = [g.op(B.TN_OP_GEMM, [i[0] for i in ins], n if tc else m, m if tc else n, **p) for _ in range(c)]
        res.append(_run_forms(g, outs, (1 << 20,), one_launch=True)[0])
        ref = T._eval_vertex("gemm", dict(p, trans_a=0), [i[1] for i in ins])
    err = R.rel_err(_wide(res[0][0]), ref)
    bound = sum(ks) * 2.0 ** -24 + 2.0 ** -8
    print(f"  rel err {err:.2e} (bound {bound:.1e})", flush=True)
    assert np.isfinite(_wide(res[0][0])).all() and err < bound
    for got in res[1]:
        assert np.array_equal(got, res[0][0])


@pytest.mark.parametrize("form", [0, -1, 1 << 20])
@pytest.mark.parametrize("copies", [1, 30])  # 30: 270 workgroups of 128x128, two to a CU
def test_what_lies_behind_the_end_of_a_row_is_not_multiplied(form, copies):
    """K of 40 and 72 in chunks of 64: the elements behind a row's end are the next row's, here infinite, and those of another tensor."""
    print(f"[case] infinite rows, small_gemm_tiles {form}, {copies} vertices", flush=True)
    rng = np.random.default_rng(7)
    ks, m, n = [40, 72], 300, 280
    g = Graph("bf16")
    full = [rng.standard_normal((m, k)) for k in ks]
    for x in full:
        x[1::3] = np.inf
    ins = [g.inp(x) for x in full] + [g.inp(rng.standard_normal((n, k))) for k in ks]
    outs = [g.op(B.TN_OP_GEMM, [i[0] for i in ins], m, n, nk=len(ks), trans_b=1) for _ in range(copies)]
    keep = np.ones(m, bool)
    keep[1::3] = False
    ref = sum(ins[q][1][keep] @ ins[q + len(ks)][1].T for q in range(len(ks)))
    for got in map(_wide, _run_forms(g, outs, (form,), one_launch=True)[0]):
        assert R.rel_err(got[keep], ref) < sum(ks) * 2.0 ** -24 + 2.0 ** -8
        assert not np.isfinite(got[1::3]).any()


def test_products_of_different_shapes_share_a_launch():
    """Ragged vertices of one launch take fewer workgroups than its largest.  (3 MB of operands: loaded by one copy, ready at once.)"""
    print("[case] seven shapes in one launch", flush=True)
    rng = np.random.default_rng(9)
    g = Graph("bf16")
    k, outs, refs = 192, [], []
    a = {m: g.inp(rng.standard_normal((m, k))) for m in (256, 259, 300, 512, 700, 2000)}
    bs = {n: g.inp(rng.standard_normal((n, k)) / np.sqrt(k)) for n in (256, 300, 520, 1000, 2100)}
    for m, n in [(256, 256), (700, 300), (259, 520), (512, 256), (300, 300), (256, 1000), (2000, 2100)]:  # 331 workgroups of 128x128
        outs.append(g.op(B.TN_OP_GEMM, [a[m][0], bs[n][0]], m, n, nk=1, trans_b=1))
        refs.append(a[m][1] @ bs[n][1].T)
    for res in _run_forms(g, outs, (0, -1, 1 << 20), one_launch=True):
        for got, ref in zip(res, refs):
            assert R.rel_err(_wide(got), ref) < k * 2.0 ** -24 + 2.0 ** -8
