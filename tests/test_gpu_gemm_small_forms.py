"""fp32 and small bf16 products in launches of few and of many workgroups (16x16 and 32x32 tiles per workgroup in fp32), with and
without whole pieces along K, and with more K tiles than a wavefront has lanes.  Tolerance as in test_gpu_gemm_small: K 2^-24, and half a unit
of 2^-8 for bf16 results; the forms agree bit for bit."""
import numpy as np
import pytest

from oracle import llama_ref as R
from oracle import tiled as T
from paper_2405_16283_amd import binding as B

from test_gpu_backward_ops import Graph

pytestmark = pytest.mark.gpu


def _products(dtype, m, n, ks, copies, tc=0, mode=0):
    """`copies` vertices on the same operands, ready at once; (results, float64 reference)."""
    rng = np.random.default_rng(m * 1000 + n + sum(ks))
    g = Graph(dtype)
    a = [g.inp(rng.standard_normal((m, k))) for k in ks]
    b = [[g.inp(rng.standard_normal((n, k)) / np.sqrt(sum(ks))) for k in ks] for _ in range(2 if mode == 2 else 1)]
    extra = [g.inp(rng.standard_normal((m, n)))] if mode == 1 else []
    ins = a + sum(b, []) + extra
    p = dict(nk=len(ks), trans_b=1, trans_c=tc, mode=mode)
    outs = [g.op(B.TN_OP_GEMM, [i[0] for i in ins], n if tc else m, m if tc else n, **p) for _ in range(copies)]
    return g.run(outs), T._eval_vertex("gemm", dict(p, trans_a=0), [i[1] for i in ins])


CASES = [
    ((16, 16, [32]), {}), ((17, 33, [32, 32]), {}), ((64, 64, [64] * 11), {}), ((40, 70, [128, 100, 36]), {}), ((33, 48, [20]), {}),
    ((31, 65, [256, 30]), {}),                                     # rows not aligned to four elements
    ((96, 80, [1024]), {}), ((50, 64, [160]), dict(tc=1)), ((48, 40, [96, 64]), dict(mode=1)), ((40, 33, [224]), dict(mode=2)),
    ((20, 24, [32] * 70), {}), ((20, 24, [36] * 66), {}),          # more K tiles than lanes
]


@pytest.mark.parametrize("shape,kw", CASES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_few_and_many_workgroups(dtype, shape, kw):
    m, n, ks = shape
    print(f"[case] gemm {dtype} {m}x{n} K {ks} {kw}", flush=True)
    many = 1 + 200 // (-(-m // 32) * -(-n // 32))  # more than 128 workgroups of 32x32
    one, ref = _products(dtype, m, n, ks, 1, **kw)
    all_, _ = _products(dtype, m, n, ks, many, **kw)
    err = R.rel_err(one[0], ref)
    bound = sum(ks) * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    print(f"  rel err {err:.2e} (bound {bound:.1e})", flush=True)
    assert err < bound
    for got in all_:
        assert np.array_equal(got, one[0])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m", [1, 40])
def test_products_of_any_depth_share_a_launch(dtype, m):
    """A launch's rings have as many stages as its deepest vertex uses, one to four: results are those of the vertices alone."""
    print(f"[case] gemm {dtype} {m}x48 of mixed depth", flush=True)
    piece = 32 if dtype == "f32" else 64
    alone, shared = [], []
    for together in ([0], [1], [2], [3], [4], [0, 1, 2], [0, 1, 2, 3, 4]):
        rng = np.random.default_rng(7)
        g = Graph(dtype)
        outs, refs = [], []
        for d, k in enumerate([piece // 2, 4 * piece, 5 * piece, 9 * piece + 8, 40 * piece]):
            a, b = g.inp(rng.standard_normal((m, k))), g.inp(rng.standard_normal((48, k)) / np.sqrt(k))
            if d in together:
                outs.append(g.op(B.TN_OP_GEMM, [a[0], b[0]], m, 48, nk=1, trans_b=1))
                refs.append((d, k, T._eval_vertex("gemm", dict(nk=1, trans_a=0, trans_b=1, trans_c=0, mode=0), [a[1], b[1]])))
        for got, (d, k, ref) in zip(g.run(outs), refs):
            assert R.rel_err(got, ref) < k * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
            (alone if len(together) == 1 else shared).append((d, got))
    for d, got in shared:
        assert np.array_equal(got, dict(alone)[d])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("nk", [64, 65])
def test_single_rows_with_many_tiles_along_k(dtype, nk):
    """The addresses of the rows' tiles lie in LDS up to 64 tiles along K."""
    print(f"[case] rows {dtype} nk {nk}", flush=True)
    rng = np.random.default_rng(nk)
    g = Graph(dtype)
    k, n, rows = 72, 40, 35
    b = [g.inp(rng.standard_normal((n, k)) / np.sqrt(nk * k)) for _ in range(nk)]
    outs, refs = [], []
    for _ in range(rows):
        a = [g.inp(rng.standard_normal((1, k))) for _ in range(nk)]
        outs.append(g.op(B.TN_OP_GEMM, [i[0] for i in a + b], 1, n, nk=nk, trans_b=1))
        refs.append(T._eval_vertex("gemm", dict(nk=nk, trans_a=0, trans_b=1, trans_c=0, mode=0), [i[1] for i in a + b]))
    err = R.rel_err(np.concatenate(g.run(outs)), np.concatenate(refs))
    print(f"  rel err {err:.2e}", flush=True)
    assert err < nk * k * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
