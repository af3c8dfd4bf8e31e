"""Row statistics over tiles of any number and width, and transposes, at the edges of what the kernels take
at once: 512 (or 64) columns of a tile, four (or eight) such pieces, 64 tiles, 64x64 pieces of a transpose.
Tolerance: fp32 sums of n terms differ from float64 by less than n 2^-24 of the sum of magnitudes; __expf adds a few
2^-22; a bf16 result adds half a unit of 2^-8.  Transposes move bits."""
import numpy as np
import pytest

from oracle import tiled as T
from paper_2405_16283_amd import binding as B

from test_gpu_backward_ops import Graph

pytestmark = pytest.mark.gpu

WIDTHS = [[1], [8], [13, 7], [64, 64, 64, 40], [512], [520, 504], [1024, 1024, 256], [128] * 9, [96] * 64 + [32], [16] * 130, [24, 5, 512]]


def _inputs(g, widths, rows, seed):
    rng = np.random.default_rng(seed)
    return [g.inp(rng.standard_normal((rows, w))) for w in widths]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("widths", WIDTHS, ids=lambda w: f"{len(w)}x{w[0]}")
def test_row_statistics(dtype, widths):
    rows, n = 13, sum(widths)
    print(f"[case] row statistics {dtype} {len(widths)} tiles, {n} columns", flush=True)
    g = Graph(dtype)
    xs = _inputs(g, widths, rows, n)
    dys = _inputs(g, widths, rows, n + 1)
    gains = _inputs(g, widths, 1, n + 2)
    ids = lambda ts: [v for v, _ in ts]
    stat = g.op(B.TN_OP_RMS_STAT, ids(xs), rows, 1, f32=True, d=n, eps=1e-6)
    dot = g.op(B.TN_OP_RMS_BWD_STAT, ids(dys) + ids(xs) + ids(gains), rows, 1, f32=True, nk=len(widths))
    p = dict(scale=0.125, causal=1, q_pos0=max(0, n - rows // 2), k_pos0=0)  # the diagonal crosses the last columns
    soft = g.op(B.TN_OP_SOFTMAX_STAT, ids(xs), rows, 2, f32=True, **p)
    q = dict(p, q_pos0=3, k_pos0=0)
    low = g.op(B.TN_OP_SOFTMAX_STAT, ids(xs), rows, 2, f32=True, **q)  # the diagonal crosses the first columns
    prob = g.op(B.TN_OP_SOFTMAX_APPLY, [xs[0][0], low], rows, widths[0], **q)
    got = g.run([stat, dot, soft, low, prob])
    x, dy, gain = (np.concatenate([a for _, a in ts], axis=1) for ts in (xs, dys, gains))
    u = n * 2.0 ** -24 + 2.0 ** -20
    want = T._eval_vertex("rms_stat", dict(d=n, eps=1e-6), [x])
    assert np.abs(got[0] / want - 1).max() < u
    terms = dy * gain * x
    assert (np.abs(got[1][:, 0] - terms.sum(axis=1)) <= u * np.abs(terms).sum(axis=1)).all()
    for out, par in ((got[2], p), (got[3], q)):
        want = T._eval_vertex("softmax_stat", par, [x])
        assert np.allclose(out, want, rtol=u, atol=0)
    want = T._eval_vertex("softmax_apply", q, [xs[0][1], T._eval_vertex("softmax_stat", q, [x])])
    assert np.allclose(got[4], want, rtol=2 * u + (2.0 ** -8 if dtype == "bf16" else 0), atol=0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1), (63, 65), (64, 64), (130, 7), (72, 136), (5, 200)])
def test_transpose(dtype, shape):
    g = Graph(dtype)
    x, X = g.inp(np.random.default_rng(0).standard_normal(shape))
    (out,) = g.run([g.op(B.TN_OP_TRANSPOSE, [x], shape[1], shape[0])])
    assert np.array_equal(out, X.T)
