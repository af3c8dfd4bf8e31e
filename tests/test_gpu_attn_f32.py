"""The attention kernels with fp32 products (fp32 graphs, and bf16 tilings the bf16 kernels do not take),
at the edges of their 64-row chunks and 16-row wavefronts and over every layout of the tile grid,
against float64.  Tolerances: the repository's 1e-4 for fp32 results (sums of at most a few hundred
fp32 products, measured 1e-6), 2e-2 where the result is stored as bf16 (half an ulp is 2^-9 of a value)."""
import numpy as np
import pytest
import torch

from oracle import llama_ref as R
from oracle import tiled as T
from paper_2405_16283_amd import binding as B

from test_gpu_attention_block import _compare, _ranges
from test_gpu_backward_ops import TOL, Graph

pytestmark = pytest.mark.gpu


def _grid(g, full, ranges, tc, transpose=False):
    vs, wide = [], np.zeros(full.shape)
    for r0, r1 in ranges:
        for c0 in range(0, full.shape[1], tc):
            v, w = g.inp(full[r0:r1, c0:c0 + tc].T if transpose else full[r0:r1, c0:c0 + tc])
            vs.append(v)
            wide[r0:r1, c0:c0 + tc] = w.T if transpose else w
    return vs, wide


FORWARD = [
    # dtype, hd, hpg, tc, q_rows, kv_rows, tq, tk, q_pos0, k_pos0, causal, v_trans
    ("f32", 64, 2, 128, 128, 128, 64, 64, 0, 0, 1, 1),      # two full chunks
    ("f32", 128, 1, 128, 65, 129, 128, 128, 64, 0, 1, 1),   # one row, one key past a chunk
    ("f32", 64, 1, 64, 15, 17, 64, 64, 2, 0, 1, 0),         # less than a wavefront's rows; V as plain tiles
    ("f32", 128, 1, 32, 70, 90, 32, 32, 20, 0, 1, 1),       # a head across four column tiles
    ("f32", 64, 1, 64, 100, 75, 100, 1, 0, 0, 0, 1),        # single-row key tiles
    ("f32", 64, 1, 64, 48, 200, 48, 96, 80, 100, 1, 1),     # tiles that straddle chunks; rows that see nothing
    ("bf16", 128, 2, 256, 130, 203, 128, 256, 73, 0, 1, 0),  # bf16, plain V
    ("bf16", 64, 1, 64, 33, 77, 64, 48, 44, 0, 1, 1),       # bf16, key tiles of 48 rows, odd last tile
]


@pytest.mark.parametrize("case", FORWARD)
def test_attention_block(case):
    dtype, hd, hpg, tc, q_rows, kv_rows, tq, tk, q_pos0, k_pos0, causal, v_trans = case
    print(f"[case] attn_block {case}", flush=True)
    rng = np.random.default_rng(q_rows)
    g = Graph(dtype)
    gw = hpg * hd
    qt, kt = _ranges(q_rows, tq), _ranges(kv_rows, tk)
    q, Q = _grid(g, rng.standard_normal((q_rows, gw)), qt, tc)
    k, K = _grid(g, rng.standard_normal((kv_rows, gw)), kt, tc)
    v, V = _grid(g, rng.standard_normal((kv_rows, gw)), kt, tc, bool(v_trans))
    p = dict(n_q_tiles=len(qt), n_kv_tiles=len(kt), n_col_tiles=gw // tc, head_dim=hd, q_pos0=q_pos0, k_pos0=k_pos0,
             causal=causal, scale=1.0 / np.sqrt(hd), v_trans=v_trans)
    blk = g.op(B.TN_OP_ATTN_BLOCK, q + k + v, q_rows, gw + 2 * hpg, f32=True, **p)
    (got,) = g.run([blk])
    ref = T._eval_vertex("attn_block", dict(p, n_q_tiles=1, n_kv_tiles=1, n_col_tiles=1, v_trans=0), [Q, K, V])
    _compare(got, ref, gw, hd, hpg)


BACKWARD = [
    # dtype, hd, tc, q_rows, kv_rows, tq, tk, q_pos0, v_trans
    ("f32", 64, 64, 160, 160, 64, 64, 0, 0),
    ("f32", 128, 128, 65, 129, 65, 129, 64, 0),
    ("f32", 64, 64, 17, 63, 17, 40, 46, 1),     # key tiles of 40 rows, V transposed
    ("f32", 128, 32, 33, 70, 32, 32, 37, 0),    # a head across four column tiles
    ("bf16", 128, 128, 131, 131, 128, 128, 0, 0),
]


@pytest.mark.parametrize("case", BACKWARD)
def test_attention_reverse(case):
    dtype, hd, tc, q_rows, kv_rows, tq, tk, q_pos0, v_trans = case
    print(f"[case] attn_bwd {case}", flush=True)
    rng = np.random.default_rng(kv_rows)
    g = Graph(dtype)
    hpg, scale = (2 if tc >= hd else 1), 1.0 / np.sqrt(hd)
    gw = hpg * hd
    qt, kt = _ranges(q_rows, tq), _ranges(kv_rows, tk)
    q, Q = _grid(g, rng.standard_normal((q_rows, gw)), qt, tc)
    k, K = _grid(g, rng.standard_normal((kv_rows, gw)), kt, tc)
    v, V = _grid(g, rng.standard_normal((kv_rows, gw)), kt, tc, bool(v_trans))
    do, DO = _grid(g, rng.standard_normal((q_rows, gw)), qt, tc)
    nc = gw // tc
    p = dict(n_q_tiles=len(qt), n_kv_tiles=len(kt), n_col_tiles=nc, head_dim=hd, q_pos0=q_pos0, k_pos0=0, causal=1, scale=scale,
             v_trans=v_trans)
    stats = []
    for i, (r0, r1) in enumerate(qt):
        ins = q[i * nc:(i + 1) * nc] + k + v + do[i * nc:(i + 1) * nc]
        stats.append(g.op(B.TN_OP_ATTN_BWD, ins, r1 - r0, 2 * hpg, f32=True, mode=0, **dict(p, n_q_tiles=1, q_pos0=q_pos0 + r0)))
    base = q + k + v + do + stats
    outs = [g.op(B.TN_OP_ATTN_BWD, base, rows, gw, mode=m, **p) for m, rows in ((1, q_rows), (2, kv_rows), (3, kv_rows))]
    got = g.run(stats + outs)
    tq_, tk_, tv_ = (torch.tensor(a, requires_grad=True) for a in (Q, K, V))
    mask = torch.arange(kv_rows)[None, :] > (q_pos0 + torch.arange(q_rows))[:, None]
    loss, lse, dd = 0.0, [], []
    for h in range(hpg):
        sl = slice(h * hd, (h + 1) * hd)
        s = (tq_[:, sl] @ tk_[:, sl].T * scale).masked_fill(mask, float("-inf"))
        o = torch.softmax(s, dim=-1) @ tv_[:, sl]
        loss = loss + (o * torch.tensor(DO[:, sl])).sum()
        lse.append(torch.logsumexp(s, dim=-1).detach().numpy())
        dd.append((o.detach().numpy() * DO[:, sl]).sum(axis=1))
    loss.backward()
    st = np.concatenate(got[:len(qt)], axis=0)
    errs = [R.rel_err(st[:, :hpg], np.stack(lse, 1)), R.rel_err(st[:, hpg:], np.stack(dd, 1))]
    errs += [R.rel_err(a, t.grad.numpy()) for a, t in zip(got[-3:], (tq_, tk_, tv_))]
    print("  lse, D, dQ, dK, dV:", ", ".join(f"{e:.1e}" for e in errs), flush=True)
    assert max(errs) < TOL[dtype]


def _masked_reference(Q, K, V, DO, scale, q_pos0):
    """lse, D, output, dQ, dK, dV in float64, every row summed over the keys it sees and nothing else."""
    q_rows, hd = Q.shape
    lse, dd = np.zeros(q_rows), np.zeros(q_rows)
    o, dq, dk, dv = np.zeros((q_rows, hd)), np.zeros((q_rows, hd)), np.zeros(K.shape), np.zeros(V.shape)
    for i in range(q_rows):
        n = min(len(K), q_pos0 + i + 1)
        s = (K[:n] * Q[i]).sum(1) * scale
        m = s.max()
        lse[i] = m + np.log(np.exp(s - m).sum())
        p = np.exp(s - lse[i])
        o[i] = (p[:, None] * V[:n]).sum(0)
        dp = (V[:n] * DO[i]).sum(1)
        dd[i] = (p * dp).sum()
        ds = p * (dp - dd[i]) * scale
        dq[i] = (ds[:, None] * K[:n]).sum(0)
        dk[:n] += ds[:, None] * Q[i]
        dv[:n] += p[:, None] * DO[i]
    return lse[:, None], dd[:, None], o, dq, dk, dv


@pytest.mark.parametrize("which,value", [("k", np.nan), ("v", np.inf), ("v", np.nan), ("q", np.nan), ("do", np.inf), ("do", np.nan)])
@pytest.mark.parametrize("dtype,hd,v_trans", [("f32", 64, 0), ("f32", 128, 1), ("bf16", 128, 0)])
def test_what_the_mask_hides_stays_hidden(dtype, hd, v_trans, which, value):
    """An infinity or NaN at one position reaches the rows that see it and no others, in the chunk on the diagonal too."""
    print(f"[case] {value} in {which}, {dtype} head size {hd}, V transposed {v_trans}", flush=True)
    rng = np.random.default_rng(hd + v_trans)
    rows, scale = 131, 1.0 / np.sqrt(hd)  # 131: no multiple of what the bf16 kernels take
    full = {k: rng.standard_normal((rows, hd)) for k in ("q", "k", "v", "do")}
    full[which][100, 5] = value  # chunk of positions 64 .. 127
    g = Graph(dtype)
    (q, Q), (k, K), (do, DO) = (g.inp(full[n]) for n in ("q", "k", "do"))
    v, V = g.inp(full["v"].T if v_trans else full["v"])
    V = V.T if v_trans else V
    p = dict(n_q_tiles=1, n_kv_tiles=1, n_col_tiles=1, head_dim=hd, q_pos0=0, k_pos0=0, causal=1, scale=scale, v_trans=v_trans)
    blk = g.op(B.TN_OP_ATTN_BLOCK, [q, k, v], rows, hd + 2, f32=True, **p)
    stat = g.op(B.TN_OP_ATTN_BWD, [q, k, v, do], rows, 2, f32=True, mode=0, **p)
    grads = [g.op(B.TN_OP_ATTN_BWD, [q, k, v, do, stat], rows, hd, mode=m, **p) for m in (1, 2, 3)]
    with np.errstate(all="ignore"):
        out, st, dq, dk, dv = g.run([blk, stat] + grads)
        got = [st[:, :1], st[:, 1:], out[:, :hd] / out[:, hd + 1:], dq, dk, dv]
        want = _masked_reference(Q, K, V, DO, scale, 0)
    for name, a, b in zip(("lse", "D", "output", "dQ", "dK", "dV"), got, want):
        fine = np.isfinite(b)
        assert np.array_equal(np.isfinite(a), fine), name
        if fine.any():
            assert R.rel_err(a[fine], b[fine]) < TOL[dtype], name


@pytest.mark.parametrize("which", ["k", "v", "q", "do"])
@pytest.mark.parametrize("dtype,hd,tc,tq,tk,q_pos0,v_trans", [("f32", 64, 32, 48, 40, 0, 0), ("f32", 128, 256, 64, 33, 21, 1),
                                                              ("bf16", 64, 128, 50, 48, 7, 0)])
def test_what_the_mask_hides_stays_hidden_over_tiles(dtype, hd, tc, tq, tk, q_pos0, v_trans, which):
    """The same with two heads, the second of which holds a NaN, over tiles that cut rows and heads anywhere."""
    print(f"[case] NaN in {which}, {dtype} head size {hd}, tiles {tq}, {tk} rows, {tc} columns, queries from {q_pos0}", flush=True)
    rng = np.random.default_rng(tq)
    kv_rows, scale, gw = 131, 1.0 / np.sqrt(hd), 2 * hd
    q_rows = kv_rows - q_pos0
    full = {n: rng.standard_normal((q_rows if n in ("q", "do") else kv_rows, gw)) for n in ("q", "k", "v", "do")}
    full[which][90, hd + 3] = np.nan
    g = Graph(dtype)
    qt, kt = _ranges(q_rows, tq), _ranges(kv_rows, tk)
    q, Q = _grid(g, full["q"], qt, tc)
    k, K = _grid(g, full["k"], kt, tc)
    v, V = _grid(g, full["v"], kt, tc, bool(v_trans))
    do, DO = _grid(g, full["do"], qt, tc)
    nc = gw // tc
    p = dict(n_q_tiles=len(qt), n_kv_tiles=len(kt), n_col_tiles=nc, head_dim=hd, q_pos0=q_pos0, k_pos0=0, causal=1, scale=scale,
             v_trans=v_trans)
    blk = g.op(B.TN_OP_ATTN_BLOCK, q + k + v, q_rows, gw + 4, f32=True, **p)
    stats = [g.op(B.TN_OP_ATTN_BWD, q[i * nc:(i + 1) * nc] + k + v + do[i * nc:(i + 1) * nc], r1 - r0, 4, f32=True, mode=0,
                  **dict(p, n_q_tiles=1, q_pos0=q_pos0 + r0)) for i, (r0, r1) in enumerate(qt)]
    grads = [g.op(B.TN_OP_ATTN_BWD, q + k + v + do + stats, rows, gw, mode=m, **p) for m, rows in ((1, q_rows), (2, kv_rows), (3, kv_rows))]
    with np.errstate(all="ignore"):
        out, *rest = g.run([blk] + stats + grads)
        st, (dq, dk, dv) = np.concatenate(rest[:-3]), rest[-3:]
        for h in range(2):
            sl = slice(h * hd, (h + 1) * hd)
            got = [st[:, h:h + 1], st[:, 2 + h:3 + h], out[:, sl] / out[:, gw + 2 + h:gw + 3 + h], dq[:, sl], dk[:, sl], dv[:, sl]]
            want = _masked_reference(Q[:, sl], K[:, sl], V[:, sl], DO[:, sl], scale, q_pos0)
            for name, a, b in zip(("lse", "D", "output", "dQ", "dK", "dV"), got, want):
                fine = np.isfinite(b)
                assert h == 1 or fine.all()
                assert np.array_equal(np.isfinite(a), fine), (h, name)
                if fine.any():
                    assert R.rel_err(a[fine], b[fine]) < TOL[dtype], (h, name)
