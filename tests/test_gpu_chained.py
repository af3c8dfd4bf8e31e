"""Transfers chained between the kernels of a single compute stream (queue_depth > 1, one stream): the
same bits, counts and valid orders as with every transfer seen complete by the host (queue_depth 1), for
each kind of memgraph that puts something else between a kernel and a copy: offloads and reloads,
evictions without a copy, joins of sums, single-row tiles, the reverse pass."""
import numpy as np
import pytest

from paper_2405_16283_amd import binding as B
from paper_2405_16283_amd import harness as H
from workloads import config, make_llama_inputs, make_lora_inputs

pytestmark = pytest.mark.gpu

POLICIES = {"by_order": B.TN_POLICY_BY_ORDER, "fifo": B.TN_POLICY_FIFO, "lifo": B.TN_POLICY_LIFO, "random": B.TN_POLICY_RANDOM}


@pytest.mark.parametrize("name,kw", [
    ("c1", {}), ("ragged_f32", {}), ("ragged_bf16", dict(kv_outputs=True)), ("mid_bf16", {}), ("decode_bf16", {}),
    ("c1", dict(k_split=2)), ("batch2_f32", dict(lora_rank=16, train=True))],
    ids=["c1", "ragged_f32", "ragged_bf16_kv", "mid_bf16", "decode_bf16", "c1_sums", "train"])
def test_chained_transfers_carry_the_same_bits(name, kw):
    cfg = config(name)
    full = make_llama_inputs(cfg, 0)
    if kw.get("train"):
        full.update(make_lora_inputs(cfg, 0, rank=16, b_std=0.02))
    s = H.GpuSession(cfg, full, n_compute=1, **kw)
    try:
        assert s.stats.n_offload > 0
        want, rep1 = s.run(B.tn_exec_opts(policy=B.TN_POLICY_BY_ORDER, queue_depth=1))
        for policy in POLICIES:
            for depth, gemms, batch, transfers, profile in ((3, 1, 1920, 0, 0), (8, 0, 3, 2, 0), (2, 1, 0, 0, 1)):
                print(f"[case] {name} {kw} {policy} depth {depth} gemms {gemms} batch {batch} transfers {transfers}", flush=True)
                out, rep = s.run(B.tn_exec_opts(policy=POLICIES[policy], order_seed=depth, queue_depth=depth, max_gemm_inflight=gemms,
                                                max_batch=batch, max_transfers=transfers, profile=profile))
                B.tn_memgraph_simulate(s.mg, s.last_order())  # the order taken respects every dependency
                for key in want:
                    assert np.array_equal(out[key], want[key]), key
                assert (rep.n_vertices, rep.n_offload, rep.n_reload) == (rep1.n_vertices, rep1.n_offload, rep1.n_reload)
                assert (rep.h2d_bytes, rep.d2h_bytes) == (rep1.h2d_bytes, rep1.d2h_bytes)
                if profile:
                    assert rep.untimed_launches == 0 and rep.h2d_ms > 0 and rep.d2h_ms > 0
    finally:
        s.close()


@pytest.mark.parametrize("shift", [0, 4, 16])
def test_small_stores_reach_host_buffers_of_any_alignment(shift):
    """The copy kernel writes 16 bytes at a time; buffers it does not fit are left to the runtime."""
    cfg = config("c1")
    s = H.GpuSession(cfg, make_llama_inputs(cfg, 0), n_compute=1, kv_outputs=True)
    try:
        want, _ = s.run(B.tn_exec_opts(policy=B.TN_POLICY_BY_ORDER, queue_depth=1))
        es = np.dtype(s.elem).itemsize
        step = [(r * c * es + 255) // 256 * 256 + 64 for r, c in s.out_shapes]
        at = np.concatenate([[0], np.cumsum(step)[:-1]]) + shift
        slab = s.torch.zeros(int(sum(step)) + 64, dtype=s.torch.uint8).pin_memory()
        ptrs = B.ptr_array([slab.data_ptr() + int(o) for o in at])
        for depth in (1, 3):
            slab.zero_()
            print(f"[case] c1 host outputs shifted by {shift}, depth {depth}", flush=True)
            B.tn_execute(s.ex, s.in_ptrs, ptrs, B.tn_exec_opts(policy=B.TN_POLICY_BY_ORDER, queue_depth=depth))
            got = slab.numpy()
            used = np.zeros(len(got), dtype=bool)
            for i, (r, c) in enumerate(s.out_shapes):
                n = r * c * es
                ref = s.out_slab[s.out_offs[i]:s.out_offs[i] + n].numpy()
                assert np.array_equal(got[at[i]:at[i] + n], ref)
                used[at[i]:at[i] + n] = True
            assert not got[~used].any()  # nothing between the buffers was written
    finally:
        s.close()
