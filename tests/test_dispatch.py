"""The executor's dispatch on the CPU: the library's host sources linked with tests/fake_gpu.cpp in place of the HIP runtime
and the kernels.  There streams run their work late and overtake each other at random, and a vertex's result is a mix of
its operands', so work enqueued without the order it needs, or a copy taken from or put in the wrong place, changes what
comes out.  What was enqueued where, behind what, can be read back."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2405_16283_amd import binding as B
from paper_2405_16283_amd import build
from paper_2405_16283_amd import harness as H
from workloads import config

ALIGN = 256
KERNEL, COPY, DEVICE_COPY, MEMCPY = range(4)  # kinds of log entries
COMPUTE, H2D, D2H = 0, 100, 101               # stream numbers (compute streams: 0, 1, ...)


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    """The library on a GPU that is not there, in place of the built one for the tests of this file."""
    out = str(tmp_path_factory.mktemp("fake") / "libturnip_fake.so")
    here = os.path.dirname(os.path.abspath(__file__))
    src = [os.path.join(here, "fake_gpu.cpp")] + [os.path.join(build.CSRC, f) for f in sorted(os.listdir(build.CSRC)) if f.endswith(".cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-Wl,-Bsymbolic", "-o", out] + src, check=True)
    lib = C.CDLL(out)
    for name, (res, args) in B.SIGNATURES.items():
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    lib.fake_stream.restype = lib.fake_alloc.restype = C.c_void_p
    lib.fake_alloc.argtypes = [C.c_uint64, C.c_int]
    lib.fake_reset.argtypes = [C.c_uint64]
    lib.fake_fail_after.argtypes = [C.c_int64]
    lib.fake_pending.restype = lib.fake_enqueued_after_failure.restype = C.c_int64
    lib.fake_log.restype, lib.fake_log.argtypes = C.c_int64, [C.c_void_p, C.c_int64]
    old, B._lib = B._lib, lib
    yield lib
    B._lib = old


class Session:
    """A memgraph, its buffers and an executor on the fake GPU.  Takes the taskgraph over."""

    def __init__(self, fake, tg, cap, compile_opts=None, n_compute=1, arena_bytes=0, order=None):
        self.fake, self.tg = fake, tg
        self.mg = B.tn_compile(tg, order, cap, compile_opts)
        self.stats = B.tn_memgraph_stats(self.mg)
        n = B.tn_taskgraph_num_vertices(tg)
        desc = [B.tn_taskgraph_vertex(tg, v) for v in range(n)]
        size = [x.desc.rows * x.desc.cols * (4 if x.desc.dtype == B.TN_F32 else 2) for x in desc]
        self.ins = [0] * n
        for v, x in enumerate(desc):
            if x.kind == B.TN_OP_INPUT:
                self.ins[v] = fake.fake_alloc(size[v] + 4, 0)
                C.memmove(self.ins[v], (0x9E3779B1 * (v + 1) % 2**32).to_bytes(4, "little"), 4)
        self.outs = [0] * B.tn_taskgraph_num_outputs(tg)
        for v, x in enumerate(desc):
            if x.output_index >= 0:
                self.outs[x.output_index] = fake.fake_alloc(size[v] + 4, 0)
        self.cap, self.dev = cap, fake.fake_alloc(cap, 1)
        self.n_compute, self.arena_bytes = n_compute, arena_bytes
        self.ex = None

    def run(self, seed=0, fail_after=-1, **opts):
        """One execution on fresh streams; (words of the outputs, report, log)."""
        f = self.fake
        f.fake_reset(seed)
        if self.ex:
            B.tn_executor_destroy(self.ex)
        self.ex = B.tn_executor_create(self.mg, self.dev, self.cap, 0, self.arena_bytes, [f.fake_stream(k) for k in range(self.n_compute)],
                                       f.fake_stream(H2D), f.fake_stream(D2H))
        for o in self.outs:
            C.memset(o, 0, 4)
        C.memset(self.dev, 0xEE, self.cap)
        B.tn_executor_place_inputs(self.ex, self.ins)
        f.fake_fail_after(fail_after)
        rep = B.tn_execute(self.ex, self.ins, self.outs, B.tn_exec_opts(**opts))
        assert f.fake_pending() == 0
        B.tn_memgraph_simulate(self.mg, B.tn_executor_last_order(self.ex, self.stats.n_vertices))
        return [C.c_uint32.from_address(o).value for o in self.outs], rep, self.log()

    def log(self):
        n = self.fake.fake_log(None, 0)
        a = np.zeros((n, 6), dtype=np.int32)
        self.fake.fake_log(a.ctypes.data, n)
        return np.rec.fromarrays(a.T, names="kind,stream,n,detail,kernels_before,to_gpu")

    def close(self):
        if self.ex:
            B.tn_executor_destroy(self.ex)
        B.tn_memgraph_destroy(self.mg)
        B.tn_taskgraph_destroy(self.tg)


def llama(fake, name, cap_pct=None, n_compute=1, arena_bytes=0, compile_opts=None, **kw):
    cfg = config(name)
    tg = B.tn_build_llama(H.llama_config_struct(cfg, **kw))
    cap = H.cap_for(cfg, tg) if cap_pct is None else H.uncapped_peak(tg) * cap_pct // 100 // ALIGN * ALIGN
    return Session(fake, tg, cap, n_compute=n_compute, arena_bytes=arena_bytes, compile_opts=compile_opts)


def chained(log):
    """Copies on a compute stream."""
    return log[(log.stream < H2D) & (log.kind != KERNEL)]


POLICIES = [B.TN_POLICY_BY_ORDER, B.TN_POLICY_FIFO, B.TN_POLICY_LIFO, B.TN_POLICY_RANDOM]


@pytest.mark.parametrize("name,kw", [("c1", {}), ("c1", dict(k_split=2)), ("ragged_f32", dict(kv_outputs=True)), ("decode_f32", {}),
                                     ("batch2_f32", dict(lora_rank=16, train=True)), ("ragged_f32", dict(materialize_scores=True))],
                         ids=["c1", "c1_sums", "ragged_kv", "decode", "train", "scores"])
def test_every_order_computes_the_same(fake, name, kw):
    """Chained copies (one compute stream, depth above 1) and copies the host waits for, on streams that overtake each other."""
    s = llama(fake, name, **kw)
    try:
        assert s.stats.n_offload > 0
        want, rep1, log1 = s.run(policy=B.TN_POLICY_IN_ORDER, max_batch=1, max_transfers=1)
        assert not len(chained(log1))
        for seed in range(8):
            got, rep, log = s.run(seed, policy=POLICIES[seed % 4], order_seed=seed, queue_depth=(3, 8, 2)[seed % 3],
                                  max_gemm_inflight=seed % 2, max_batch=(0, 3, 1920)[seed % 3], max_transfers=(0, 2)[seed // 4])
            assert got == want and len(chained(log)) > 0
            assert (rep.n_offload, rep.n_reload, rep.h2d_bytes, rep.d2h_bytes) == (rep1.n_offload, rep1.n_reload, rep1.h2d_bytes, rep1.d2h_bytes)
        for kw in (dict(queue_depth=1), dict(queue_depth=3, max_delay_us=5), dict(queue_depth=3, copy_engine=B.TN_COPY_MEMCPY)):
            got, _, log = s.run(1, policy=B.TN_POLICY_RANDOM, order_seed=1, **kw)
            assert got == want and not len(chained(log))
    finally:
        s.close()


def test_several_streams_compute_the_same(fake):
    s = llama(fake, "c1", n_compute=3)
    try:
        want, _, _ = s.run(policy=B.TN_POLICY_IN_ORDER, max_batch=1, max_transfers=1)
        for seed in range(4):
            got, _, log = s.run(seed, policy=POLICIES[seed], order_seed=seed, queue_depth=1 + seed)
            assert got == want and not len(chained(log))
    finally:
        s.close()


@pytest.mark.parametrize("opts", [dict(queue_depth=3), dict(queue_depth=3, copy_engine=B.TN_COPY_KERNEL), dict(queue_depth=1),
                                  dict(queue_depth=3, copy_engine=B.TN_COPY_MEMCPY)], ids=["chained", "kernel", "depth1", "memcpy"])
def test_after_a_hip_error_every_stream_is_idle(fake, opts):
    """Whichever call fails: nothing is enqueued after it, and the buffers are the caller's again when the call returns."""
    s = llama(fake, "c1", cap_pct=45)
    try:
        failed = 0
        for at in list(range(20)) + list(range(20, 900, 67)):
            try:
                s.run(at, fail_after=at, policy=B.TN_POLICY_BY_ORDER, max_gemm_inflight=1, **opts)
            except B.TurnipError as e:
                assert e.status == B.TN_ERR_HIP
                assert fake.fake_pending() == 0, at
                assert fake.fake_enqueued_after_failure() == 0, at
                failed += 1
                with pytest.raises(B.TurnipError, match="poisoned"):
                    B.tn_execute(s.ex, s.ins, s.outs, None)
        assert failed > 20
    finally:
        s.close()


@pytest.mark.parametrize("depth", [1, 3])
def test_an_offload_waits_for_room_in_the_arena(fake, depth):
    """An arena no larger than some orders need: reloads that kernels in flight are about to allow give slots back."""
    s = llama(fake, "ragged_f32")
    try:
        want, rep, _ = s.run(policy=B.TN_POLICY_BY_ORDER, queue_depth=1)
        assert rep.arena_high_water < s.stats.host_arena_bytes
        s.arena_bytes = rep.arena_high_water
        for seed in range(8):
            got, rep, log = s.run(seed, policy=B.TN_POLICY_BY_ORDER, queue_depth=depth, max_gemm_inflight=1)
            assert got == want and rep.arena_high_water <= s.arena_bytes
            assert not len(chained(log))  # chained offloads would take slots earlier than others
        s.arena_bytes = 4096
        with pytest.raises(B.TurnipError, match="exhausted") as e:
            s.run(policy=B.TN_POLICY_BY_ORDER, queue_depth=depth)
        assert e.value.status == B.TN_ERR_ARENA and fake.fake_pending() == 0
    finally:
        s.close()


@pytest.mark.parametrize("policy", [B.TN_POLICY_BY_ORDER, B.TN_POLICY_FIFO])
def test_a_store_nobody_waits_for_does_not_hold_up_offloads(fake, policy):
    """Small tensors, so that every GPU -> host copy that something waits for can follow the kernel before it."""
    s = llama(fake, "c1", kv_outputs=True)
    try:
        e = H.export_memgraph(s.mg)
        waited = {a for a, _, _ in e["edges"] if e["kind"][a] in ("offload", "store")}
        assert 0 < len(waited) < s.stats.n_offload + s.stats.n_store
        _, _, log = s.run(policy=policy, queue_depth=3, max_gemm_inflight=1)
        c = chained(log)
        assert c.n[c.to_gpu == 0].sum() == len(waited)
    finally:
        s.close()


def test_options_of_the_copies_hold_for_chained_and_small_groups(fake):
    s = llama(fake, "c1", kv_outputs=True)
    try:
        want, _, log = s.run(policy=B.TN_POLICY_BY_ORDER, queue_depth=3)
        to_host = log[(log.kind == COPY) & (log.to_gpu == 0)]
        assert len(chained(log)) and (to_host.stream == D2H).any()  # what the default does with groups of this size
        # the copy engines take what goes to the host
        for depth in (1, 3):
            got, _, log = s.run(policy=B.TN_POLICY_BY_ORDER, queue_depth=depth, copy_engine=B.TN_COPY_KERNEL_IN)
            assert got == want and not len(chained(log))
            assert ((log.kind == MEMCPY) & (log.to_gpu == 0)).any() and not ((log.kind == COPY) & (log.to_gpu == 0)).any()
        # workgroups per direction, tensors per group
        for engine in (B.TN_COPY_AUTO, B.TN_COPY_KERNEL):
            got, _, log = s.run(policy=B.TN_POLICY_BY_ORDER, queue_depth=3, copy_engine=engine, copy_workgroups=3, d2h_workgroups=2,
                                max_transfers=2)
            c = log[(log.kind == COPY) & ((log.to_gpu == 0) | (log.stream != D2H))]  # (not the gathering into a staging slot)
            assert got == want and len(chained(c)) and (c.n <= 2).all()
            assert (c.detail == np.where(c.to_gpu == 1, 3, 2)).all()
    finally:
        s.close()


def _behind(fake, make):
    """Six vertices that each read a small tensor of their own, loaded into the place of the one before, and what `make`
    keeps in GPU memory; returns for every chained load how many kernels it stood behind."""
    tg = B.tn_taskgraph_create()
    add = lambda r, c, where=B.TN_DEVICE: B.tn_taskgraph_add_input(tg, B.TN_F32, r, c, where)
    shape, op, held = make(tg, add)
    for _ in range(6):
        B.tn_taskgraph_mark_output(tg, op(add(*shape, B.TN_HOST)))
    small = max(B.tn_taskgraph_vertex(tg, B.tn_taskgraph_num_vertices(tg) - 1).desc.rows * B.tn_taskgraph_vertex(
        tg, B.tn_taskgraph_num_vertices(tg) - 1).desc.cols, shape[0] * shape[1]) * 4
    s = Session(fake, tg, held + 3 * ((small + 255) // 256 * 256))
    try:
        want, _, _ = s.run(queue_depth=1)
        got, _, log = s.run(queue_depth=3, policy=B.TN_POLICY_BY_ORDER)
        c = chained(log)
        assert got == want and len(c) > 0
        return c.kernels_before[c.to_gpu == 1]
    finally:
        s.close()


def _rows(k, n):
    def make(tg, add):
        b = add(n, k)
        return (1, k), lambda x: B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, B.tn_op_params(nk=1, trans_b=1), [x, b], B.TN_F32, 1, n), k * n * 4
    return make


def _product(m, n, k):
    def make(tg, add):
        a, b = add(m, k), add(n, k)
        p = B.tn_op_params(nk=1, trans_b=1, mode=1)
        return (m, n), lambda x: B.tn_taskgraph_add_op(tg, B.TN_OP_GEMM, p, [a, b, x], B.TN_F32, m, n), (m + n) * k * 4
    return make


def _attention(keys):
    def make(tg, add):
        k, v = add(keys, 64), add(keys, 64)
        p = B.tn_op_params(n_q_tiles=1, n_kv_tiles=1, n_col_tiles=1, head_dim=64, scale=0.125)
        return (4, 64), lambda x: B.tn_taskgraph_add_op(tg, B.TN_OP_ATTN_BLOCK, p, [x, k, v], B.TN_F32, 4, 66), 2 * keys * 64 * 4
    return make


@pytest.mark.parametrize("brief,long", [(_rows(512, 512), _rows(2048, 2048)), (_product(64, 64, 1024), _product(64, 64, 8192)),
                                        (_product(32, 1024, 256), _product(32, 1024, 2048)), (_attention(256), _attention(32768))],
                         ids=["rows", "deep", "thin", "attention"])
def test_copies_are_chained_behind_brief_kernels_only(fake, brief, long):
    """A kernel bound by what it reads, or by its walk along K, keeps the stream from a copy for long however few its operations are."""
    assert (_behind(fake, brief) > 0).any()
    assert not _behind(fake, long).any()


@pytest.mark.parametrize("rows,chains", [(384, True), (385, False)])
def test_chaining_goes_by_the_mean_size_of_the_copies(fake, rows, chains):
    tg = B.tn_taskgraph_create()
    for _ in range(12):
        x = B.tn_taskgraph_add_input(tg, B.TN_F32, rows, 256, B.TN_HOST)  # a KiB per row
        B.tn_taskgraph_mark_output(tg, B.tn_taskgraph_add_op(tg, B.TN_OP_ADD, B.tn_op_params(), [x, x], B.TN_F32, rows, 256))
    s = Session(fake, tg, 4 * rows * 1024)
    try:
        want, _, _ = s.run(queue_depth=1)
        got, _, log = s.run(queue_depth=3, policy=B.TN_POLICY_BY_ORDER)
        assert got == want and (len(chained(log)) > 0) == chains
    finally:
        s.close()


@pytest.mark.parametrize("depth,limit", [(1, 1), (2, 24)])
def test_brief_kernels_of_a_program_without_copies_go_beyond_the_depth(fake, depth, limit):
    """A chain of 40 additions on resident inputs: how many are enqueued and not over at a time."""
    tg = B.tn_taskgraph_create()
    x = v = B.tn_taskgraph_add_input(tg, B.TN_F32, 1, 256, B.TN_DEVICE)
    for _ in range(40):
        v = B.tn_taskgraph_add_op(tg, B.TN_OP_ADD, B.tn_op_params(), [v, x], B.TN_F32, 1, 256)
    B.tn_taskgraph_mark_output(tg, v)
    s = Session(fake, tg, 1 << 16)
    try:
        want, _, _ = s.run(queue_depth=1)
        got, _, log = s.run(3, queue_depth=depth, policy=B.TN_POLICY_BY_ORDER)
        most = 1 + log.kernels_before[log.kind == KERNEL].max()
        assert got == want and (most == limit if depth == 1 else depth < most <= limit)
    finally:
        s.close()
