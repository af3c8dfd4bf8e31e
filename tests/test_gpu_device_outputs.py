"""Results that stay on the GPU, and inputs that are already there: the buffers handed to
tn_execute and tn_executor_place_inputs lie in GPU memory outside the capped device buffer, so
the store and load vertices are copies inside GPU memory.  The bits must be those of the run that
goes through pinned host memory, with either copy engine, and the oracle's."""
import numpy as np
import pytest
import torch

from oracle import llama_ref as R
from oracle import tiled as T
from paper_2405_16283_amd import binding as B
from paper_2405_16283_amd import harness as H
from workloads import bf16_bits_to_f32, config, make_llama_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,tol", [("c1", 1e-4), ("ragged_bf16", 2e-2)])
def test_outputs_in_gpu_memory_carry_the_same_bits(name, tol):
    cfg = config(name)
    full = make_llama_inputs(cfg, 0)
    tg = T.build_llama_taskgraph(cfg)
    ref = T.assemble_outputs(tg, T.evaluate(tg, T.cut_inputs(tg, R.widen(cfg, full))), cfg.tokens, cfg.d_model)
    s = H.GpuSession(cfg, full, kv_outputs=True)
    try:
        want, _ = s.run(B.tn_exec_opts(policy=B.TN_POLICY_BY_ORDER, max_batch=64))
    finally:
        s.close()
    s = H.GpuSession(cfg, full, kv_outputs=True, device_outputs=True)
    try:
        assert s.out_slab.is_cuda and s.stats.n_offload > 0
        for engine in (B.TN_COPY_AUTO, B.TN_COPY_KERNEL, B.TN_COPY_MEMCPY, B.TN_COPY_KERNEL_IN):
            for seed in (0, 1):
                print(f"[case] {name} device outputs, copy engine {engine}, order_seed {seed}", flush=True)
                out, rep = s.run(B.tn_exec_opts(policy=B.TN_POLICY_RANDOM, order_seed=seed, copy_engine=engine,
                                                max_delay_us=50 * seed))
                assert rep.n_vertices == s.stats.n_vertices and out.keys() == want.keys()
                for k in want:
                    np.testing.assert_array_equal(out[k], want[k])
        y = (bf16_bits_to_f32(out["y"]) if cfg.dtype == "bf16" else out["y"]).astype(np.float64)
        assert R.rel_err(y, ref) < tol
    finally:
        s.close()


@pytest.mark.parametrize("resident", [False, True])
def test_inputs_in_gpu_memory_carry_the_same_bits(resident):
    """resident=False: every input is a load vertex reading GPU memory; True: the inputs are placed
    by tn_executor_place_inputs from GPU memory."""
    cfg = config("ragged_bf16").with_(weights_resident=resident, x_resident=resident)
    full = make_llama_inputs(cfg, 0)
    cap = 64 << 20 if resident else None  # resident inputs alone exceed the workload's own 40 % cap
    s = H.GpuSession(cfg, full, cap=cap)
    try:
        want, _ = s.run(B.tn_exec_opts(policy=B.TN_POLICY_BY_ORDER, max_batch=64))
    finally:
        s.close()
    s = H.GpuSession(cfg, full, cap=cap, device_inputs=True, device_outputs=True)
    try:
        assert s.in_slab.is_cuda and s.out_slab.is_cuda
        assert (s.stats.n_load == 0) == resident
        for engine in (B.TN_COPY_AUTO, B.TN_COPY_MEMCPY):
            print(f"[case] ragged_bf16 inputs in GPU memory, resident {resident}, copy engine {engine}", flush=True)
            out, rep = s.run(B.tn_exec_opts(policy=B.TN_POLICY_RANDOM, order_seed=3, copy_engine=engine))
            assert rep.n_vertices == s.stats.n_vertices
            np.testing.assert_array_equal(out["y"], want["y"])
    finally:
        s.close()


def test_an_output_buffer_inside_the_device_buffer_is_refused():
    """The host-side check turns the mistake into an error before anything is launched."""
    cfg = config("c1")
    full = make_llama_inputs(cfg, 0)
    s = H.GpuSession(cfg, full, device_outputs=True)
    try:
        bad = list(s.out_ptrs)
        bad[0] = s.dev.data_ptr() + 256  # inside the capped buffer the memgraph's locations refer to
        s.place_inputs()
        with pytest.raises(B.TurnipError, match="overlaps"):
            B.tn_execute(s.ex, s.in_ptrs, B.ptr_array(bad), None)
        out, rep = s.run()  # the executor is still usable
        assert rep.n_vertices == s.stats.n_vertices
    finally:
        s.close()


@pytest.mark.parametrize("shift", [0, 4, 16])
def test_inputs_are_placed_from_gpu_memory_of_any_alignment(shift):
    """Sources that the grouped copies do not take (not 16-byte aligned) go through the runtime; ragged tile sizes."""
    cfg = config("ragged_f32").with_(weights_resident=True, x_resident=True)
    full = make_llama_inputs(cfg, 0)
    print(f"[case] ragged_f32 inputs placed from GPU memory, {shift} bytes off", flush=True)
    s = H.GpuSession(cfg, full, cap=64 << 20, device_inputs=True)
    try:
        want, _ = s.run()
        slab = torch.zeros(s.in_slab.numel() + 64, dtype=torch.uint8, device="cuda:0")
        slab[shift:shift + s.in_slab.numel()] = s.in_slab
        torch.cuda.synchronize()
        moved = slab.data_ptr() + shift - s.in_slab.data_ptr()
        s.in_ptrs = B.ptr_array([p + moved if p else 0 for p in s.in_ptrs])
        s.dev.fill_(0xFF)
        torch.cuda.synchronize()
        out, _ = s.run()
        np.testing.assert_array_equal(out["y"], want["y"])
    finally:
        s.close()


def test_inputs_are_placed_in_their_order():
    """A source inside the device buffer is read after the inputs before it have been placed."""
    n = 1 << 16
    tg = B.tn_taskgraph_create()
    ins = [B.tn_taskgraph_add_input(tg, B.TN_F32, 1, n, B.TN_DEVICE) for _ in range(2)]
    B.tn_taskgraph_mark_output(tg, B.tn_taskgraph_add_op(tg, B.TN_OP_ADD, B.tn_op_params(), ins, B.TN_F32, 1, n))
    cap = 1 << 20
    mg = B.tn_compile(tg, None, cap, None)
    dev = torch.zeros(cap, dtype=torch.uint8, device="cuda:0")
    src = torch.arange(n, dtype=torch.float32, device="cuda:0")
    out = torch.zeros(n, dtype=torch.float32).pin_memory()
    torch.cuda.synchronize()
    st = [torch.cuda.Stream() for _ in range(3)]
    ex = B.tn_executor_create(mg, dev.data_ptr(), cap, 0, 0, [st[0].cuda_stream], st[1].cuda_stream, st[2].cuda_stream)
    try:
        print("[case] second input placed from where the first one went", flush=True)
        B.tn_executor_place_inputs(ex, [src.data_ptr(), dev.data_ptr() + B.tn_memgraph_vertex(mg, ins[0]).offset, 0])
        B.tn_execute(ex, [0, 0, 0], [out.data_ptr()], None)
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(tg)
    np.testing.assert_array_equal(out.numpy(), 2.0 * np.arange(n, dtype=np.float32))
