"""Inputs in GPU memory that lie one behind the other in both places are placed by one copy of at most 8 MiB, on the CPU (the fake GPU of
test_dispatch): every order and spacing of the sources places the same bytes."""
import ctypes as C
import random

import numpy as np
import pytest

from paper_2405_16283_amd import binding as B

from test_dispatch import ALIGN, DEVICE_COPY, D2H, H2D, fake  # noqa: F401  (fixture)

MOST = 8 << 20  # bytes of a merged copy


def _words(address, n):
    return np.ctypeslib.as_array((C.c_uint32 * n).from_address(address))


@pytest.mark.parametrize("spacing", ["packed", "packed_reversed", "gaps", "shuffled"])
@pytest.mark.parametrize("rows,cols,packed_copies", [
    (128, 128, 1), (1024, 1024, 20), (768, 1024, 20), (1100, 2048, 40),
    (3, 5, 40), (64, 64, 40)])  # (tensors below 64 KiB are placed from the end of the buffer down)
def test_sources_in_any_order_arrive(fake, rows, cols, packed_copies, spacing):  # noqa: F811
    n, size = 40, rows * cols * 4
    step = (size + ALIGN - 1) // ALIGN * ALIGN
    tg = B.tn_taskgraph_create()
    vids = [B.tn_taskgraph_add_input(tg, B.TN_F32, rows, cols, B.TN_DEVICE) for _ in range(n)]
    mg = B.tn_compile(tg, None, n * step, None)
    fake.fake_reset(1)
    dev = fake.fake_alloc(n * step, 1)
    at = list(range(n))
    if spacing == "packed_reversed":
        at.reverse()
    elif spacing == "shuffled":
        random.Random(3).shuffle(at)
    pitch = step + (ALIGN if spacing == "gaps" else 0)
    src = fake.fake_alloc(n * pitch, 1)
    ptrs = [src + at[k] * pitch for k in range(n)]
    pattern = np.arange(rows * cols, dtype=np.uint32)
    for k, p in enumerate(ptrs):
        _words(p, rows * cols)[:] = pattern * np.uint32(2 * k + 1) + np.uint32(0x9E3779B1 * k % 2**32)
    ex = B.tn_executor_create(mg, dev, n * step, 0, 0, [fake.fake_stream(0)], fake.fake_stream(H2D), fake.fake_stream(D2H))
    try:
        C.memset(dev, 0xEE, n * step)
        B.tn_executor_place_inputs(ex, ptrs)
        log = np.zeros((fake.fake_log(None, 0), 6), dtype=np.int32)
        fake.fake_log(log.ctypes.data, len(log))
        assert set(log[:, 0]) == {DEVICE_COPY}
        where = {}
        copies, last = 0, (0, 0, MOST)  # source, destination and bytes of the copy at hand
        for m in range(B.tn_memgraph_num_vertices(mg)):
            v = B.tn_memgraph_vertex(mg, m)
            if v.kind != B.TN_MG_INPUT:
                continue
            where[v.src] = dev + v.offset
            s, d = ptrs[v.src], where[v.src]
            if last[0] + last[2] == s and last[1] + last[2] == d and last[2] + size <= MOST:
                last = (last[0], last[1], last[2] + size)
            else:
                copies, last = copies + 1, (s, d, size)
        assert log[:, 2].sum() == copies
        assert copies == packed_copies if spacing == "packed" else copies == n if spacing != "shuffled" else packed_copies <= copies <= n
        for k, v in enumerate(vids):
            assert np.array_equal(_words(where[v], rows * cols), _words(ptrs[k], rows * cols)), k
            assert _words(where[v], 2)[1] == (2 * k + 1 + 0x9E3779B1 * k) % 2**32
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(tg)
