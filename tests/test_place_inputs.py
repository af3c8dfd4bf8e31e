"""Inputs in GPU memory that lie one behind the other are placed by one copy, on the CPU (the fake GPU of test_dispatch): every order and
spacing of the sources places the same bytes."""
import ctypes as C
import random

import pytest

from paper_2405_16283_amd import binding as B

from test_dispatch import ALIGN, DEVICE_COPY, D2H, H2D, fake  # noqa: F401  (fixture)


@pytest.mark.parametrize("spacing", ["packed", "packed_reversed", "gaps", "shuffled"])
@pytest.mark.parametrize("rows,cols", [(64, 64), (1024, 1024), (3, 5), (1100, 2048)])
def test_sources_in_any_order_arrive(fake, rows, cols, spacing):  # noqa: F811
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
    for k, p in enumerate(ptrs):
        C.memset(p, 0, size)
        C.memmove(p, (k + 1).to_bytes(4, "little"), 4)
        C.memmove(p + size - 4, (1000 + k).to_bytes(4, "little"), 4)
    ex = B.tn_executor_create(mg, dev, n * step, 0, 0, [fake.fake_stream(0)], fake.fake_stream(H2D), fake.fake_stream(D2H))
    try:
        C.memset(dev, 0xEE, n * step)
        B.tn_executor_place_inputs(ex, ptrs)
        where = {}
        for m in range(B.tn_memgraph_num_vertices(mg)):
            v = B.tn_memgraph_vertex(mg, m)
            if v.kind == B.TN_MG_INPUT:
                where[v.src] = dev + v.offset
        for k, v in enumerate(vids):
            assert C.c_uint32.from_address(where[v]).value == k + 1
            assert C.c_uint32.from_address(where[v] + size - 4).value == 1000 + k
    finally:
        B.tn_executor_destroy(ex)
        B.tn_memgraph_destroy(mg)
        B.tn_taskgraph_destroy(tg)
