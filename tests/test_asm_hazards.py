"""What the compiler cannot know about the instructions that the tile-product kernels write as inline assembly, checked in the listings of the
kernels as they are built, along every path of control flow.  The compiler does not see that such a statement is an MFMA, or a load that
takes its descriptor from scalar registers, and leaves out the wait states between it and its neighbours."""
import os
import re
import subprocess

import pytest

from paper_2405_16283_amd import build

SGPR_STATES = 5  # wait states between a vector instruction that writes a scalar register and a load that reads it


def _registers(text):
    """{(file, number)} of the registers an operand names."""
    out = set()
    for kind, one, lo, hi in re.findall(r"\b([sva])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        out |= {(kind, i) for i in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1))}
    return out


def _kernels(path):
    """{kernel: blocks}; a block: label, instructions (opcode, operands, inside an asm statement), where it goes."""
    kernels, blocks, inside = {}, None, False
    for line in open(path):
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
            continue
        s = line.split(";")[0].strip()
        if s.startswith("_Z") and s.endswith(":"):
            blocks = kernels.setdefault(s[:-1], [dict(label=s[:-1], code=[], jump=None, falls=True)])
        elif s.startswith(".Lfunc_end"):
            blocks = None
        elif blocks is None or not s or (s.startswith(".") and not s.endswith(":")):
            continue
        elif s.endswith(":"):
            blocks.append(dict(label=s[:-1], code=[], jump=None, falls=True))
        else:
            op, _, rest = s.partition(" ")
            blocks[-1]["code"].append((op, [a.strip() for a in re.split(r",(?![^\[]*\])", rest)], inside, s))
            if op.startswith("s_cbranch") or op in ("s_branch", "s_endpgm"):
                blocks[-1].update(jump=rest.strip() or None, falls=op.startswith("s_cbranch"))
                blocks.append(dict(label=None, code=[], jump=None, falls=True))
    return kernels


def _flow(blocks, transfer, merge):
    """Runs `transfer` over the blocks until the states at their starts (empty at first) no longer grow."""
    index = {b["label"]: i for i, b in enumerate(blocks) if b["label"]}
    start = [{} for _ in blocks]
    todo = list(range(len(blocks)))
    while todo:
        i = todo.pop(0)
        end = transfer(blocks[i], dict(start[i]))
        for j in ([i + 1] if blocks[i]["falls"] and i + 1 < len(blocks) else []) + ([index[blocks[i]["jump"]]] if blocks[i]["jump"] in index else []):
            new = merge(start[j], end)
            if new != start[j]:
                start[j] = new
                if j not in todo:
                    todo.append(j)


def _accumulators_not_waited_for(blocks):
    """Accesses of an accumulator that an MFMA in assembly has written, without a wait (a s_nop of 8 states and more) between."""
    found = set()

    def transfer(block, pending):
        for op, args, inside, text in block["code"]:
            if op.startswith("v_mfma"):
                if any(r in pending for a in args[1:3] for r in _registers(a)):
                    found.add(text)
                if inside:
                    pending.update({r: True for r in _registers(args[0])})
            elif op == "s_nop":
                if int(args[0], 0) >= 7:
                    pending = {}
            elif any(r in pending for a in args for r in _registers(a)):
                found.add(text)
        return pending

    _flow(blocks, transfer, lambda a, b: {**a, **b})
    return sorted(found)


def _scalars_read_too_early(blocks):
    """Loads in assembly that read a scalar register which a vector instruction wrote less than SGPR_STATES before."""
    found = set()

    def transfer(block, age):
        for op, args, inside, text in block["code"]:
            if inside and op.startswith(("buffer_", "global_")) and any(r in age for a in args for r in _registers(a)):
                found.add(text)
            step = int(args[0], 0) + 1 if op == "s_nop" else 1
            age = {r: n + step for r, n in age.items() if n + step < SGPR_STATES}
            for a in args[:2] if op.startswith("v_") else args[:1] if op.startswith("s_") else []:
                for r in _registers(a):
                    if r[0] == "s":
                        age.pop(r, None)
                        if op.startswith("v_") and (a is args[0] or "_co_" in op or "div_scale" in op or "_mad_" in op):
                            age[r] = 0
        return age

    _flow(blocks, transfer, lambda a, b: {r: min(a.get(r, 99), b.get(r, 99)) for r in {**a, **b}})
    return sorted(found)


@pytest.mark.parametrize("source", ["gemm_bf16", "gemm_small"])
def test_instructions_in_assembly_keep_their_distance(source, tmp_path):
    out = str(tmp_path / "listing.s")
    subprocess.run([build.HIPCC] + build.COMMON + build.DEVICE + ["-w", "--cuda-device-only", "-S", os.path.join(build.CSRC, source + ".hip"), "-o", out],
                   check=True, capture_output=True)
    scratch = [int(n) for n in re.findall(r"\.private_segment_fixed_size:\s+(\d+)", open(out).read())]
    assert scratch and not any(scratch)  # a spilled accumulator is stored wherever there is room, behind its MFMA
    kernels = _kernels(out)
    assert len(kernels) == len(scratch)
    n_loads = 0
    for name, blocks in kernels.items():
        n_loads += sum(inside and "lds" in text for b in blocks for _, _, inside, text in b["code"])
        assert not _accumulators_not_waited_for(blocks), name
        assert not _scalars_read_too_early(blocks), name
    assert n_loads > 0


def test_the_checks_see_what_they_look_for(tmp_path):
    """Hand-written listings with and without the faults."""
    def blocks(*code):
        p = tmp_path / "x.s"
        p.write_text("_Zk:\n" + "\n".join(code) + "\n\ts_endpgm\n.Lfunc_end0:\n")
        return _kernels(str(p))["_Zk"]

    mfma = ("\t;;#ASMSTART", "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "\t;;#ASMEND")
    read = "\tv_accvgpr_read_b32 v9, a2"
    assert _accumulators_not_waited_for(blocks(*mfma, read))
    assert _accumulators_not_waited_for(blocks(*mfma, "\ts_cbranch_scc0 .LBB0_1", "\ts_nop 15", ".LBB0_1:", read))
    assert not _accumulators_not_waited_for(blocks(*mfma, *mfma, "\ts_nop 15", read))
    assert not _accumulators_not_waited_for(blocks(*mfma, "\tv_accvgpr_read_b32 v9, a4"))
    load = ("\t;;#ASMSTART", "\ts_add_u32 m0, s9, 0", "\ts_nop 0", "\tbuffer_load_dwordx4 v0, s[4:7], s8 offen lds", "\t;;#ASMEND")
    assert _scalars_read_too_early(blocks("\tv_readfirstlane_b32 s8, v1", *load))
    assert not _scalars_read_too_early(blocks("\tv_readfirstlane_b32 s8, v1", "\ts_nop 4", *load))
    assert not _scalars_read_too_early(blocks("\tv_readfirstlane_b32 s8, v1", "\ts_lshl_b32 s8, s8, 4", *load))
    assert not _scalars_read_too_early(blocks("\tv_readfirstlane_b32 s10, v1", *load))
