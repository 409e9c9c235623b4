"""What the compiler cannot check for the kernels, in the instructions of the library that was built: it pads the hazards of the instructions
it knows with wait states, but does not look into a block of inline assembly."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2511_09741_amd.binding as taw
from paper_2511_09741_amd.build import HIPCC, build

OBJDUMP = next((p for p in (os.path.join(os.path.dirname(HIPCC), "..", "llvm", "bin", "llvm-objdump"), "/opt/rocm/llvm/bin/llvm-objdump")
                if os.path.exists(p)), None)


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """the folder and names of the device code objects in the library"""
    if OBJDUMP is None:
        pytest.skip("no llvm-objdump beside hipcc")
    if not os.path.exists(taw.LIB_PATH):
        build()
    d = tmp_path_factory.mktemp("isa")
    shutil.copy(taw.LIB_PATH, d / "libtaw.so")
    subprocess.run([OBJDUMP, "--offloading", "libtaw.so"], cwd=d, check=True, capture_output=True)
    return d, [f for f in sorted(os.listdir(d)) if "amdgcn" in f]


@pytest.fixture(scope="module")
def kernels(code_objects):
    """{kernel: its instructions in order, as text}"""
    d, files = code_objects
    out = {}
    for f in files:
        name = None
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=d, check=True, capture_output=True, text=True).stdout.splitlines():
            head = re.match(r"[0-9a-f]+ <(.*)>:", line)
            text = line.split("//")[0].strip()
            if head:
                name = head[1]
                out[name] = []
            elif name and text:
                out[name].append(text)
    return out


@pytest.fixture(scope="module")
def static_lds(code_objects):
    """{kernel: bytes of LDS beside what its launch asks for}"""
    d, files = code_objects
    out = {}
    for f in files:
        notes = subprocess.run([OBJDUMP.replace("objdump", "readelf"), "--notes", f], cwd=d, check=True, capture_output=True, text=True).stdout
        out.update((name, int(size)) for size, name in re.findall(r"\.group_segment_fixed_size: (\d+)\n(?:.*\n)*?\s+\.name:\s+(_Z\S+)", notes))
    return out


def m0_distances(instructions):
    """wait states between each load from global memory into LDS and the write of m0 (the place in LDS) before it"""
    out, since = [], None
    for text in instructions:
        op, _, args = text.partition(" ")
        if "_load_lds_" in op:
            out.append(since)
        if op.startswith("s_") and args.split(",")[0].strip() == "m0":
            since = 0
        elif since is not None:
            since += int(args, 0) + 1 if op == "s_nop" else 1
    return out


def test_m0_distances():
    assert m0_distances(["s_mov_b32 m0, s4", "global_load_lds_dwordx4 v0, s[0:1]"]) == [0]
    assert m0_distances(["s_add_u32 m0, s4, 0x1000", "s_nop 0", "global_load_lds_dword v0, s[0:1]", "global_load_lds_dword v1, s[0:1]"]) == [1, 2]
    assert m0_distances(["s_mov_b32 s4, m0", "global_load_lds_dwordx4 v0, s[0:1]"]) == [None]


def test_loads_into_lds_wait_for_m0(kernels):
    """A load into LDS needs one wait state after the scalar instruction that writes m0: hipcc puts s_nop 0 between the two where it
    places both; in inline assembly it is ours to place."""
    loads = {name: d for name, d in ((name, m0_distances(text)) for name, text in kernels.items()) if d}
    assert any("gemm_pipe" in n for n in loads) and any("attn_fwd" in n for n in loads) and any("mfma_loop" in n for n in loads)
    assert {name: d for name, d in loads.items() if any(x is None or x < 1 for x in d)} == {}


def test_flipped_stage_addresses(kernels, static_lds):
    """The 256 x 256 tiles go from one stage of A to the other by flipping a bit (0x8000) of absolute LDS addresses, which holds while the ring starts at
    a multiple of twice that: it is declared so, and whatever LDS a kernel has beside it is padded to that (and then too much to launch with)."""
    flip = [name for name, text in kernels.items() if any(t.startswith("v_xor") and "0x8000," in t for t in text)]
    assert len(flip) == 8
    assert {name: static_lds[name] for name in flip if static_lds[name] % 0x10000} == {}


def registers(operand):
    m = re.fullmatch(r"-?\|?([va])(\d+)\|?", operand) or re.fullmatch(r"-?([va])\[(\d+):(\d+)\]", operand)
    return [(m[1], r) for r in range(int(m[2]), int(m[m.lastindex]) + 1)] if m else []


def unwaited_reads(instructions):
    """instructions that use what an LDS read returns before a wait for it; LDS reads return in order, lgkmcnt(n) leaves the last n"""
    out, pending = [], []
    for text in instructions:
        op, _, args = text.partition(" ")
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            pending = []
        elif op == "s_waitcnt":
            n = re.search(r"lgkmcnt\((\d+)\)", args)
            if n:
                pending = pending[-int(n[1]):] if int(n[1]) else []
        else:
            operands = [a.split(" ")[0] for a in re.sub(r"offset\S*|nt\b", "", args).split(", ")]
            busy = {r for regs in pending for r in regs}
            if any(r in busy for a in operands for r in registers(a)):
                out.append(text)
            if op.startswith("ds_"):      # every LDS instruction counts, a write as one that returns nothing
                pending.append(registers(operands[0]) if op.startswith(("ds_read", "ds_bpermute")) else [])
            elif op.startswith(("s_load", "s_buffer_load", "s_memtime", "s_memrealtime")):
                pending.append([])
    return out


def test_unwaited_reads():
    read = "ds_read_b64 v[2:3], v1 offset:8"
    assert unwaited_reads([read, "v_add_u32_e32 v4, v4, v3"]) == ["v_add_u32_e32 v4, v4, v3"]
    assert unwaited_reads([read, "ds_read_b32 v5, v1", "s_waitcnt lgkmcnt(1)", "v_add_u32_e32 v4, v4, v3"]) == []
    assert unwaited_reads([read, "ds_read_b32 v5, v1", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v6, v5"]) == ["v_mov_b32_e32 v6, v5"]
    assert unwaited_reads([read, "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v3, 0"]) == ["v_mov_b32_e32 v3, 0"]      # taken as free while the read is under way
    assert unwaited_reads([read, "s_waitcnt vmcnt(0) lgkmcnt(0)", "v_mov_b32_e32 v3, 0"]) == []


def test_lds_reads_are_waited_for(kernels):
    """An LDS read in inline assembly counts as done when its block ends: the wait for it stands in the same block, or its register may be used,
    or handed to something else, while the read is under way."""
    assert {name: bad[:3] for name, bad in ((name, unwaited_reads(text)) for name, text in kernels.items()) if bad} == {}
