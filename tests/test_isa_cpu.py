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
def kernels(tmp_path_factory):
    """{kernel: its instructions in order, as text}"""
    if OBJDUMP is None:
        pytest.skip("no llvm-objdump beside hipcc")
    if not os.path.exists(taw.LIB_PATH):
        build()
    d = tmp_path_factory.mktemp("isa")
    shutil.copy(taw.LIB_PATH, d / "libtaw.so")
    subprocess.run([OBJDUMP, "--offloading", "libtaw.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(d)):
        if "amdgcn" not in f:
            continue
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


def test_large_tiles_move_between_stages_by_addition(kernels):
    """The fragments of a 256 x 256 tile are read at absolute LDS addresses.  Flipping the bit of the stage's size (0x8000) in them would
    hold only while the ring starts at a multiple of twice that, which nothing guarantees; adding the size holds for any start."""
    large = {name: text for name, text in kernels.items() if "v216gemm_pipe" in name or "v216gemm_dual" in name}
    assert len(large) == 8
    for name, text in large.items():
        assert not [t for t in text if t.startswith("v_xor") and "0x8000" in t], name
