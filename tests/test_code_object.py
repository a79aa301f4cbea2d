"""Properties of the compiled kernels that no result shows reliably: read from the gfx950 code objects in libfier.so."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2508_08256_amd import binding as B
from paper_2508_08256_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _sections(elf):
    shoff = struct.unpack_from("<Q", elf, 0x28)[0]
    size, n, names = struct.unpack_from("<HHH", elf, 0x3A)
    sec = [struct.unpack_from("<IIQQQQ", elf, shoff + i * size) for i in range(n)]
    text = lambda at: elf[at:elf.index(b"\0", at)].decode()  # noqa: E731
    return {text(sec[names][4] + s[0]): elf[s[4]:s[4] + s[5]] for s in sec}


def _code_objects(lib):
    """The gfx950 ELF images of a library: one offload bundle per translation unit."""
    fat, magic, at, out = _sections(open(lib, "rb").read())[".hip_fatbin"], b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (at := fat.find(magic, at)) >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", fat, at + len(magic))[0]):
            off, size, name = struct.unpack_from("<QQQ", fat, pos)
            if size and b"gfx950" in fat[pos + 24:pos + 24 + name]:
                out.append(fat[at + off:at + off + size])
            pos += 24 + name
        at += len(magic)
    return out


@pytest.fixture(scope="module")
def objects():
    objs = _code_objects(B.LIB_PATH)
    assert len(objs) >= len(build.SOURCES)
    return objs


def _kernels(obj):
    note = _sections(obj)[".note"]
    name, desc, _ = struct.unpack_from("<III", note)
    at = 12 + (name + 3) // 4 * 4
    return msgpack.unpackb(note[at:at + desc])["amdhsa.kernels"]


def test_no_kernel_spills_registers(objects):
    """Scratch per lane means registers written to memory and read back."""
    bad = [(k[".name"], k[".private_segment_fixed_size"]) for o in objects for k in _kernels(o)
           if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]
    assert not bad, bad


def test_every_variant_of_the_gather_has_both_kinds_of_loads(objects):
    """step_attend_kernel<type, heads, ranges, STREAM, layers>: the launcher's rule on STREAM has both to choose from."""
    names = " ".join(k[".name"] for o in objects for k in _kernels(o))
    for dt in (0, 1):
        for heads in range(1, 9):
            for ranges in (1, 2, 4, 8):
                for stream in (0, 1):
                    for layers in ("8OneLayer", "10LayerBatch"):
                        assert f"18step_attend_kernelILi{dt}ELi{heads}ELi{ranges}ELb{stream}ENS_{layers}E" in names


def test_registers_allow_the_workgroups_the_grids_are_sized_for(objects):
    """The launchers cut the step's work into as many workgroups of four wavefronts as the 256 CUs hold at once: 512 registers
    per SIMD lane, given out in eights, for one wavefront of each workgroup of the CU."""
    seen = set()
    for k in (k for o in objects for k in _kernels(o)):
        want = None
        if m := re.match(r"_ZN4fier12score_kernelILi(\d)ELi(\d)ELb1ELb\dELb(\d)ENS_", k[".name"]):
            want = 6 if m[3] == "0" else 5 if int(m[2]) <= 7 else 4  # 32-token groups; longer ones
        elif m := re.match(r"_ZN4fier18step_attend_kernelILi(\d)ELi(\d)E", k[".name"]):
            want = 5 if int(m[2]) <= 2 else 4
        if want:
            fit = 512 // (-(-k[".vgpr_count"] // 8) * 8)
            assert fit >= want, (k[".name"], k[".vgpr_count"])
            seen.add((k[".name"][9:14], m[1], m[2]))
    assert len(seen) == 2 * 2 * 8


def _vgprs(operand):
    m = re.fullmatch(r"v(\d+)|v\[(\d+):(\d+)\]", operand)
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def _too_close(lines):
    """Cross-lane reads (permlane swaps, DPP) of a vector register less than two wait states after a vector instruction
    wrote it.  The hardware does not wait by itself; the compiler does not count inline assembly.  Straight-line code."""
    past, bad, seen = [], [], 0        # past: (wait states, registers written) of the last few instructions
    for line in lines:
        line = line.split("//")[0].strip()
        if line.endswith(">:"):
            kernel, past = line, []
            continue
        op, _, rest = line.partition(" ")
        if not op or not rest and not op.startswith("s_"):
            continue
        args = [a.split()[0] for a in rest.split(",") if a.strip()]
        swap = op.startswith("v_permlane") and "_swap" in op
        reads = set()
        if swap:
            reads = _vgprs(args[0]) | _vgprs(args[1])
        elif "_dpp" in op:
            reads = _vgprs(args[1])
        if reads:
            seen += 1
            waited = 0
            for states, writes in reversed(past):
                if waited >= 2:
                    break
                if writes & reads:
                    bad.append((kernel, line, waited))
                    break
                waited += states
        writes = set()
        if op.startswith("v_") and args:
            writes = _vgprs(args[0]) | (_vgprs(args[1]) if swap else set())
        past = (past + [(int(args[0]) + 1 if op == "s_nop" else 1, writes)])[-4:]
    return seen, bad


def test_cross_lane_reads_keep_their_distance(objects, tmp_path):
    assert _too_close(["<k>:", "v_pk_max_f16 v1, v2, v3", "s_nop 0", "v_permlane32_swap_b32_e32 v0, v1"])[1]
    assert not _too_close(["<k>:", "v_pk_max_f16 v1, v2, v3", "s_nop 1", "v_permlane32_swap_b32_e32 v0, v1"])[1]
    assert _too_close(["<k>:", "v_add_u32_e32 v1, v2, v3", "v_mov_b32_dpp v0, v1 quad_perm:[1,0,3,2]"])[1]
    seen = 0
    for i, obj in enumerate(objects):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(obj)
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)], check=True,
                             capture_output=True, text=True).stdout
        n, bad = _too_close(out.splitlines())
        assert not bad, bad[:4]
        seen += n
    assert seen > 100
