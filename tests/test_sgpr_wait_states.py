"""The built GPU code keeps the wait states the hardware needs between a vector instruction that writes a scalar register
and a memory instruction that takes its address from it: 5 on gfx950, or the load may use the old address.  The compiler
sees to that for its own loads but does not look inside inline asm, and which scalar registers are fresh where a tile load
starts is up to register allocation; so the library as built is looked over, along every path of every kernel."""
import os
import re
import subprocess

import pytest

from paper_2409_15104_amd import binding

LLVM = "/opt/rocm/llvm/bin"
WAIT_STATES = 5


def sgprs(text):
    """Scalar registers named in an operand text."""
    found = set()
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        found.update(range(int(lo), int(hi) + 1))
    found.update(int(n) for n in re.findall(r"\bs(\d+)\b", text))
    return found


def written_by_vector(name, operands):
    if name.startswith(("v_readlane", "v_readfirstlane", "v_cmp")):
        return sgprs(operands[0])
    if name.startswith("v_") and len(operands) > 1 and ("_co_" in name or name.startswith(("v_mad_u64", "v_mad_i64", "v_div_scale"))):
        return sgprs(operands[1])
    return set()


def too_close(listing):
    """(kernel, load, writer, wait states) of every violation in a disassembly."""
    bad = []
    for kernel in re.split(r"\n(?=[0-9a-f]{16} <)", listing):
        head = re.match(r"[0-9a-f]{16} <(\S+)>:", kernel)
        if not head:
            continue
        code, at = [], {}
        for m in re.finditer(r"^\t(\S+)([^\n]*?)\s*// ([0-9A-F]{12}):([^\n]*)$", kernel, re.M):
            at[int(m[3], 16)] = len(code)
            code.append((m[1], [x.strip() for x in m[2].split(",")], int(m[3], 16), m[4]))
        start = min(at, default=0)
        before = [[] for _ in code]
        for i, (name, _, _, rest) in enumerate(code):
            if i + 1 < len(code) and name not in ("s_branch", "s_endpgm"):
                before[i + 1].append(i)
            target = re.search(r"<\S+?(?:\+0x([0-9a-f]+))?>", rest)
            if name.startswith(("s_branch", "s_cbranch")):
                before[at[start + int(target[1] or "0", 16)]].append(i)
        for i, (name, operands, _, _) in enumerate(code):
            if not name.startswith(("global_", "scratch_", "buffer_", "flat_")) or not sgprs(",".join(operands)):
                continue
            todo, seen = [(j, 0, frozenset(sgprs(",".join(operands)))) for j in before[i]], set()
            while todo:
                j, states, regs = todo.pop()
                if states >= WAIT_STATES or (j, states, regs) in seen:
                    continue
                seen.add((j, states, regs))
                n, ops, addr, _ = code[j]
                if written_by_vector(n, ops) & regs:
                    bad.append((head[1], "%s %s at %x" % (name, ", ".join(operands), code[i][2]), "%s %s" % (n, ", ".join(ops)), states))
                if n.startswith("s_") and not n.startswith(("s_cmp", "s_bitcmp", "s_store", "s_cbranch", "s_nop", "s_wait")):
                    regs = regs - sgprs(ops[0])      # a scalar instruction rewrites it
                states += int(ops[0], 0) + 1 if n == "s_nop" else 1
                todo.extend((k, states, regs) for k in before[j] if regs)
    return bad


def line(text, addr):
    return "\t%s // %012X: 00000000" % (text, addr)


def test_the_check_sees_what_is_too_close_and_nothing_else():
    def listing(gap):
        code = ["v_readlane_b32 s9, v1, 2", *gap, "global_load_lds_dword v4, s[8:9]", "s_endpgm"]
        return "%016x <k>:\n" % 0x100 + "\n".join(line(c, 0x100 + 8 * i) for i, c in enumerate(code))

    assert too_close(listing(["s_mov_b32 m0, s3", "s_nop 0"]))[0][3] == 2
    assert not too_close(listing(["s_nop 4"])) and too_close(listing(["s_nop 3"]))[0][3] == 4
    assert not too_close(listing(["s_add_u32 s8, s8, s2", "s_addc_u32 s9, s9, 0"]))
    loop = ["v_mov_b32 v0, 0", "global_load_lds_dword v4, s[8:9]", "s_nop 1", "v_readlane_b32 s8, v1, 1", "s_branch -5"]
    text = "%016x <k>:\n" % 0x100 + "\n".join(line(c, 0x100 + 8 * i) for i, c in enumerate(loop)) + " <k>"
    assert too_close(text)[0][3] == 2      # found around the back edge


def test_no_load_of_the_library_reads_a_scalar_register_too_soon(tmp_path):
    if not os.path.exists(binding.LIB_PATH):
        from paper_2409_15104_amd import build

        build.build()
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no disassembler")
    fat, dev = str(tmp_path / "fat.bin"), str(tmp_path / "dev.o")
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout  # noqa: E731
    run(LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, binding.LIB_PATH, os.devnull)
    run(LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat, "--output=" + dev,
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950")
    listing = run(LLVM + "/llvm-objdump", "-d", dev)
    assert listing.count("global_load_lds_dwordx4") > 100      # the tile loads are in it
    bad = too_close(listing)
    assert not bad, "\n".join("%s: %s after %s, %d wait states" % b for b in bad)
