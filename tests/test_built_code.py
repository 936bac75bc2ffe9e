"""What the kernels' assembly MFMAs rely on, read from the built library's own code objects (no GPU needed): the compiler keeps
wait states and handles scratch around its own MFMAs only, so a register copy or a reload that it puts beside one written in
assembly would give wrong results without an error.
  - no kernel has scratch memory or spilled vector registers;
  - along every path, an MFMA comes at least two wait states after a vector ALU write of one of its operands, and nothing touches
    its result within the next eight unless another MFMA has taken it as accumulator input, for which the matrix pipe waits by
    itself (the distances that the compiler keeps around the 16x16x32 MFMA; 16 for the 32x32x16 one);
  - M0, which a copy to LDS takes over from the copy before it, is written by the copies alone.
And what a time depends on: the copying waves of whole 32 x 64 tiles reach the copies behind a barrier without a branch."""
import os
import re
import shutil
import struct
import subprocess

import pytest

BIN = "/opt/rocm/llvm/bin"
BEFORE, AFTER = 2, {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x16_bf16": 16}
# its loop fills the register file: one register lives in scratch outside the loop
ONE_SPILL = "mfma32_ceiling_kernel"

REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for kind, one, lo, hi in REG.findall(text):
        out |= {(kind, i) for i in ([int(one)] if one else range(int(lo), int(hi) + 1))}
    return out


def parse(listing):
    """Disassembly -> {function: [(mnemonic, operands, index of the branch target)]}."""
    functions = {}
    for block in re.split(r"\n(?=[0-9a-f]+ <[^>]+>:)", listing):
        head = re.match(r"([0-9a-f]+) <([^>]+)>:", block)
        if not head:
            continue
        base, code, index = int(head.group(1), 16), [], {}
        for line in block.splitlines()[1:]:
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<\S+?(?:\+0x([0-9a-f]+))?>)?", line)
            if m:
                index[int(m.group(3), 16)] = len(code)
                branch = m.group(1).startswith(("s_branch", "s_cbranch"))
                code.append((m.group(1), m.group(2).split(", "), base + int(m.group(4) or "0", 16) if branch else None))
        functions[head.group(2)] = [(name, ops, index[to] if to is not None else None) for name, ops, to in code]
    return functions


def _after(code, start, states, visit):
    """Calls visit(instruction) along every path for what comes within `states` wait states after instruction `start`, until it
    returns True on that path."""
    todo, best = [(start + 1, states)], {}
    while todo:
        i, left = todo.pop()
        if left <= 0 or i >= len(code) or best.get(i, 0) >= left:
            continue
        best[i] = left
        name, ops, to = code[i]
        if name == "s_nop":
            todo.append((i + 1, left - int(ops[0], 0) - 1))
            continue
        if visit(code[i]):
            continue
        if to is not None:
            todo.append((to, left - 1))
        if name not in ("s_branch", "s_endpgm"):
            todo.append((i + 1, left - 1))


def violations(code):
    bad = []
    for i, (name, ops, _) in enumerate(code):
        if name.startswith("v_mfma"):
            result = _regs(ops[0])

            def reads(ins):
                n, o, _ = ins
                if n.startswith("v_mfma"):
                    if result & (_regs(o[1]) | _regs(o[2])):
                        bad.append((i, name, ops, n, o))
                    return result <= _regs(o[0]) | _regs(o[3])     # (it waits by itself, and is looked at from there on)
                if result & _regs(", ".join(o)):
                    bad.append((i, name, ops, n, o))
                return False
            _after(code, i, AFTER[name], reads)
        elif name.startswith("v_") and not name.startswith(("v_cmp", "v_readlane", "v_readfirstlane", "v_nop")):
            written = _regs(ops[0])

            def feeds(ins):
                n, o, _ = ins
                if n.startswith("v_mfma") and written & _regs(", ".join(o[1:])):
                    bad.append((i, name, ops, n, o))
                return False
            _after(code, i, BEFORE, feeds)
    return bad


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    from paper_2510_00206_amd import binding
    if not all(shutil.which(f"{BIN}/{t}") for t in ("llvm-objcopy", "llvm-objdump", "llvm-readelf")):
        pytest.skip("the ROCm binary tools are not here")
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    d = tmp_path_factory.mktemp("code")
    subprocess.run([f"{BIN}/llvm-objcopy", f"--dump-section=.hip_fatbin={d}/fat", binding.LIB_PATH, os.devnull], check=True)
    fat, out = (d / "fat").read_bytes(), []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", fat):
        at = m.start() + 32
        for _ in range(struct.unpack_from("<Q", fat, at - 8)[0]):
            offset, size, length = struct.unpack_from("<QQQ", fat, at)
            target, at = fat[at + 24:at + 24 + length], at + 24 + length
            if b"gfx950" in target and size:
                out.append(str(d / f"{len(out)}.o"))
                with open(out[-1], "wb") as f:
                    f.write(fat[m.start() + offset:m.start() + offset + size])
    return out


def test_nothing_spills(objects):
    kernels = {}
    for o in objects:
        notes = subprocess.run([f"{BIN}/llvm-readelf", "--notes", o], check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n  - (?=\.agpr_count)", notes)[1:]:
            field = lambda f: re.search(rf"\.{f}:\s+(\S+)", k).group(1)
            kernels[field("name")] = (int(field("private_segment_fixed_size")), int(field("vgpr_spill_count")))
    assert len(kernels) > 50
    assert {n: v for n, v in kernels.items() if v != (0, 0) and not (ONE_SPILL in n and v == (8, 1))} == {}


@pytest.fixture(scope="module")
def functions(objects):
    dump = [f"{BIN}/llvm-objdump", "-d", "--no-show-raw-insn"]
    return [f for o in objects for f in parse(subprocess.run(dump + [o], check=True, capture_output=True, text=True).stdout).items()]


def test_mfma_wait_states(functions):
    assert sum(c[0].startswith("v_mfma") for _, code in functions for c in code) > 4000
    for name, code in functions:
        assert violations(code) == [], name


def test_only_the_copies_write_m0(functions):
    writes = 0
    for name, code in functions:
        for i, (mnemonic, ops, _) in enumerate(code):
            if ops[0] == "m0":
                writes += 1
                assert (mnemonic, code[i + 1][0], code[i + 2][0]) == ("s_mov_b32", "s_nop", "global_load_lds_dwordx4"), (name, i)
    assert writes > 100


def _straight_loops(code):
    """Loops that hold a barrier and copies behind it, and nothing else but scalar arithmetic."""
    n = 0
    for i, (_, _, to) in enumerate(code):
        body = [c[0] for c in code[to:i]] if to is not None and to < i else []
        n += "s_barrier" in body and "global_load_lds_dwordx4" in body[body.index("s_barrier"):] and \
            all(c.startswith(("s_", "global_load_lds")) and not c.startswith(("s_branch", "s_cbranch")) for c in body)
    return n


def test_copies_of_whole_narrow_tiles_follow_the_barrier(functions):
    """In (2) those of the token and of the out waves; in (5), where that is no faster, neither."""
    tile = r"_kernelINS_4RingILi32ELi64E(Li\d+E){5}Li1EE"
    forward = [code for name, code in functions if re.search(rf"ring_gemm{tile}ELb0E", name)]
    backward = [code for name, code in functions if re.search(rf"ring_gemm{tile}ELb1E|ring_strips{tile}", name)]
    assert len(forward) == 2 and len(backward) >= 4          # both sizes of the adapter table; with strips both ranks
    assert {_straight_loops(code) for code in forward} == {2} and {_straight_loops(code) for code in backward} == {0}


def test_kernels_of_whole_narrow_tiles(functions):
    """Of 32 x 64 tiles by themselves only what a launch can choose is built: waves in rows and columns, stages, copying waves, slabs to a stage."""
    found = {m.groups() for name, _ in functions if (m := re.search(r"ring_gemm_kernelINS_4RingILi32ELi64E((?:Li\d+E){6})EELb(\d)E", name))}
    of = lambda *v: "".join(f"Li{x}E" for x in v)
    assert found == {(of(2, 2, 6, 1, 2, 1), "0"), (of(1, 2, 6, 1, 1, 1), "1"), (of(2, 2, 6, 2, 2, 1), "1"), (of(2, 2, 3, 1, 2, 2), "1")}


@pytest.mark.parametrize("body,expected", [
    ("\tv_mov_b32_e32 v4, v9 // 100:\n\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3] // 104:\n\ts_nop 15 // 10C:\n", 1),
    ("\tv_mov_b32_e32 v4, v9 // 100:\n\ts_nop 1 // 102:\n\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3] // 104:\n", 0),
    ("\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3] // 100:\n\ts_nop 6 // 108:\n\tv_add_f32_e32 v9, v0, v9 // 10C:\n", 1),
    ("\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3] // 100:\n\ts_nop 7 // 108:\n\tv_add_f32_e32 v9, v0, v9 // 10C:\n", 0),
    # behind a jump: the instruction that follows in the listing is not the one that follows in time
    ("\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3] // 100:\n\ts_branch 1 // 108: BF820001 <f+0x10>\n"
     "\tv_mov_b32_e32 v0, 0 // 10C:\n\ts_nop 7 // 110:\n\tv_mov_b32_e32 v0, 0 // 114:\n", 0),
    ("\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[0:3] // 100:\n\ts_cbranch_scc1 1 // 108: BF820001 <f+0x10>\n"
     "\ts_endpgm // 10C:\n\tds_write_b128 v9, v[0:3] // 110:\n", 1),
])
def test_the_check_itself(body, expected):
    assert len(violations(parse("\n0000000000000100 <f>:\n" + body)["f"])) == expected
