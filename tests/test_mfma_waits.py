"""The bf16 GEMM kernels issue their matrix instructions through inline assembly, which the compiler's hazard logic does not
see: the waits around them are the source's own.  Here the built kernels are read back (llvm-objdump on the library that was
built from csrc/) and every path is followed: whatever copies and spills the compiler put around the k-loop, no instruction
touches an accumulator between the matrix instruction that writes it and a wait, and no matrix instruction reads what a
vector instruction has written within the two wait states before it."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2512_12977_amd as vlc

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# v_mfma_f32_16x16x32_bf16 takes 4 passes; gfx950 wants 4 more wait states before anything but another MFMA's addend touches the result
NEED_AFTER = 8
NEED_BEFORE = 2
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+?(?: <.*\+0x([0-9a-f]+)>)?$")


def registers(operand):
    """Vector and accumulation registers of an operand (or of several, separated by spaces) as a bit set."""
    bits = 0
    for part in operand.split():
        m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", part)
        if m:
            lo = int(m[2] or m[3])
            for r in range(lo, int(m[4] or lo) + 1):
                bits |= 1 << (r + (256 if m[1] == "a" else 0))
    return bits


def parse(text):
    """{function: [(address, mnemonic, [register sets of the operands], first operand's text, branch target or None)]}"""
    functions, name = {}, None
    for line in text.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
        if head:
            name = head[1]
            functions[name] = []
            continue
        m = LINE.match(line)
        if m and name:
            ops = [o.strip() for o in m[2].split(",")] if m[2] else []
            functions[name].append((int(m[3], 16), m[1], [registers(o) for o in ops], ops[0] if ops else "",
                                    int(m[4], 16) if m[4] else None))
    return functions


def successors(code):
    start, index = code[0][0], {c[0]: i for i, c in enumerate(code)}
    succ = []
    for i, (_, mnemonic, _, _, target) in enumerate(code):
        assert not mnemonic.startswith(("s_setpc", "s_swappc", "s_call")), mnemonic
        nxt = []
        if mnemonic != "s_endpgm":
            if mnemonic.startswith(("s_cbranch", "s_branch")):
                nxt.append(index[start + target])
            if mnemonic != "s_branch" and i + 1 < len(code):
                nxt.append(i + 1)
        succ.append(nxt)
    return succ


def wait_states(mnemonic, first):
    return int(first, 0) + 1 if mnemonic == "s_nop" else 1


def follow(code, step, empty):
    """Forward over all paths to a fixed point: step(i, state) -> state behind instruction i; states are tuples of bit sets,
    united where paths meet."""
    succ, before, work = successors(code), [None] * len(code), [(0, empty)]
    while work:
        i, state = work.pop()
        if before[i] is not None:
            joined = tuple(a | b for a, b in zip(before[i], state))
            if joined == before[i]:
                continue
            state = joined
        before[i] = state
        after = step(i, state)
        work.extend((k, after) for k in succ[i])


def touched_before_the_wait(code):
    """Instructions that touch a matrix instruction's result on a path without a wait of NEED_AFTER states in between
    (only s_nop counts: what the compiler puts in between is not the source's to rely on)."""
    bad = set()

    def step(i, state):
        pending, = state
        _, mnemonic, regs, first, _ = code[i]
        if mnemonic.startswith("v_mfma"):
            d, a, b, c = regs[:4]
            if (a | b) & pending or (c & pending and c != d):
                bad.add(i)
            return (pending | d,)
        if mnemonic == "s_nop":
            return (0 if wait_states(mnemonic, first) >= NEED_AFTER else pending,)
        touched = pending
        for r in regs:
            if r & touched:
                bad.add(i)
                pending &= ~r
        return (pending,)

    follow(code, step, (0,))
    return bad


def read_too_early(code):
    """Matrix instructions that read a register which a vector instruction wrote less than NEED_BEFORE wait states earlier."""
    bad = set()

    def step(i, state):
        _, mnemonic, regs, first, _ = code[i]
        if mnemonic.startswith("v_mfma"):
            if any(r & written for r in regs[1:4] for written in state):
                bad.add(i)
        wrote = regs[0] if regs and mnemonic.startswith("v_") and not mnemonic.startswith("v_mfma") else 0
        states = wait_states(mnemonic, first)
        return ((wrote,) + state + (0,) * NEED_BEFORE)[:NEED_BEFORE] if states == 1 else ((0,) * states + state)[:NEED_BEFORE]

    follow(code, step, (0,) * NEED_BEFORE)
    return bad


def test_checks_see_planted_mistakes():
    """Both checks on a few lines of code: a store before the wait, one behind it, one on a branch round it; a fragment copied
    right in front of a matrix instruction."""
    def lines(*instr):
        out = ["0000000000000100 <f>:"]
        for k, s in enumerate(instr):
            target = s.split("-> ")[1] if "-> " in s else None
            out.append("\t%s // %012X: 00000000%s" % (s.split(" ->")[0], 0x100 + 4 * k, " <f+0x%x>" % (4 * int(target)) if target else ""))
        return parse("\n".join(out))["f"]

    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"
    store = "scratch_store_dwordx4 off, a[0:3], off"
    assert touched_before_the_wait(lines(mfma, store, "s_nop 7", "s_endpgm")) == {1}
    assert not touched_before_the_wait(lines(mfma, mfma, "s_nop 7", store, "s_endpgm"))
    assert touched_before_the_wait(lines(mfma, "s_nop 6", store, "s_endpgm")) == {2}
    assert touched_before_the_wait(lines(mfma, "s_cbranch_scc1 1 -> 3", "s_nop 15", store, "s_endpgm")) == {3}
    assert touched_before_the_wait(lines(mfma, "v_mfma_f32_16x16x32_bf16 a[4:7], a[0:3], v[8:11], a[4:7]", "s_endpgm")) == {1}
    assert read_too_early(lines("v_mov_b32_e32 v9, v1", "s_nop 0", mfma, "s_endpgm")) == {2}
    assert not read_too_early(lines("v_mov_b32_e32 v9, v1", "s_nop 1", mfma, "s_endpgm"))
    assert read_too_early(lines("v_accvgpr_write_b32 a0, 0", mfma, "s_endpgm")) == {1}


@pytest.fixture(scope="module")
def gemm_kernels(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(vlc.lib_path(), d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    found = {}
    for f in sorted(d.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", f.name], cwd=d, check=True, capture_output=True, text=True).stdout
        found.update({n: c for n, c in parse(text).items() if "gemm_bf16_kernel" in n})
    assert len(found) > 50
    return found


def test_waits_around_the_matrix_instructions(gemm_kernels):
    bad = {}
    for name, code in gemm_kernels.items():
        assert sum(c[1] == "v_mfma_f32_16x16x32_bf16" for c in code) > 0, name
        early, late = touched_before_the_wait(code), read_too_early(code)
        if early or late:
            bad[re.search(r"gemm_bf16_kernelI(.*?)EEv", name)[1]] = [code[i][1] for i in sorted(early | late)]
    assert not bad, bad
