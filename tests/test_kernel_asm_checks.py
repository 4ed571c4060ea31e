"""Checks on the compiler's output for the kernels that issue LDS reads behind the compiler's back.

The large-agent kernels place some operand reads by hand: a `ds_read` inside an asm statement, and later an
`s_waitcnt lgkmcnt(n)` asm statement that ties the registers.  Between the two the compiler believes the registers
already hold their values, so nothing it emits may read or write them before the wait that covers them (a copy
would take stale data, a reuse would be overwritten when the read arrives).  This test compiles the three
large-agent units to gfx950 assembly with the build's flags and scans every kernel in emission order: LDS reads
of a wave complete in order, so after a hand-written `lgkmcnt(n)` only the youngest n hand-issued reads are still
in flight."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import __graft_entry__ as entry      # noqa: E402


def _regs(tok):
    tok = tok.strip()
    m = re.match(r"v\[(\d+):(\d+)\]", tok)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"v(\d+)$", tok)
    return {int(m.group(1))} if m else set()


def scan_in_flight(text):
    """Returns (number of hand-issued reads seen, list of offending lines)."""
    in_asm, flight, issued, bad, kernel = False, [], 0, [], ""
    for ln, line in enumerate(text.split("\n"), 1):
        t = line.strip()
        if re.match(r"^_Z\w+:", line):
            kernel, flight = line.split(":")[0], []
        if t.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if t.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not t or t[0] in ";.":
            continue
        op = t.split()[0]
        ops = t.split(None, 1)[1].split(",") if " " in t else []
        wait = re.search(r"lgkmcnt\((\d+)\)", t) if op == "s_waitcnt" else None
        if in_asm:
            if op.startswith("ds_read"):
                flight.append((_regs(ops[0]), ln))
                issued += 1
            elif wait:
                n = int(wait.group(1))
                flight = flight[len(flight) - n:] if n else []
            continue
        if wait and int(wait.group(1)) == 0:      # the compiler's own full wait covers them as well
            flight = []
            continue
        if op == "s_endpgm":
            flight = []
            continue
        used = set()
        for o in ops:
            used |= _regs(o.split()[0] if o.strip() else "")
        for rs, at in flight:
            if used & rs:
                bad.append("%s line %d: '%s' touches v%s, in flight since line %d" % (kernel[:60], ln, t[:60],
                                                                                   sorted(used & rs)[:4], at))
                break
    return issued, bad


def test_scanner_sees_a_planted_touch():
    text = ("_Zfoo:\n\t;;#ASMSTART\n\tds_read_b128 v[4:7], v1 offset:0\n\t;;#ASMEND\n\tv_mov_b32_e32 v9, v5\n"
            "\t;;#ASMSTART\n\ts_waitcnt lgkmcnt(0)\n\t;;#ASMEND\n\tv_mov_b32_e32 v9, v5\n")
    issued, bad = scan_in_flight(text)
    assert issued == 1 and len(bad) == 1 and "line 5" in bad[0]


@pytest.fixture(scope="module")
def large_units(tmp_path_factory):
    """{unit: its assembly} of the three large-agent units."""
    units = ["large_agent_dp32.hip", "large_agent_dp64.hip", "large_agent_dp128.hip"]
    flags = [f for f in entry.HIPCC_FLAGS if f not in ("-shared", "-Wall")] + ["-fno-honor-nans", "-S", "--cuda-device-only"]
    procs = []
    for u in units:
        out = str(tmp_path_factory.mktemp("asm") / (u + ".s"))
        procs.append((u, out, subprocess.Popen(["hipcc"] + flags + [os.path.join(entry.CSRC, u), "-o", out],
                                               stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    texts = {}
    for u, out, p in procs:
        log, _ = p.communicate()
        assert p.returncode == 0, log
        texts[u] = open(out).read()
    return texts


def test_no_instruction_touches_a_register_with_a_hand_issued_read_in_flight(large_units):
    for u, text in large_units.items():
        issued, bad = scan_in_flight(text)
        assert issued > 100, "%s: the hand-issued reads were not found (%d)" % (u, issued)
        assert not bad, "\n".join(bad[:10])


def test_row_broadcast_with_bias_tables_keeps_its_loop_in_registers(large_units):
    """large_broadcast3_kernel with tables (MODE 1) up to 64 channels: 32 spilled registers took it from 38.8 to 46.1 us (104 units
    of 612 tokens x 96 agents, d = 64)."""
    sizes = []
    for u in ("large_agent_dp32.hip", "large_agent_dp64.hip"):
        kernel = ""
        for line in large_units[u].split("\n"):
            if re.match(r"^_Z\w+:", line):
                kernel = line.split(":")[0]
            elif line.strip().startswith("; ScratchSize:") and re.search(r"large_broadcast3_kernelINS_\d+Elem(BF16|F16)ELi1ELb0E", kernel):
                sizes.append(int(line.split(":")[1]))
    assert sizes == [0] * 4


# Backward kernels that the compiler may give scratch memory or accumulator-file copies: (kernel, element, padded width,
# role of the enums in backward_fused.h, agent bias) -> (bytes of scratch a lane may take, copies allowed)
ALLOWED = {
    # dK / dV at 128 channels, and fp32's agent kernels there: more than 256 registers, left at one block per CU
    ("token", "16", 128, 2, 0): (0, True), ("token", "16", 128, 2, 1): (0, True),
    ("agent", "32", 128, 0, 0): (0, True), ("agent", "32", 128, 1, 0): (0, True), ("agent", "32", 128, 2, 0): (0, True),
    ("agent", "32", 128, 0, 1): (0, True), ("agent", "32", 128, 1, 1): (0, True), ("agent", "32", 128, 2, 1): (0, True),
    # with a bias: dQ at 128 channels, dK / dV at 32 (all but 4 bytes in the form for large references, which few calls
    # take) and in fp32 at 64 and 128
    ("token", "16", 128, 1, 1): (200, False), ("token", "16", 32, 2, 1): (100, False),
    ("token", "32", 64, 2, 1): (130, False), ("token", "32", 128, 2, 1): (60, False),
    # agent kernels that take the tokens' side as well, with a bias: dK / dV at 32 channels (three blocks per CU), dQ at 128,
    # fp32 dK / dV at 64
    ("both", "16", 32, 2, 1): (12, False), ("both", "16", 128, 1, 1): (40, False), ("both", "32", 64, 2, 1): (24, False),
}


def _backward_kernel(symbol):
    """The key of ALLOWED for a mangled kernel name (None: another kernel)."""
    m = re.search(r"(fused_token|fused_agent|bias_agent)_kernelINS_\d+Elem(BF16|F16|F32)ELi(\d+)ELi(\d+)ELi\d+E(Lb(\d)E)?", symbol)
    if not m:
        return None
    kind = "token" if m.group(1) == "fused_token" else "both" if m.group(6) == "1" else "agent"
    bias = int(m.group(6)) if kind == "token" else int(m.group(1) == "bias_agent")      # agent kernels: group 6 is BOTH
    return kind, "32" if m.group(2) == "F32" else "16", int(m.group(3)), int(m.group(4)), bias


def test_backward_product_kernels_keep_their_accumulators_in_ordinary_registers(tmp_path):
    """The MFMA kernels of the backward pass ask for two blocks per CU, i.e. at most 256 registers per lane: then
    the compiler has no reason to place MFMA accumulators in the accumulator file, and every copy in or out of it
    (`v_accvgpr_read` / `_write`) would be a vector instruction spent on nothing.  The recomputing kernels are
    bound by their vector arithmetic, so the copies cost a tenth of their time when they were there.  Registers spilled
    to scratch memory cost more: 40 of them took the dK / dV kernel of 32 channels from 58 to 77 us.  What has either is
    named above."""
    units = ["backward_fused_kernels.hip", "backward_kernels.hip", "backward_bias_bf16.hip", "backward_bias_f16.hip",
             "backward_f32.hip"]
    flags = [f for f in entry.HIPCC_FLAGS if f not in ("-shared", "-Wall")] + ["-S", "--cuda-device-only"]
    procs = []
    for u in units:
        out = str(tmp_path / (u + ".s"))
        procs.append((u, out, subprocess.Popen(["hipcc"] + flags + [os.path.join(entry.CSRC, u), "-o", out],
                                               stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    seen = set()
    for u, out, p in procs:
        log, _ = p.communicate()
        assert p.returncode == 0, log
        text = open(out).read()
        assert text.count("v_mfma_f32_16x16x") > 50, u
        kernel, copies, scratch = "", {}, {}
        for line in text.split("\n"):
            if re.match(r"^_Z\w+:", line):
                kernel = line.split(":")[0]
            elif "v_accvgpr" in line:
                copies[kernel] = copies.get(kernel, 0) + 1
            elif line.strip().startswith("; ScratchSize:"):
                scratch[kernel] = int(line.split(":")[1])
        assert len(scratch) >= 10, u
        for k, size in scratch.items():
            key = _backward_kernel(k)
            seen.add(key)
            allowed = ALLOWED.get(key, (0, False))
            assert size <= allowed[0], "%s: %d bytes of scratch in %s" % (u, size, k)
            assert allowed[1] or not copies.get(k), "%s: %d accumulator-file copies in %s" % (u, copies[k], k)
    assert seen > set(ALLOWED)      # every entry names a kernel that exists
