"""Wait states before the broadcast operands of the built synthesis kernels.

The synthesis reads its coefficients with v_fmac_f64_dpp row_newbcast, written in
inline assembly: the compiler's hazard handling does not look inside, and the two
wait states that such an operand needs after a vector instruction wrote it come
from an s_nop of the source's.  A register copy that a compiler put between the
two would be silently wrong, so this looks at the code that was built here: at
every such instruction, back along every way to it.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_1202_6522_amd import shtn as S

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEEDED = 2       # wait states from the write of an operand to its read by DPP
NEEDED_EXEC = 5  # from a vector write of EXEC to any DPP instruction


def parse(text):
    """Kernels of a disassembly: lists of (address, mnemonic, operands, branch target or None)."""
    kernels, base, code = {}, 0, None
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(\S+)>:$", line)
        if head:
            base = int(head[1], 16)
            code = kernels.setdefault(head[2], [])
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):[0-9A-F ]*(?:<\S+?(?:\+0x([0-9a-f]+))?>)?$", line)
        if m and code is not None:
            target = base + int(m[4] or "0", 16) if "branch" in m[1] else None
            code.append((int(m[3], 16), m[1], m[2], target))
    return kernels


def registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$|v(\d+)$", operand.strip())
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def hazards(code):
    """(number of broadcast instructions, those with an operand written too late before)."""
    at = {ins[0]: i for i, ins in enumerate(code)}
    into = {}
    for i, ins in enumerate(code):
        if ins[3] is not None:
            into.setdefault(at[ins[3]], []).append(i)

    def late(i, regs, waits):
        before = list(into.get(i, []))
        if i and code[i - 1][1] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before.append(i - 1)
        for j in before:
            op, args = code[j][1], code[j][2]
            if op.startswith("v_cmpx"):
                return j
            if waits < NEEDED and op.startswith("v_") and registers(args.split(",")[0]) & regs:
                return j
            w = waits + (int(args, 0) + 1 if op == "s_nop" else 1)
            if w < NEEDED_EXEC:
                k = late(j, regs, w)
                if k is not None:
                    return k
        return None

    n, bad = 0, []
    for i, (_, op, args, _) in enumerate(code):
        if "row_newbcast" in args:
            n += 1
            j = late(i, registers(args.split(",")[1].split()[0]), 0)
            if j is not None:
                bad.append((code[j], code[i]))
    return n, bad


def test_a_copy_before_a_broadcast_is_seen():
    good = """
0000000000000100 <k>:
\tv_mov_b32_e32 v4, v9       // 000000000100: 00000000
\ts_nop 1                    // 000000000104: 00000000
\tv_fmac_f64_dpp v[22:23], v[4:5], v[0:1] row_newbcast:0 row_mask:0xf bank_mask:0xf// 000000000108: 00000000 00000000
\ts_cbranch_scc1 65533       // 000000000110: 00000000 <k+0x8>
"""
    assert hazards(parse(good)["k"]) == (1, [])
    for bad in (good.replace("s_nop 1", "s_nop 0"),
                good.replace("\ts_cbranch", "\tv_mov_b32_e32 v5, v9 // 00000000010C: 00000000\n\ts_cbranch"),
                good.replace("v_mov_b32_e32 v4, v9", "v_cmpx_eq_u32_e32 v4, v9")):
        assert len(hazards(parse(bad)["k"])[1]) == 1, bad


def test_built_kernels_wait(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(S.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    seen = 0
    for name in sorted(os.listdir(tmp_path)):
        path = tmp_path / name
        if not name.endswith("gfx950") or b"k_legendre_synth" not in path.read_bytes():
            continue
        text = subprocess.run([OBJDUMP, "-d", str(path)], check=True, capture_output=True, text=True).stdout
        for kernel, code in parse(text).items():
            n, bad = hazards(code)
            assert not bad, (kernel, bad[:3])
            seen += n
    assert seen >= 1000, seen
