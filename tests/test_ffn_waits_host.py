"""Wait states around the FFN kernels' direct-to-LDS loads, in the built code.

These loads are inline asm, which the compiler's hazard pass does not look
into: a vector memory instruction may read a scalar register only five wait
states after a vector instruction (v_readfirstlane, v_readlane of a spilled
register) wrote it, and M0 one after its write.  The kernel is compiled to
assembly as the library is and every path into each load is followed
backwards."""

import os
import re
import subprocess

import pytest

from paper_2505_08944_amd import build

WAITS = 5


def _sregs(op):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", op)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", op)
    return {int(m[1])} if m else {op} if op in ("m0", "vcc_lo", "vcc_hi") else {"vcc_lo", "vcc_hi"} if op == "vcc" else set()


def _kernels(asm):
    """name -> {block: [(opcode, operands)]}, blocks in order."""
    out, blocks = {}, None
    for line in asm.splitlines():
        m = re.match(r"(\w+):", line)
        if m and m[1].startswith("_Z"):
            blocks = out.setdefault(m[1], {})
            cur = blocks.setdefault("entry", [])
            continue
        m = re.match(r"(\.LBB\w+):", line)
        if m and blocks is not None:
            cur = blocks.setdefault(m[1], [])
            continue
        t = line.split(";")[0].strip()
        if blocks is None or not t or t.startswith(".") or t.endswith(":"):
            continue
        op, _, rest = t.partition(" ")
        cur.append((op, [a for a in re.split(r",\s*|\s+", rest.strip()) if a]))
    return out


def _too_close(blocks):
    """Loads that a vector write of one of their scalar registers reaches in
    fewer than WAITS wait states, or a write of M0 in fewer than 1."""
    names = list(blocks)
    pred = {n: [] for n in names}
    for i, n in enumerate(names):
        falls = True
        for k, (op, args) in enumerate(blocks[n]):
            if op.startswith(("s_branch", "s_cbranch")) and args[0] in pred:
                pred[args[0]].append((n, k + 1))
            falls = falls and not op.startswith(("s_branch", "s_endpgm"))
        if falls and i + 1 < len(names):
            pred[names[i + 1]].append((n, len(blocks[n])))

    def reaches(n, at, waits, reg, seen):
        for k in range(at - 1, -1, -1):
            if waits >= WAITS:
                return False
            op, args = blocks[n][k]
            if args and reg in _sregs(args[0]) and not op.startswith(("s_cmp", "s_bitcmp")):
                if op.startswith("v_") or (reg == "m0" and waits < 1):
                    return True
                return False
            waits += int(args[0], 0) + 1 if op == "s_nop" else 1
        for p, k in pred[n]:
            if waits < WAITS and (p, waits) not in seen:
                seen.add((p, waits))
                if reaches(p, k, waits, reg, seen):
                    return True
        return False

    loads, bad = 0, []
    for n in names:
        for k, (op, args) in enumerate(blocks[n]):
            if op.startswith("buffer_load") and args[-1] == "lds":
                loads += 1
                regs = set().union(*[_sregs(a) for a in args]) | {"m0"}
                bad += [(n, k, op, args, r) for r in regs if reaches(n, k, 0, r, set())]
    return loads, bad


def test_scan_finds_planted_hazards():
    load = "\tbuffer_load_dwordx4 v1, s[8:11], s3 offen lds\n"
    near = "_Zk:\n\tv_readlane_b32 s3, v9, 1\n\ts_mov_b32 m0, s7\n\ts_nop 0\n"
    far = "_Zk:\n\tv_readlane_b32 s3, v9, 1\n\ts_mov_b32 m0, s7\n\ts_nop 3\n"
    loop = "_Zk:\n\ts_mov_b32 m0, s7\n\ts_nop 7\n.LBB0_1:\n" + load + "\tv_readfirstlane_b32 s9, v4\n\ts_cbranch_scc1 .LBB0_1\n"
    m0 = "_Zk:\n\ts_mov_b32 m0, s7\n"
    for text, n in ((near + load, 1), (far + load, 0), (loop, 1), (m0 + load, 1)):
        loads, bad = _too_close(_kernels(text)["_Zk"])
        assert loads == 1 and len(bad) == n, text


def test_loads_wait_for_their_scalar_registers(tmp_path):
    try:
        cc = build.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    out = str(tmp_path / "k_ffn.s")
    flags = [f for f in build.CFLAGS if f not in ("-fPIC",)]
    subprocess.run([cc, *flags, "-w", "-S", "--cuda-device-only", os.path.join(build.CSRC, "k_ffn.hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    kernels = {n: b for n, b in _kernels(open(out).read()).items() if "ffn_mfma_kernel" in n}
    assert len(kernels) == 4
    for name, blocks in kernels.items():
        loads, bad = _too_close(blocks)
        assert loads > 50, name
        assert not bad, (name, bad[:4])
