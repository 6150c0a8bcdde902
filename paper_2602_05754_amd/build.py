"""Build libtf.so (the C-ABI library) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtf.so")
SOURCES = ["tf_api.hip", "gemm_generic.hip", "gemm_split_f32.hip", "gemm_narrow_bf16.hip", "gemm_short_bf16.hip", "gemm_mfma_bf16.hip", "elementwise.hip", "selection.hip", "schedule_lp.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU forms
    "-Wall", "-Wno-unused-command-line-argument",
    "-Wno-inline-asm",          # the direct-to-LDS loads name M0 in their clobber list on purpose
    "-Rpass-analysis=kernel-resource-usage",      # per-kernel register / scratch report, checked below
]


# Scalar instructions that read the carry / condition bit SCC, and those that leave it alone.
_SCC_READERS = re.compile(r"^(s_addc_u32|s_subb_u32|s_cselect_b32|s_cselect_b64|s_cmov_b32|s_cmov_b64|"
                          r"s_cbranch_scc0|s_cbranch_scc1)\b")
_SCC_KEEPERS = re.compile(r"^(s_mov|s_movk|s_cmov|s_cselect|s_mul_i32|s_mul_hi|s_load|s_buffer_load|s_waitcnt|s_nop|"
                          r"s_barrier|s_branch|s_cbranch|s_sleep|s_setprio|s_getpc|s_setpc|s_swappc|s_sext|s_pack|"
                          r"s_bitset|s_ff1|s_ff0|s_flbit|s_brev|s_endpgm|s_sendmsg|s_getreg|s_setreg|s_memtime|"
                          r"s_memrealtime|s_dcache|s_icache|s_lshl1_add|s_lshl2_add|s_lshl3_add|s_lshl4_add)")


def scc_hazards(asm_text: str) -> list:
    """Inline assembly placed between a writer and a reader of SCC.

    The direct-to-LDS loads of the GEMM kernel are inline assembly that sets SCC.  The
    compiler is told so (clobber list), which keeps it from putting such a statement between,
    say, the s_add_u32 and the s_addc_u32 of a 64-bit address addition; a lost carry there is
    a wild global address.  This scan of the generated code is the belt to those braces: it
    walks every function linearly and reports each reader of SCC whose nearest preceding
    scalar instruction that writes SCC lies before an inline-assembly block that sets SCC itself.
    Returns a list of (function, line number, instruction)."""
    bad = []
    func = None
    in_asm = False
    asm_since_write = False
    for ln, raw in enumerate(asm_text.splitlines(), 1):
        line = raw.strip()
        if not line or line.startswith(";") and "ASM" not in line:
            continue
        if re.match(r"^[A-Za-z_.$][\w.$]*:", line) and not line.startswith(".L"):
            func = line.split(":")[0]
            asm_since_write = False
            continue
        if "#ASMSTART" in line:
            in_asm = True
            continue
        if "#ASMEND" in line:
            in_asm = False
            continue
        if in_asm:
            # only assembly that itself sets SCC can lose a carry (a vector addition without carry,
            # a plain move or a load leaves it alone)
            if line.startswith("s_") and not _SCC_KEEPERS.match(line.split()[0]):
                asm_since_write = True
            continue
        if not line.startswith("s_"):
            continue
        op = line.split()[0]
        if _SCC_READERS.match(op) and asm_since_write:
            bad.append((func, ln, line))
        if not _SCC_KEEPERS.match(op):      # every other scalar ALU / compare instruction writes SCC
            asm_since_write = False
    return bad


# Wait states between a matrix instruction and the first other instruction that reads its result, by the
# passes it takes (f64 16x16x4: 16, and LDS reads need 18; fp32 16x16x4: 8; bf16 16x16x32: 4).
_MFMA_WAIT = (("f64", 18), ("16x16x4_f32", 10), ("", 8))
_REGISTERS = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")
_VECTOR_OPS = ("v_", "ds_", "global_", "buffer_", "flat_", "scratch_")


def _registers(operands) -> set:
    out = set()
    for kind, one, lo, hi in (m for o in operands for m in _REGISTERS.findall(o)):
        out.update(kind + str(i) for i in range(int(one or lo), int(one or hi) + 1))
    return out


def mfma_hazards(asm_text: str) -> list:
    """Readers of a matrix instruction's result that come too early, waits and barriers not counted.

    The compiler keeps readers away by wait states, and lets s_waitcnt and s_barrier in between count
    as one each.  The hardware does not: a sum read that way was the one before.  Follows every path through
    every function with the distance of each register from the matrix instruction that wrote it.
    Returns a list of (function, line number, instruction)."""
    functions, name, block = {}, None, None
    for ln, raw in enumerate(asm_text.splitlines(), 1):
        line = raw.split(";")[0].strip()
        m = re.match(r"^([\w.$]+):$", line)
        if m:
            if not line.startswith("."):
                name = m.group(1)
            if name:
                block = (m.group(1), [])
                functions.setdefault(name, []).append(block)
        elif name and re.match(r"^[a-z]", line):
            block[1].append((ln, line))
    bad = {}
    for name, blocks in functions.items():
        index = {label: i for i, (label, _) in enumerate(blocks)}
        entry = [None] * len(blocks)               # register -> (states since its instruction, states needed)
        entry[0], work = {}, [0]

        def flow(to, state):
            if to is None or to >= len(blocks):
                return
            if entry[to] is None:
                entry[to] = dict(state)
            else:
                nearer = {r: v for r, v in state.items() if r not in entry[to] or v[1] - v[0] > entry[to][r][1] - entry[to][r][0]}
                if not nearer:
                    return
                entry[to].update(nearer)
            work.append(to)

        while work:
            i = work.pop()
            state, falls = dict(entry[i]), True
            for ln, line in blocks[i][1]:
                op, _, rest = line.partition(" ")
                operands, states, written = rest.split(","), 1, {}
                if op.startswith(("s_cbranch", "s_branch")):
                    flow(index.get(rest.strip()), state)
                if op in ("s_branch", "s_endpgm"):
                    falls = False
                    break
                if op == "s_nop":
                    states = int(rest, 0) + 1
                elif op in ("s_waitcnt", "s_barrier"):
                    states = 0
                elif op.startswith("v_mfma"):
                    need = next(n for key, n in _MFMA_WAIT if key in op)
                    written = {r: (0, need) for r in _registers(operands[:1])}
                elif op.startswith(_VECTOR_OPS):
                    stores = "store" in op or "write" in op
                    for r in _registers(operands if stores else operands[1:]):
                        if r in state and state[r][0] < state[r][1]:
                            bad[(name, ln)] = line
                    for r in _registers([] if stores else operands[:1]):
                        state.pop(r, None)
                state = {r: (n + states, need) for r, (n, need) in state.items() if n + states < need}
                state.update(written)
            if falls:
                flow(i + 1, state)
    return [(name, ln, line) for (name, ln), line in sorted(bad.items())]


def check_generated_code(hipcc: str, extra: list) -> None:
    flags = [f for f in HIPCC_FLAGS if f not in ("-fPIC", "-shared", "-Rpass-analysis=kernel-resource-usage")]
    sources = ("gemm_mfma_bf16.hip", "gemm_generic.hip", "gemm_split_f32.hip", "gemm_narrow_bf16.hip", "gemm_short_bf16.hip")
    assemble = lambda source: subprocess.run([hipcc] + flags + extra + ["-S", "--cuda-device-only", os.path.join(CSRC, source), "-o", "-"],
                                             capture_output=True, text=True)
    with ThreadPoolExecutor(len(sources)) as pool:
        results = list(pool.map(assemble, sources))
    for source, res in zip(sources, results):
        if res.returncode != 0:
            raise RuntimeError("hipcc -S failed:\n" + res.stderr)
        for what, bad in (("inline assembly between a writer and a reader of SCC", scc_hazards(res.stdout)),
                          ("a matrix instruction's result is read too early", mfma_hazards(res.stdout))):
            if bad:
                raise RuntimeError(f"{source}: {what}:\n" + "\n".join(f"  {f} line {ln}: {ins}" for f, ln, ins in bad[:10]))


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = os.environ.get("TF_BUILD_FLAGS", "").split()      # developer experiments
    cmd = [hipcc] + HIPCC_FLAGS + extra + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    remarks = [l for l in err.splitlines() if "-Rpass-analysis=kernel-resource-usage" in l]
    err = "\n".join(l for l in err.splitlines() if "-Rpass-analysis=kernel-resource-usage" not in l)
    if remarks:   # source-context lines that clang prints under every remark
        err = "\n".join(l for l in err.splitlines() if not re.match(r"^\s*(\d+\s*)?\|", l))
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    # The staged registers of the GEMM kernels must stay in registers: a kernel that uses
    # scratch memory has lost an order of magnitude of speed, so treat it as a build error.
    name = None
    for l in remarks:
        m = re.search(r"Function Name: (\S+)", l)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", l)
        if m and int(m.group(1)) != 0:
            raise RuntimeError(f"kernel {name} uses {m.group(1)} bytes/lane of scratch memory")
    check_generated_code(hipcc, extra)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
