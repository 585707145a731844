"""Build libechokv.so (HIP, gfx950) in-tree.  (The oracle is NumPy: there is no C to compile for it.)"""
from __future__ import annotations

import concurrent.futures
import os
import re
import shutil
import subprocess
import sys
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libechokv.so")
# the Python binding's shorter way into the library, for the running Python alone
HOSTCALL_PATH = os.path.join(HERE, "_hostcall" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-Rpass-analysis=kernel-resource-usage",
]

# Kernels that count their own outstanding global loads (manual s_waitcnt vmcnt(N) around
# global -> LDS copies).  Register spills and stack objects go through the same counter, so any
# scratch memory in one of them would make those waits meaningless: the build refuses it.
NO_SPILL_KERNELS = ("fused_decode_kernel", "fused_kscores_kernel", "recon_mfma_kernel", "prefill_attn_dma_kernel",
                    "absorbed13scores_kernel")


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; libechokv needs the ROCm toolchain")


def build_library(verbose: bool = False, extra_flags=()) -> str:
    """Compile every HIP source into libechokv.so.  Always recompiles."""
    srcs = [f for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f + ".o") for f in srcs]
        base = [hipcc_path(), *HIPCC_FLAGS, *extra_flags, "-I", os.path.join(HERE, "..", "include")]
        cmds = [[*base, "-c", "-save-temps=obj", "-o", o, os.path.join(CSRC, f)] for f, o in zip(srcs, objs)]

        def run(cmd):
            if verbose:
                print(" ".join(cmd), flush=True)
            res = subprocess.run(cmd, capture_output=True, text=True)
            if res.returncode != 0:
                sys.stderr.write(res.stdout + res.stderr)
                raise RuntimeError("hipcc failed building libechokv.so")
            return res.stdout + res.stderr

        with concurrent.futures.ThreadPoolExecutor(4) as ex:      # one compiler per source file
            remarks = "".join(ex.map(run, cmds))
        run([hipcc_path(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH + ".tmp", *objs])
        listings = [f for f in os.listdir(tmp) if f.endswith("gfx950.s")]
        if len(listings) != len(srcs):
            raise RuntimeError(f"expected one gfx950 listing per source, found {listings}")
        early = [e for f in listings for e in check_early_uses(open(os.path.join(tmp, f)).read())]
    if early:
        raise RuntimeError("registers of a requested LDS read used before its wait: "
                           + "; ".join(f"{k} line {n}: {text}" for k, n, text in early[:5]))
    spilled = check_spills(remarks)
    if spilled:
        raise RuntimeError("scratch memory (spills or stack objects) in kernels that count their own loads: "
                           + ", ".join(f"{k} ({n})" for k, n in spilled))
    build_hostcall(verbose)
    os.replace(LIB_PATH + ".tmp", LIB_PATH)
    return LIB_PATH


def build_hostcall(verbose: bool = False):
    """Compile the call helper of the binding.  It needs a C compiler and Python.h, which the library itself does not: without them this
    says so and returns None, and the binding calls by ctypes."""
    cmd = [shutil.which("gcc") or "cc", "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"],
           "-o", HOSTCALL_PATH + ".tmp", os.path.join(CSRC, "hostcall.c")]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.run(cmd, capture_output=True, text=True, check=True)
    except (OSError, subprocess.CalledProcessError) as e:
        print(f"_hostcall not built, calls of a decode loop go by ctypes: {e}\n{getattr(e, 'stderr', '')}", file=sys.stderr, flush=True)
        return None
    os.replace(HOSTCALL_PATH + ".tmp", HOSTCALL_PATH)
    return HOSTCALL_PATH


def check_spills(remarks: str):
    """(kernel, amount) for every NO_SPILL_KERNELS instance that spills registers or keeps objects
    in scratch memory, from the compiler's resource-usage remarks."""
    bad, cur = [], None
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = m.group(1)
            continue
        m = re.search(r"(?:VGPRs Spill|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and cur and int(m.group(1)) > 0 and any(k in cur for k in NO_SPILL_KERNELS):
            bad.append((cur, int(m.group(1))))
    return bad


_REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _registers(operands: str):
    out = set()
    for kind, one, lo, hi in _REG.findall(operands):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def _step(text: str, in_asm: bool, state):
    """One instruction: (early, state after it).  state: ({register of a requested LDS read: LDS and scalar memory
    operations issued since}, whether any that return out of order may be among them).  Those of LDS return in the order issued."""
    pending, scalar = state
    op, _, operands = text.partition(" ")
    if op == "s_waitcnt":
        m = re.search(r"lgkmcnt\((\d+)\)", operands)
        if operands.strip() == "0" or (m and int(m.group(1)) == 0):
            return False, ({}, False)
        if m and not scalar:
            pending = {r: n for r, n in pending.items() if n < int(m.group(1))}
        return False, (pending, scalar)
    early = bool(pending) and not pending.keys().isdisjoint(_registers(operands))
    if op.startswith(("ds_", "s_load", "s_buffer_load", "flat_")):
        pending = {r: n + 1 for r, n in pending.items()}
        scalar = scalar or not op.startswith("ds_")
        if in_asm and op.startswith("ds_read"):
            pending.update((r, 0) for r in _registers(operands.split(",")[0]))
    return early, (pending, scalar)


def check_early_uses(listing: str):
    """(kernel, line, instruction) wherever a register that an LDS read of an asm statement fills is read or written on some
    path before the wait for it.  The reads are requested in one asm statement and waited for in another (fused_gemm.h,
    prefill_kernels.h), and for the compiler the registers hold their values from the first one on: a copy of
    one between the two, or another use of one that it takes for dead, would be wrong and nothing else would show it."""
    bad, name, blocks, order = [], None, {}, []
    cur, in_asm = None, False

    def flush():
        if any(a and t.startswith("ds_read") for b in blocks.values() for t, a, _ in b["code"]):
            bad.extend((name, n, t) for n, t in _early_in(blocks, order))

    for no, line in enumerate(listing.splitlines(), 1):
        text = line.split("//")[0].strip()
        if text.startswith(";;#ASM"):
            in_asm = text == ";;#ASMSTART"
            continue
        text = re.sub(r"\s+", " ", text.split(";")[0].strip())
        label = re.match(r"(\.LBB\w+|_Z\w+):$", text)
        if label and label.group(1).startswith("_Z"):
            name, blocks, order, cur = label.group(1), {}, [], None
        if label and name:
            cur = label.group(1)
            blocks[cur] = {"code": [], "next": [], "ends": False}
            order.append(cur)
        elif text.startswith(".Lfunc_end") and name:
            flush()
            name, cur = None, None
        elif cur and text and not text.startswith("."):
            b = blocks[cur]
            b["code"].append((text, in_asm, no))
            branch = re.match(r"s_c?branch\w* (\.LBB\w+)", text)
            if branch:                            # what follows a branch is a block of its own
                b["next"].append(branch.group(1))
                b["ends"] = text.startswith("s_branch")
                cur = f"{cur}+"
                blocks[cur] = {"code": [], "next": [], "ends": False}
                order.append(cur)
            elif text.startswith(("s_endpgm", "s_setpc")):
                b["ends"] = True
    return bad


def _early_in(blocks, order):
    for a, b in zip(order, order[1:]):
        if not blocks[a]["ends"]:
            blocks[a]["next"].append(b)
    entry = {order[0]: ({}, False)}
    todo, found = [order[0]], {}
    while todo:
        at = todo.pop()
        state = entry[at]
        for text, in_asm, no in blocks[at]["code"]:
            early, state = _step(text, in_asm, state)
            if early:
                found[no] = text
        for n in blocks[at]["next"]:
            old = entry.get(n)
            new = state
            if old is not None:                   # what is pending on any path, with the fewest operations since
                new = (dict(old[0]), old[1] or state[1])
                for r, c in state[0].items():
                    new[0][r] = min(c, new[0].get(r, c))
            if new != old:
                entry[n] = new
                todo.append(n)
    return sorted(found.items())


if __name__ == "__main__":
    print(build_library(verbose=True))
