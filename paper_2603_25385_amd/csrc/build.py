"""Build libglowq.so (the C-ABI library) for gfx950 with hipcc.

    python paper_2603_25385_amd/csrc/build.py

The library lands in paper_2603_25385_amd/lib/ (git-ignored, in-tree so that a
snapshot of the tree carries it to the GPU machine).  This file is a plain script on
purpose: it must run when the library does not exist yet, so it cannot live
behind the package import, which loads the library.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile

CSRC = os.path.dirname(os.path.abspath(__file__))
LIB_DIR = os.path.join(os.path.dirname(CSRC), "lib")
LIB = os.path.join(LIB_DIR, "libglowq.so")
SOURCES = ["api.hip", "prepare.hip", "proj.hip", "decode.hip", "prefill.hip", "probe.hip", "factorize.hip", "mx.hip"]
# packed-fp32 instructions are switched off for device code on purpose
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Rpass-analysis=kernel-resource-usage"]
# Per-file flags.  decode.hip: matrix-instruction results stay in ordinary vector registers
# (the few-token kernels issue one correction product per workgroup; with it in an
# accumulation register the 2- and 4-token kernels measured 4-7 % slower).
FILE_FLAGS = {"decode.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}
# Kernels that count their own outstanding memory operations (hand-placed s_waitcnt): a
# register spill would add loads of the compiler's to that count, so they must have none.
NO_SPILL = ("k_prefill", "k_wide", "k_mx_wide")
# ... and whose sums live in accumulation registers on purpose (no load writes those)
ACC_REGS = ("k_wide", "k_mx_wide")


def check_no_spills(src: str, remarks: str) -> None:
    name = None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].strip()
        elif "AGPRs:" in line and name and any(k in name for k in NO_SPILL) and not any(k in name for k in ACC_REGS):
            # values parked in accumulation registers are copies too, and a copy of a
            # register whose load is still in flight (hand-counted waits) reads garbage
            if int(line.split("AGPRs:")[1].split()[0]):
                raise RuntimeError(f"{src}: {name} uses accumulation registers; this kernel "
                                   "must keep everything in vector registers")
        elif "ScratchSize [bytes/lane]:" in line and name:
            n = int(line.split("ScratchSize [bytes/lane]:")[1].split()[0])
            if n and any(k in name for k in NO_SPILL):
                raise RuntimeError(f"{src}: {name} uses {n} bytes of scratch per lane (register "
                                   "spills); this kernel must not spill")


# Kernels whose products are assembly: the compiler places no wait states around them.
ASM_PRODUCTS = {"prefill.hip": "k_wide", "mx.hip": "k_mx_wide"}
# ... and whose sums are accumulation registers named by number: nothing else may live there
NAMED_SUMS = ("k_mx_wide",)
OPERAND_STATES = 2       # from a vector-ALU write of an operand (a sum) to the product
SUM_STATES = 18          # from a product to anything else that names its sum


def _registers(operand: str) -> set:
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\w+)(?::(\w+))?\])", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3], 0), int(m[4] or m[3], 0))
    return {(m[1], k) for k in range(lo, hi + 1)}


def check_products(src: str, assembly: str, kernel: str) -> int:
    """Checks the wait states around the matrix instructions that add in accumulation registers, in every function
    whose name holds `kernel` and along every path to them.  Returns how many there are."""
    ins, label_at, jumps, names, fn = [], {}, {}, [], ""      # (name, operands) in order, labels, their branches
    for line in assembly.splitlines():
        label = re.match(r"([\w$.]+):", line)
        if label:
            if not label[1].startswith(".L"):
                fn = label[1]
            label_at[label[1]] = len(ins)
            continue
        text = line.split(";")[0].split("//")[0].strip()
        if not text or not line[0].isspace() or text.startswith("."):
            continue
        name, _, rest = text.partition(" ") if " " in text else text.partition("\t")
        ops = [o.strip() for o in rest.replace("\t", " ").split(",")] if rest.strip() else []
        if name.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(ops[0], []).append(len(ins))
        ins.append((name, ops))
        names.append(fn)
    at_label = {}
    for label, k in label_at.items():
        at_label.setdefault(k, []).extend(jumps.get(label, []))

    def product(k):
        name, ops = ins[k]
        return name.startswith("v_mfma") and ops[0].startswith("a")

    def before(k, states):
        # (instruction, wait states between it and k) back to `states`, on every path
        seen, todo = {}, [(k, 0)]
        while todo:
            j, n = todo.pop()
            for p in ([j - 1] if j and names[j - 1] == names[j] and not ins[j - 1][0].startswith(("s_branch", "s_endpgm")) else []) + at_label.get(j, []):
                if n >= states or seen.get(p, states) <= n:
                    continue
                seen[p] = n
                yield p, n
                todo.append((p, n + (int(ins[p][1][0], 0) + 1 if ins[p][0] == "s_nop" else 1)))

    def fail(k, j, what):
        raise RuntimeError(f"{src}: {names[k]}: '{ins[k][0]} {', '.join(ins[k][1])}' {what} of "
                           f"'{ins[j][0]} {', '.join(ins[j][1])}'")

    count = 0
    for k, (name, ops) in enumerate(ins):
        if kernel not in names[k]:
            continue
        if product(k):
            count += 1
            if ops[0] != ops[3]:
                raise RuntimeError(f"{src}: {names[k]}: a product does not add in place")
            reads = set().union(*(_registers(o.split(" ")[0]) for o in ops[1:]))
            for j, _ in before(k, OPERAND_STATES):
                if ins[j][0].startswith("v_") and not ins[j][0].startswith("v_mfma"):
                    wrote = set().union(*map(_registers, ins[j][1][:2 if "swap" in ins[j][0] else 1]))
                    if wrote & reads:
                        fail(k, j, "follows too closely the write of its operand")
        else:
            mine = {r for o in ops for r in _registers(o.split(" ")[0]) if r[0] == "a"}
            if mine and any(n in names[k] for n in NAMED_SUMS):
                if name != "v_accvgpr_read_b32" and (name, ops[1:]) != ("v_accvgpr_write_b32", ["0"]):
                    raise RuntimeError(f"{src}: {names[k]}: '{name} {', '.join(ops)}' touches a sum")
            for j, _ in before(k, SUM_STATES) if mine else ():
                if product(j) and _registers(ins[j][1][0]) & mine:
                    fail(k, j, "uses too early the sum")
    return count


def build(verbose: bool = False, extra: list | None = None) -> str:
    os.makedirs(LIB_DIR, exist_ok=True)
    extra = list(extra or []) + os.environ.get("GLOWQ_EXTRA_HIPCC_FLAGS", "").split()
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(LIB_DIR, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, *FILE_FLAGS.get(src, []), *(extra or []), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                            text=True)))
        objs.append(obj)
    listings = []
    for src, kernel in ASM_PRODUCTS.items():
        out = tempfile.NamedTemporaryFile(suffix=".s")
        cmd = ["hipcc", *FLAGS, *FILE_FLAGS.get(src, []), *extra, "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out.name]
        listings.append((src, kernel, out, subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        check_no_spills(src, out)
        out = "\n".join(l for l in out.splitlines()
                        if "is not a recognized feature" not in l and "remark:" not in l)
        if p.returncode != 0:
            failed = True
            print(f"--- {src} failed ---\n{out}", file=sys.stderr)
        elif out.strip() and verbose:
            print(out)
    for src, kernel, out, p in listings:
        failed = p.wait() != 0 or failed
        if not failed and check_products(src, open(out.name).read(), kernel) == 0:
            raise RuntimeError(f"{src}: no products of {kernel} found")
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
