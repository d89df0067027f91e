"""Builds libwlb.so (the C-ABI library) for gfx950 with hipcc, in-tree.

Run as `python -m paper_2503_17924_amd.build` or through `__graft_entry__.build()`.
hipcc cross-compiles, so no GPU is needed to build.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libwlb.so")
SOURCES = ["wlb_host.cpp", "wlb_plan.hip", "wlb_attn_fwd.hip", "wlb_attn_fwd_pair.hip", "wlb_attn_bwd.hip", "wlb_attn_dq_pair.hip", "wlb_attn_dkv.hip", "wlb_attn_span.hip", "wlb_calib.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 instructions are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


# Sources whose kernels use the accumulation registers by number, in statements marked "; acc"
OWN_ACC_REGISTERS = ["wlb_attn_dkv.hip", "wlb_attn_fwd_pair.hip", "wlb_attn_dq_pair.hip"]


def check_acc_registers(asm: str) -> None:
    """Refuses code in which the compiler itself uses an accumulation register (as a place to spill to, for
    instance): it does not know that they hold values between the statements that name them."""
    with open(asm) as fh:
        for number, line in enumerate(fh, 1):
            code, _, comment = line.partition(";")
            if re.search(r"(^|[\s,])a(\[|\d)", code) and not code.lstrip().startswith(".") and comment.strip() != "acc":
                raise RuntimeError(f"{asm}:{number}: accumulation register used by the compiler: {line.strip()}")


def _registers(operand: str, kind: str) -> set[int]:
    """Numbers of the registers of a kind ("v", "a", "s") that an operand names; vcc counts as scalar register -1, m0 as -2."""
    out = set()
    for m in re.finditer(r"\b%s(?:(\d+)\b|\[(\w+):(\w+)\])" % kind, operand):
        lo, hi = (m[1], m[1]) if m[1] else (m[2], m[3])
        out.update(range(int(lo, 0), int(hi, 0) + 1))
    if kind == "s":
        out |= {n for name, n in (("vcc", -1), ("m0", -2)) if re.search(r"\b%s\b" % name, operand)}
    return out


_TRANS = re.compile(r"v_(exp|log|rcp|rsq|sqrt|sin|cos)_")
_MFMA_RESULT = 19      # wait states until the result of an MFMA of at most 16 passes is read by anything but the next MFMA's sum


def _wait_states(producer: tuple, consumer: tuple) -> int:
    """Wait states that must lie between two instructions (opcode, operands): those that the hardware does not insert by itself."""
    (op, dst), (use, src) = producer[:2], consumer[:2]
    if op.startswith("s_") and op != "s_nop":
        return 1 if use.startswith("buffer_") and src[-1].endswith(" lds") and dst and "m0" in dst[0] else 0
    if not op.startswith("v_") or not dst:
        return 0

    def both(kind: str, written: list) -> set:
        reads = src[1:] if use.startswith("v_") else src
        return set().union(*(_registers(x, kind) for x in written)) & set().union(*(_registers(x, kind) for x in reads))

    if op.startswith("v_mfma"):
        if use.startswith("v_mfma") and src[-1] == src[0] == dst[0]:
            src = src[:-1]          # the sum that the next MFMA continues: the hardware orders it
        return _MFMA_RESULT if both("v", dst[:1]) or not use.startswith("v_mfma") and both("a", dst[:1]) else 0
    written = dst[:2] if re.search(r"_co_|_swap|div_scale|mad_[ui]64", op) else dst[:1]
    if op.startswith("v_cmp") and len(dst) == 2:
        written = ["vcc"]
    need = 0
    if both("v", written):
        need = 2 if use.startswith("v_mfma") else 1 if use.startswith("v_read") or use.startswith("v_") and _TRANS.match(op) else 0
    if both("s", written):
        need = max(need, 2 if use.startswith("v_") else 5 if use.startswith(("buffer_", "global_")) else 0)
    return need


def check_wait_states(asm: str) -> None:
    """Refuses code in which an instruction of a hand-written statement follows what it depends on, or is followed by what
    depends on it, without the wait states between: the compiler, which puts them between its own instructions, does not look into the statements."""
    code, labels, branches, written = [], {}, {}, False      # (opcode, operands, line, written by hand)
    with open(asm) as fh:
        for number, line in enumerate(fh, 1):
            written = written and ";#ASMEND" not in line or ";#ASMSTART" in line
            text = line.partition(";")[0].strip()
            if re.match(r"[\w.$]+:", text):
                labels[text.split(":")[0]] = len(code)
            elif text and not text.startswith("."):
                op, _, rest = text.partition(" " if " " in text.partition("\t")[0] else "\t")
                operands = [x.strip() for x in rest.split(",")] if rest.strip() else []
                if op.startswith(("s_branch", "s_cbranch")):
                    branches.setdefault(operands[0], []).append(len(code))
                code.append((op, operands, number, written))
    targets = {}
    for label, sources in branches.items():
        targets.setdefault(labels.get(label, -1), []).extend(sources)

    def look_back(at: int, waited: int, consumer: tuple, seen: dict) -> None:
        if waited >= _MFMA_RESULT or seen.get(at, waited + 1) <= waited:
            return
        seen[at] = waited
        before = list(targets.get(at, []))
        if at > 0 and not code[at - 1][0].startswith(("s_branch", "s_endpgm")):
            before.append(at - 1)
        for i in before:
            producer = code[i]
            if (producer[3] or consumer[3]) and _wait_states(producer, consumer) > waited:
                raise RuntimeError(f"{asm}:{consumer[2]}: {consumer[0]} needs more wait states after {producer[0]} in line {producer[2]}")
            look_back(i, waited + (int(producer[1][0], 0) + 1 if producer[0] == "s_nop" else 1), consumer, seen)

    for at, instruction in enumerate(code):
        if instruction[0].startswith(("v_", "buffer_", "ds_", "global_")):
            look_back(at, 0, instruction, {})


def check_scratch(asm: str) -> None:
    """Refuses code that keeps registers in memory: these kernels count the copies that are under way, and a load among them waits for all of those."""
    with open(asm) as fh:
        for number, line in enumerate(fh, 1):
            if line.lstrip().startswith("scratch_"):
                raise RuntimeError(f"{asm}:{number}: register kept in memory: {line.strip()}")


def build(verbose: bool = False, keep_asm: bool = False, lib_out: str | None = None) -> str:
    """Compiles every source and links the library (to `lib_out`, default in-tree libwlb.so).
    WLB_HIPCC_EXTRA adds compiler flags (space separated) to every compile line."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    extra = os.environ.get("WLB_HIPCC_EXTRA", "").split()
    lib_out = lib_out or LIB
    bdir = os.path.join(ROOT, "_build" if lib_out == LIB else "_build/" + os.path.basename(lib_out))
    os.makedirs(bdir, exist_ok=True)
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(bdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if src.endswith(".cpp"):
            # host code: no fused multiply-add contraction, so the latency estimates are the same
            # doubles on every machine
            cmd[1:1] = ["-x", "hip", "-ffp-contract=off"]
        if "attn" in src:
            # kernels only: lets max() compile to bare v_max3 (no NaN quieting); the host-side
            # argument checks live in other files and keep full NaN semantics
            cmd += ["-fno-honor-nans"]
        if src in OWN_ACC_REGISTERS:
            # results of MFMAs that the vector ALU reads stay out of the accumulation registers, which the kernels
            # of this file number themselves (check_acc_registers)
            cmd += ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
            # the assembly that is checked is the one that is linked (the source's own switch for this warning is lost on the way)
            cmd += ["-save-temps=obj", "-Wno-inline-asm"]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, cwd=bdir)))
        if keep_asm and src.endswith(".hip") and src not in OWN_ACC_REGISTERS:
            asm = [c for c in cmd if c != "-c"]
            asm[asm.index("-o") + 1] = os.path.join(bdir, os.path.splitext(src)[0] + ".s")
            asm += ["-S", "--cuda-device-only"]
            procs.append((src + " (asm)", subprocess.Popen(asm, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, cwd=bdir)))
        objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    for src in OWN_ACC_REGISTERS:
        asm = os.path.join(bdir, os.path.splitext(src)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")
        check_acc_registers(asm)
        check_wait_states(asm)
        check_scratch(asm)
    tmp = lib_out + ".tmp"
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    os.replace(tmp, lib_out)
    return lib_out


if __name__ == "__main__":
    _out = [a.split("=", 1)[1] for a in sys.argv if a.startswith("--out=")]
    print(build(verbose=True, keep_asm="--asm" in sys.argv, lib_out=os.path.abspath(_out[0]) if _out else None))
