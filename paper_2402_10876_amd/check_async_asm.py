"""Build-time check of the kernels' split asynchronous loads.

The kernels issue LDS reads (ds_read_*) and scalar loads (s_load_*) from inline
assembly and wait for them in a LATER inline-assembly statement
(`s_waitcnt lgkmcnt(0)`), so that matrix instructions and copies can be issued in
between.  The compiler does not know that the destination registers of such a
load are not valid until the wait; it is free to copy or reuse them right after
the load statement (register coalescing of a loop-carried value does exactly
that).  This script compiles each kernel source to assembly and walks every
kernel in layout order (fall-through paths; the pending set is dropped at a label
that follows an unconditional jump): a register written by a load inside an
inline-assembly block is "pending" until the next `s_waitcnt` with `lgkmcnt(0)`, or
for a `global_load` until the next `s_waitcnt vmcnt(..)` in an inline-assembly block
(the kernels place these loads so that this wait covers them; the compiler's own
waits count other loads);
any instruction that names a pending register before that wait is reported.
The vector loads are also followed along every branch, up to the first wait for them on each
path: there the compiler's own instructions are reported (whether a path can reach one of
the kernels' own uses without a wait depends on the conditions of its branches).

A vector memory instruction needs five wait states behind a vector instruction that wrote a scalar register of its
address (v_readlane of a spilled one, say).  The compiler sees to that for its own instructions and does not look into
inline assembly: such an instruction there is reported unless the block itself waits.

    python -m paper_2402_10876_amd.check_async_asm          # exit status 1 on a finding
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
KERNEL_SOURCES = ["gemm_kernels.hip", "gemm_dma.hip", "gemm_mk.hip", "gemm_small.hip", "gemm_small_i8.hip", "gemm_tvw.hip", "gemm_i8.hip", "gemm_tvw_i8.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "--cuda-device-only", "-S", "-Wno-unused-command-line-argument"]

_REG = re.compile(r"\b([vsa])(?:(\d+)|\[(\d+):(\d+)\])")
_ASYNC = re.compile(r"^(ds_read\w*|ds_load\w*|s_load_\w+|s_buffer_load_\w+)$")
_ASYNC_VM = re.compile(r"^global_load_dword\w*$")


def _regs(text):
    out = set()
    for m in _REG.finditer(text):
        if m.group(2) is not None:
            out.add((m.group(1), int(m.group(2))))
        else:
            out.update((m.group(1), i) for i in range(int(m.group(3)), int(m.group(4)) + 1))
    return out


def check_assembly(asm_text: str):
    """Returns a list of (kernel, line number, instruction, registers) findings."""
    findings = []
    kernel, in_app, pending, pending_vm, prev_op = None, False, {}, {}, ""
    for ln, raw in enumerate(asm_text.split("\n"), 1):
        line = raw.strip()
        if line.startswith(";;#ASMSTART"):
            in_app = True
            continue
        if line.startswith(";;#ASMEND"):
            in_app = False
            continue
        code = line.split(";")[0].strip()
        if not code:
            continue
        if code.endswith(":"):
            if raw[0].isspace():
                continue
            if code.startswith("."):               # a local label: reached by fall-through unless the
                if prev_op in ("s_branch", "s_endpgm", "s_setpc_b64"):   # block before it ends in a jump
                    pending, pending_vm = {}, {}
            else:
                kernel, pending, pending_vm = code[:-1], {}, {}    # a new function
            continue
        if code.startswith("."):
            continue
        parts = code.split(None, 1)
        op, args = parts[0], (parts[1] if len(parts) > 1 else "")
        prev_op = op
        if op == "s_waitcnt":
            if "lgkmcnt(0)" in args:
                pending = {}
            if in_app and "vmcnt" in args:
                pending_vm = {}
            continue
        if op == "s_endpgm":
            pending, pending_vm = {}, {}
            continue
        if in_app and (_ASYNC.match(op) or _ASYNC_VM.match(op)):
            dst_txt, _, src_txt = args.partition(",")
            bad = _regs(src_txt) & (set(pending) | set(pending_vm))
            if bad:
                findings.append((kernel, ln, code, sorted(bad)))
            for r in _regs(dst_txt):
                (pending if _ASYNC.match(op) else pending_vm)[r] = ln
            continue
        bad = _regs(args) & (set(pending) | set(pending_vm))
        if bad:
            findings.append((kernel, ln, code, sorted(bad)))
    return findings


def check_branches(asm_text: str):
    """Findings as check_assembly's, for inline-assembly global loads along the branches of a kernel."""
    code, labels, kernel, in_app = [], {}, None, False
    for ln, raw in enumerate(asm_text.split("\n"), 1):
        line = raw.strip()
        if line.startswith(";;#ASM"):
            in_app = line.startswith(";;#ASMSTART")
            continue
        text = line.split(";")[0].strip()
        if text.endswith(":"):
            labels[text[:-1]] = len(code)
            if not text.startswith("."):
                kernel = text[:-1]
        elif text and not text.startswith("."):
            op, _, args = text.partition(" ")
            code.append((kernel, ln, op, args.strip(), in_app, text))
    findings = []
    for i, (kernel, _, op, args, app, _) in enumerate(code):
        if not (app and _ASYNC_VM.match(op)):
            continue
        regs, seen, todo = _regs(args.partition(",")[0]), set(), [i + 1]
        while todo:
            j = todo.pop()
            while j < len(code) and j not in seen:
                seen.add(j)
                _, ln, op, args, app, text = code[j]
                if op == "s_endpgm" or (app and op == "s_waitcnt" and "vmcnt" in args):
                    break
                if op == "s_branch":
                    j = labels[args]
                    continue
                if op.startswith("s_cbranch"):
                    todo.append(labels[args])
                elif not app and _regs(args) & regs:
                    findings.append((kernel, ln, text, sorted(_regs(args) & regs)))
                    break
                j += 1
    return findings


_VMEM = re.compile(r"^(global|flat|buffer|scratch)_\w+$")
_TWO_DST = re.compile(r"^v_(add|sub|subrev|addc|subb|subbrev)_co_|^v_mad_[ui]64_|^v_div_scale_")
_WAIT_STATES = 5


def check_scalar_addresses(asm_text: str):
    """Findings as check_assembly's: inline-assembly vector memory instructions too close behind a vector instruction
    that wrote a scalar register of theirs (in layout order)."""
    findings, kernel, in_app, age = [], None, False, {}     # age: wait states since the register was written
    for ln, raw in enumerate(asm_text.split("\n"), 1):
        line = raw.strip()
        if line.startswith(";;#ASM"):
            in_app = line.startswith(";;#ASMSTART")
            continue
        code = line.split(";")[0].strip()
        if code.endswith(":"):
            if not code.startswith(".") and not raw[0].isspace():
                kernel, age = code[:-1], {}
            continue
        if not code or code.startswith("."):
            continue
        op, _, args = code.partition(" ")
        operands = re.split(r",\s*", args)
        if in_app and _VMEM.match(op):
            bad = {r for r in _regs(args) if r[0] == "s" and age.get(r, _WAIT_STATES) < _WAIT_STATES}
            if bad:
                findings.append((kernel, ln, code, sorted(bad)))
        states = int(args, 0) + 1 if op == "s_nop" else 1
        age = {r: a + states for r, a in age.items() if a + states < _WAIT_STATES}
        if op.startswith("v_"):
            for r in _regs(",".join(operands[:2 if _TWO_DST.match(op) else 1])):
                if r[0] == "s":
                    age[r] = 0
    return findings


def compile_to_asm(src: str) -> str:
    with tempfile.TemporaryDirectory() as td:
        out = os.path.join(td, "k.s")
        cmd = [HIPCC, *FLAGS, "-I" + os.path.join(ROOT, "include"), os.path.join(PKG, "csrc", src), "-o", out]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc -S failed:\n" + " ".join(cmd) + "\n" + r.stderr[-3000:])
        return open(out).read()


def check_sources(sources=KERNEL_SOURCES):
    with ThreadPoolExecutor(max_workers=len(sources)) as ex:
        texts = list(ex.map(compile_to_asm, sources))
    res = []
    for src, text in zip(sources, texts):
        res += [(src,) + f for f in check_assembly(text) + check_branches(text) + check_scalar_addresses(text)]
    return res


def main():
    res = check_sources()
    for src, kernel, ln, code, regs in res:
        print(f"{src}: {kernel}: line {ln}: `{code}` touches {regs} before the wait for its load")
    print(f"{len(res)} finding(s)")
    return 1 if res else 0


if __name__ == "__main__":
    sys.exit(main())
