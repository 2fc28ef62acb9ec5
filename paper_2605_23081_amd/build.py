"""Build the HIP library in-tree: hipcc for gfx950, one shared object next to this file."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libthrift_hip.so")
CALL = os.path.join(HERE, "_call.so")          # the Python entry of the calls of a serving loop (host code only)
SOURCES = ["thrift_api.hip", "thrift_prepass.hip", "thrift_prefill.hip", "thrift_prefill_split.hip", "thrift_decode.hip", "thrift_decode_split.hip", "thrift_cache.hip", "thrift_probe.hip"]
DMA_SOURCES = ["thrift_prefill.hip", "thrift_prefill_split.hip", "thrift_decode.hip", "thrift_decode_split.hip"]      # kernels whose inline assembly sets M0 and keeps DMA in flight
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # NaN inputs are outside the contract (include/thrift.h); without this every maximum of matrix-unit results
         # is preceded by instructions that only quiet signalling NaNs
         "-fno-honor-nans",
         # packed-FP32 VALU forms are kept out of the generated code on the test machines
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


def scratch_in_loops(asm_text: str):
    """Kernel names whose generated code touches scratch memory (register spills) inside a loop.

    The fused kernel keeps LDS DMA in flight across key blocks; a spill reload inside the walk would sit in the
    same in-order memory queue and wait for those transfers at every block.  A spill that is stored before the
    walk and reloaded after it costs nothing.  The compiler's listing marks every basic block that belongs to a
    loop in the comment of its label line."""
    bad, kernel, depth = set(), None, 0
    kernels, blocks, loop_blocks = 0, 0, 0
    for line in asm_text.splitlines():
        t = line.strip()
        if t.startswith("_Z") and t.split(":")[0].isidentifier() and ":" in t:
            kernel, depth = t.split(":")[0], 0
            kernels += 1
        elif t.startswith(".LBB") or t.startswith("; %bb."):
            depths = [int(d) for d in re.findall(r"Depth=(\d+)", t)]
            depth = max(depths) if depths else 0
            blocks += 1
            loop_blocks += depth > 0
        elif t.startswith(";") and "Loop" in t and "Depth=" in t:
            # continuation lines of a label's comment: a nested loop's header names its parent first, itself below
            depth = max([depth] + [int(d) for d in re.findall(r"Depth=(\d+)", t)])
        elif t.startswith("scratch_") and kernel and depth >= (2 if "persistent" in kernel else 1):
            # in a persistent kernel the outermost loop is the loop over work items: a reload at an item's start or end
            # is outside the walk over the key blocks, like a reload before or after the walk of the other kernels
            bad.add(kernel)
    # The labels are the compiler's listing format, not a stable interface: a listing in which no kernel, no basic
    # block or no loop annotation is recognised cannot be checked and must not pass for clean.
    if kernels == 0 or blocks == 0 or loop_blocks == 0:
        raise RuntimeError("the prefill kernel's listing has no recognisable kernel labels / basic blocks / loop annotations: "
                           "the spill check cannot read this compiler's output")
    return sorted(bad)


def m0_outside_inline_asm(asm_text: str) -> int:
    """Number of compiler-generated instructions that touch M0.

    The LDS DMA instruction takes its LDS base from M0, which the inline assembly sets without the compiler knowing.
    That is sound only while the compiler itself never keeps a value in M0 across those statements: the fused
    kernel's listing must mention M0 nowhere but between the ASMSTART / ASMEND markers."""
    inside, count, statements, seen_inside = False, 0, 0, 0
    for line in asm_text.splitlines():
        t = line.strip()
        if t.startswith(";;#ASMSTART"):
            inside = True
            statements += 1
        elif t.startswith(";;#ASMEND"):
            inside = False
        elif not t.startswith(";") and "m0" in t.replace(",", " ").split():
            if inside:
                seen_inside += 1
            else:
                count += 1
    # the kernel does set M0 in its DMA statements: a listing in which that cannot be seen is in a format this check cannot read
    if statements == 0 or seen_inside == 0:
        raise RuntimeError("the prefill kernel's listing shows no inline-assembly markers around its M0 writes: "
                           "the M0 check cannot read this compiler's output")
    return count


_REGISTERS = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _registers(operand):
    return {(m[1], n) for m in _REGISTERS.finditer(operand)
            for n in range(int(m[2] or m[4]), int(m[3] or m[4]) + 1)}


class _Listing:
    """A device listing as one graph of basic blocks per kernel, in which wait states are followed along every branch."""

    def __init__(self, asm_text: str):
        self.kernels = []                                  # (kernel, label -> ([(line, op, operands, by_hand)], labels that follow))
        self.statements = 0                                # inline assembly
        blocks, block, inside = None, None, False
        for number, line in enumerate(asm_text.splitlines()):
            t = line.strip()
            if t.startswith("_Z") and t.split(":")[0].isidentifier() and ":" in t:
                block = t.split(":")[0]
                blocks = {block: ([], [])}
                self.kernels.append((block, blocks))
            elif t.startswith(";;#ASMSTART"):
                inside = True
                self.statements += 1
            elif t.startswith(";;#ASMEND"):
                inside = False
            elif blocks is None or not t or t.startswith((";", "//")):
                pass
            elif t.startswith(".LBB"):
                label = t.split(":")[0]
                if block is not None:
                    blocks[block][1].append(label)
                block = label
                blocks[block] = ([], [])
            elif line[:1] == "\t" and t[:1].isalpha():
                if block is None:                          # behind an unconditional branch without a label: never reached
                    continue
                op, _, rest = t.split(";")[0].strip().partition(" ")
                operands = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)] if rest else []
                blocks[block][0].append((number, op, operands, inside))
                if op == "s_branch" or op.startswith("s_cbranch"):
                    blocks[block][1].append(operands[0])
                if op.startswith("s_cbranch"):             # what follows is a block of its own
                    name = f"{block}+{number}"
                    blocks[block][1].append(name)
                    block = name
                    blocks[block] = ([], [])
                elif op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                    block = None

    def instructions(self):
        return (i for _, blocks in self.kernels for code, _ in blocks.values() for i in code)

    def early(self, reads, writes):
        """(kernel, instruction) wherever reads(op, operands, by_hand) names a result that is needed longer than it has been there.
        reads: pairs (result, wait states that may be left); writes(op, operands, by_hand): pairs (result, wait states, 0 for none)."""
        found = []
        for kernel, blocks in self.kernels:
            # the wait states that each result still needs at a block's start, over all ways to it
            start, todo, here = {b: {} for b in blocks}, list(blocks), set()
            while todo:
                b = todo.pop()
                wait = dict(start[b])
                instructions, follow = blocks[b]
                for line, op, operands, by_hand in instructions:
                    if wait and any(wait.get(r, 0) > left for r, left in reads(op, operands, by_hand)):
                        here.add((line, op + " " + ", ".join(operands)))
                    states = int(operands[0], 0) + 1 if op == "s_nop" else 1
                    wait = {r: n - states for r, n in wait.items() if n > states}
                    for r, n in writes(op, operands, by_hand):
                        if n:
                            wait[r] = n
                        else:
                            wait.pop(r, None)
                for f in follow:
                    if f in start:
                        more = {r: n for r, n in wait.items() if n > start[f].get(r, 0)}
                        if more:
                            start[f].update(more)
                            todo.append(f)
            found.extend((kernel, what) for _, what in sorted(here))
        return found


def matrix_results_read_early(asm_text: str):
    """(kernel, instruction) of every hand-written instruction that touches a matrix result before it is written.

    A matrix instruction of 32 x 32 (16 x 16) values writes its result 8 (4) passes later; a vector instruction has to stay
    12 (8) wait states away from it, and here as far from overwriting the addend as well.  The compiler spaces its own instructions
    like that but not the inside of an asm statement, so the listing is followed along every branch: an instruction between
    the ASMSTART / ASMEND markers must find no result or addend of its registers in flight."""
    listing = _Listing(asm_text)
    if listing.statements == 0 or not any(op.startswith("v_mfma") for _, op, _, _ in listing.instructions()):
        raise RuntimeError("the listing shows no inline assembly or no matrix instructions: the wait-state check cannot read "
                           "this compiler's output")

    def reads(op, operands, by_hand):
        if not by_hand or op[:2] == "s_" or not operands:
            return []
        return [(("d", r), 0) for x in operands for r in _registers(x)] + [(("c", r), 0) for r in _registers(operands[0])]

    def writes(op, operands, by_hand):
        if not op.startswith(("v_mfma", "v_smfmac")):
            return []
        n = 12 if "_32x32x" in op else 8
        return [(("d", r), n) for r in _registers(operands[0])] + [(("c", r), n) for r in _registers(operands[3])]

    return listing.early(reads, writes)


_SCALARS = re.compile(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)|\b(vcc)(_lo|_hi)?\b")


def _scalars(operand):
    found = set()
    for m in _SCALARS.finditer(operand):
        if m[4]:
            found |= {"vcc" + m[5]} if m[5] else {"vcc_lo", "vcc_hi"}
        else:
            found |= set(range(int(m[1] or m[3]), int(m[2] or m[3]) + 1))
    return found


def scalars_read_early(asm_text: str):
    """(kernel, instruction) of every instruction that reads a scalar register too soon behind the vector instruction that wrote it,
    where one of the two is hand-written.

    A comparison or another vector instruction that leaves its result in vcc or a scalar register has to stay two wait states
    away from a vector instruction that reads it (four where it selects a lane, and in front of v_div_fmas) and five
    from a load or store.  The compiler spaces its own instructions like that but sees nothing of the inside of an asm statement."""
    listing = _Listing(asm_text)
    if not any(op.startswith(("v_cmp", "v_readfirstlane")) for _, op, _, _ in listing.instructions()):
        raise RuntimeError("the listing shows no vector instruction that writes a scalar register: the wait-state check cannot read "
                           "this compiler's output")
    longest = 5

    def results(op):                                       # the operands that it writes, of which some are scalar registers
        if op.startswith(("v_cmp", "v_readfirstlane", "v_readlane")):
            return 1
        return 2 if "_co_" in op or op.startswith(("v_div_scale", "v_mad_u64", "v_mad_i64")) else 0

    def reads(op, operands, by_hand):
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            apart = 5
        elif not op.startswith("v_"):
            return []
        else:
            apart = 4 if op.startswith(("v_readlane", "v_writelane", "v_div_fmas")) else 2
        read = set().union(*map(_scalars, operands[results(op):]), {"vcc_lo", "vcc_hi"} if op.startswith("v_div_fmas") else set())
        return [((written_by_hand, r), longest - apart) for r in read for written_by_hand in ((False, True) if by_hand else (True,))]

    def writes(op, operands, by_hand):
        if op.startswith("s_") and not op.startswith(("s_cmp", "s_bitcmp", "s_cbranch")):      # a scalar instruction's result is waited for
            return [((written_by_hand, r), 0) for x in operands[:1] for r in _scalars(x) for written_by_hand in (False, True)]
        if not op.startswith("v_"):
            return []
        return [((by_hand, r), longest) for x in operands[:results(op)] for r in _scalars(x)]

    return listing.early(reads, writes)


def unmet_launch_bounds(compiler_output: str):
    """Kernels whose launch bounds ask for more wavefronts per SIMD than their LDS or registers let a CU hold.

    The compiler says so in a warning, drops the bound and allocates registers as if there were none."""
    return sorted(set(re.findall(r"failed to meet occupancy target given by 'amdgpu-waves-per-eu' in '(\w+)'", compiler_output)))


def _start_call_module(obj):
    """Compile csrc/thrift_call.cpp against the headers of the installed torch (host compiler)."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths

    inc = [INCLUDE, sysconfig.get_paths()["include"], *include_paths()]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           *[f"-I{inc[0]}"], *[a for d in inc[1:] for a in ("-isystem", d)], "-c", os.path.join(CSRC, "thrift_call.cpp"), "-o", obj]
    return cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _link_call_module(obj):
    import torch

    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    # the HIP library stands next to the module; torch's libraries are those of the process that imports it
    cmd = ["g++", "-shared", "-o", CALL, obj, "-L" + HERE, "-lthrift_hip", "-Wl,-rpath,$ORIGIN", "-L" + tlib,
           "-ltorch_python", "-ltorch_cpu", "-lc10"]
    subprocess.run(cmd, check=True)


def build(verbose: bool = False, extra=()):
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    call_obj = os.path.join(CSRC, "thrift_call.o")
    procs.append(_start_call_module(call_obj))
    # the device listings of the kernels that stage by LDS DMA, for the spill, M0 and wait-state checks (run beside the object builds)
    listings = []
    for src in DMA_SOURCES:
        listing = os.path.join(CSRC, src.replace(".hip", ".gfx950.s"))
        lcmd = ["hipcc", *FLAGS, *extra, "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", listing]
        listings.append((src, listing, lcmd, subprocess.Popen(lcmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "not a recognized feature for this target" not in l)
        if p.returncode != 0:
            sys.stderr.write(out + "\n")
            raise RuntimeError("compilation failed: " + " ".join(cmd))
        unmet = unmet_launch_bounds(out)
        if unmet:
            raise RuntimeError("launch bounds that cannot be met: " + ", ".join(unmet))
        if verbose and out.strip():
            print(out)
    for src, listing, lcmd, lproc in listings:
        lout, _ = lproc.communicate()
        if lproc.returncode != 0:
            sys.stderr.write(lout + "\n")
            raise RuntimeError("hipcc failed: " + " ".join(lcmd))
        with open(listing) as f:
            text = f.read()
        os.remove(listing)
        spilling = scratch_in_loops(text)
        if spilling:
            raise RuntimeError(f"{src}: spilled registers are reloaded inside a loop: " + ", ".join(spilling))
        if m0_outside_inline_asm(text):
            raise RuntimeError(f"{src}: the compiler uses M0: the LDS DMA statements would clobber it")
        early = matrix_results_read_early(text)
        if early:
            raise RuntimeError(f"{src}: hand-written instructions read matrix results too early: " + ", ".join(sorted({f"{k}: {i}" for k, i in early})[:8]))
        early = scalars_read_early(text)
        if early:
            raise RuntimeError(f"{src}: scalar registers are read too soon behind or by hand-written instructions: " + ", ".join(sorted({f"{k}: {i}" for k, i in early})[:8]))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    _link_call_module(call_obj)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=tuple(sys.argv[1:])))
