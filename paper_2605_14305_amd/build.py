"""Build libfef.so (the C-ABI verify-step library) in-tree with hipcc for gfx950.

    python -m paper_2605_14305_amd.build
"""
import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfef.so")
SOURCES = ["fef_api.hip", "head_gemm.hip", "head_gemm_tiled256.hip", "head_slices.hip", "head_runs.hip", "head_loss.hip", "verify_kernels.hip", "ce_kernels.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def build(verbose=True, extra_flags=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=8) as pool:
        def compile_one(src):
            obj = os.path.join(tmp, src + ".o")
            cmd = [hipcc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj
        check = pool.submit(check_accumulators_isa, verbose, extra_flags)
        objs = list(pool.map(compile_one, sorted(SOURCES, key=lambda s: -os.path.getsize(os.path.join(CSRC, s)))))
        fresh = LIB + ".new"  # takes the library's place only when the check has passed
        cmd = [hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", fresh]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        try:
            check.result()
        except BaseException:
            os.remove(fresh)
            raise
        os.replace(fresh, LIB)
    return LIB


def _assembly(src, extra_flags=()):
    """Lines of the device assembly of one source."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out.s")
        flags = [f for f in FLAGS if f != "-fPIC"]
        subprocess.run([hipcc, *flags, *extra_flags, "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out], check=True,
                       stderr=subprocess.DEVNULL)
        with open(out) as f:
            return f.read().split("\n")


def _regs(text):
    """Vector and accumulation registers named in an operand list."""
    out = set()
    for m in re.finditer(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        if m.group(1):
            out.update(m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1))
        else:
            out.add(m.group(4) + m.group(5))
    return out


def check_accumulators_isa(verbose=True, extra_flags=()):
    """The multiplies of head_gemm_tiled256.hip are inline assembly on accumulators in place, so the compiler does not
    know that a multiply's result, or a register that a multiply is about to read, needs wait states around other
    vector instructions.  That is sound as long as between the first and the last multiply of a kernel nothing but
    multiplies touches an accumulator, a multiply finds its own accumulator at least four multiplies old (it would need
    no wait states behind the very multiply that wrote it: the same instruction on the same registers is forwarded, and
    the compiler issues such chains back to back; four is what the smallest tile gives), and no vector instruction
    writes a register within two wait states of a multiply that reads it (most come from LDS reads, which are waited
    for).  This checks exactly that for each instantiation."""
    check_accumulators(_assembly("head_gemm_tiled256.hip", extra_flags), verbose)


def check_accumulators(lines, verbose=True):
    starts = [i for i, l in enumerate(lines) if re.match(r"^_Z\w*head_tiled256_kernel\w*:", l)]
    if not starts:
        raise RuntimeError("check_accumulators_isa: no kernel in the assembly")
    for start in starts:
        end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
        name = lines[start].split(":")[0]
        mfma = [i for i in range(start, end) if lines[i].strip().startswith("v_mfma")]
        ops = [lines[i].strip().split(None, 1)[1].split(",") for i in mfma]
        if not ops:
            raise RuntimeError(f"check_accumulators_isa: {name}: no multiply")
        acc = set().union(*[_regs(o[0]) for o in ops])
        for n, (o, i) in enumerate(zip(ops, mfma)):
            if o[0].strip() != o[3].strip():
                raise RuntimeError(f"check_accumulators_isa: {name}: '{lines[i].strip()}' is not in place")
            if any(_regs(o[0]) & _regs(p[0]) for p in ops[max(0, n - 3):n]):
                raise RuntimeError(f"check_accumulators_isa: {name}: '{lines[i].strip()}' is less than four behind the last on its registers")
        recent = []  # vector instructions just before a multiply
        for i in range(mfma[0], mfma[-1] + 1):
            t = lines[i].strip()
            if t.startswith("v_mfma"):
                if any(_regs(t) & w for w in recent[-2:]):
                    raise RuntimeError(f"check_accumulators_isa: {name}: '{t}' reads what a vector instruction just wrote")
                recent.append(set())
            elif t.startswith("v_") and not t.startswith("v_cmp"):
                args = t.split(None, 1)[1] if len(t.split(None, 1)) > 1 else ""
                if _regs(args) & acc:
                    raise RuntimeError(f"check_accumulators_isa: {name}: '{t}' touches an accumulator between multiplies")
                recent.append(_regs(args.split(",")[0]))
            elif t and not t.startswith((";", ".")):
                recent += [set()] * (int(t.split()[1]) + 1 if t.startswith("s_nop") else 1)
        if verbose:
            print(f"check_accumulators_isa: {name}: {len(mfma)} multiplies in place on {len(acc)} registers", flush=True)


HARNESS_SRC = os.path.join(os.path.dirname(HERE), "tests", "c_abi", "abi_harness.cpp")
HARNESS = os.path.join(HERE, "abi_harness")


def build_harness(verbose=True):
    """The C++ program that calls libfef.so through include/fef.h alone (run by the GPU tests)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(os.path.dirname(HERE), "include"), HARNESS_SRC,
           "-L", HERE, "-lfef", "-Wl,-rpath,$ORIGIN", "-o", HARNESS]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return HARNESS


if __name__ == "__main__":
    build(extra_flags=sys.argv[1:])
    build_harness()
