"""Build ``libcube3d.so`` (the C-ABI library) for gfx950 with hipcc, in-tree."""
import glob
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
# CUBE3D_OUT: another file name for the library (a variant build, e.g. with CUBE3D_EXTRA_FLAGS=-DCUBE3D_PROFILE,
# beside the product's libcube3d.so); its objects go to a folder of their own
LIB = os.path.join(HERE, os.environ.get("CUBE3D_OUT", "libcube3d.so"))
OBJDIR = os.path.join(HERE, "_build" if "CUBE3D_OUT" not in os.environ else "_build_" + os.environ["CUBE3D_OUT"].replace(".", "_"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC,
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option", "-Wno-inline-asm"] + \
    os.environ.get("CUBE3D_EXTRA_FLAGS", "").split()


SCRATCH_LIMIT = 1024   # bytes per lane
# The any-size kernels' K loops span several basic blocks, which the search below does not recognise as loops: no
# scratch at all (none of them needs any).
SCRATCH_LIMITS = {"gemm_edge_kernel": 0, "gemm_ring_kernel": 0}
MFMA_BLOCK = 8         # a basic block with at least this many MFMAs belongs to a K loop


def scratch_limit(kernel):
    """Bytes of scratch memory per lane that a kernel (mangled name) may use."""
    return min([limit for part, limit in SCRATCH_LIMITS.items() if part in kernel], default=SCRATCH_LIMIT)


def _spills_in_k_loops(asm_path):
    """Names of the kernels whose device assembly has a scratch access in a K loop: a basic block
    with many MFMAs that branches back to its own label."""
    bad, func, label, mfma, scratch, loops = [], None, None, 0, 0, False

    def close_block():
        if func and loops and mfma >= MFMA_BLOCK and scratch:
            bad.append(func)

    with open(asm_path) as f:
        for line in f:
            head = line.split(";")[0].strip()
            if head.endswith(":") and not head.startswith("."):
                close_block()
                func, label, mfma, scratch, loops = head[:-1], None, 0, 0, False
            elif head.startswith(".LBB") and head.endswith(":"):
                close_block()
                label, mfma, scratch, loops = head[:-1], 0, 0, False
            elif head.startswith("v_mfma") or head.startswith("v_smfmac"):
                mfma += 1
            elif head.startswith("scratch_"):
                scratch += 1
            elif head.startswith("s_cbranch") or head.startswith("s_branch"):
                if label and head.split()[-1] == label:
                    loops = True
    close_block()
    return sorted(set(bad))


SCALAR_WAIT = 5     # wait states between a vector instruction that writes a scalar register and a memory instruction that reads it
_SCALARS = re.compile(r"\bs(?:(\d+)|\[(\d+):(\d+)\])")
_NO_RESULT = ("s_cmp", "s_bitcmp", "s_cbranch", "s_branch", "s_nop", "s_wait", "s_barrier", "s_setprio", "s_endpgm")


def _scalars(operands):
    return {r for one, first, last in _SCALARS.findall(operands)
            for r in (range(int(first), int(last) + 1) if first else (int(one),))}


def early_scalar_reads(asm):
    """Loads straight into LDS (lines of device assembly) that may read a scalar register less than SCALAR_WAIT wait states
    after a vector instruction wrote it: (kernel, writer, load).  They are inline assembly, where the compiler sees no memory
    instruction and keeps no distance.  A copy by a scalar instruction is as good as the distance."""
    found, kernel, code = [], None, []

    def close():
        loads = [i for i, x in enumerate(code) if "load" in x and (x.endswith(" lds") or "load_lds" in x)]
        if not loads:
            return
        into = {}           # label -> branches to it
        for i, x in enumerate(code):
            if x.startswith(("s_cbranch", "s_branch")):
                into.setdefault(x.split()[-1], []).append(i)

        def before(i):
            out = list(into.get(code[i][:-1], ())) if code[i].endswith(":") else []
            if i > 0 and not code[i - 1].startswith(("s_branch", "s_endpgm")):
                out.append(i - 1)
            return out

        for load in loads:
            todo, seen = [(p, 0, frozenset(_scalars(code[load]))) for p in before(load)], set()
            while todo:
                state = i, waited, regs = todo.pop()
                if waited >= SCALAR_WAIT or not regs or state in seen:
                    continue
                seen.add(state)
                x = code[i]
                if not x.endswith(":"):
                    op, _, operands = x.partition(" ")
                    result = operands.split(",")[0]
                    if op.startswith("v_"):
                        # (the second operand is a result too where there is a carry)
                        if "_co_" in op or op.startswith(("v_mad_u64", "v_mad_i64", "v_div_scale")):
                            result = ",".join(operands.split(",")[:2])
                        if _scalars(result) & regs:
                            found.append((kernel, x, code[load]))
                    elif op.startswith("s_") and not op.startswith(_NO_RESULT):
                        regs = regs - _scalars(result)
                    waited += int(operands, 0) + 1 if op == "s_nop" else 1
                todo += [(p, waited, regs) for p in before(i)]

    for line in asm:
        head = line.split(";")[0].strip()
        if not head or head.startswith(".") and not head.startswith(".LBB"):
            continue
        if head.endswith(":") and not head.startswith("."):
            close()
            kernel, code = head[:-1], []
        else:
            code.append(" ".join(head.split()))
    close()
    return found


def _compile(src):
    """Compile one source; refuse kernels that spill registers inside a K loop (the tuned kernels
    are sized to live in the register file: a spill there is a performance bug) or that spill
    wholesale, and loads into LDS that may read a scalar register too early.  What the persistent
    kernel parks between two work items (lane-constant addresses, a few dozen registers, reloaded
    once per item) is accepted."""
    base = os.path.basename(src)
    obj = os.path.join(OBJDIR, base + ".o")
    res = subprocess.run([HIPCC, *FLAGS, "-Rpass-analysis=kernel-resource-usage", "-save-temps=obj", "-c", src, "-o", obj],
                         stderr=subprocess.PIPE, text=True)
    name, spilled, keep = None, [], []
    for line in res.stderr.splitlines():
        if "kernel-resource-usage" in line:
            if "Function Name:" in line:
                name = line.split("Function Name:")[1].split()[0]
            elif "ScratchSize" in line:
                if int(line.split(":")[-1].split()[0]) > scratch_limit(name):
                    spilled.append(name)
            continue
        if "packed-fp32-ops" in line and "not a recognized feature" in line:
            continue
        keep.append(line)
    # the remark lines come with source excerpts; print diagnostics only when the compile failed
    if res.returncode != 0:
        sys.stderr.write("\n".join(keep) + "\n")
        raise subprocess.CalledProcessError(res.returncode, HIPCC)
    asm = glob.glob(os.path.join(OBJDIR, base + "-hip-amdgcn-amd-amdhsa-gfx950.s")) + \
        glob.glob(os.path.join(OBJDIR, os.path.splitext(base)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s"))
    for path in asm:
        spilled += _spills_in_k_loops(path)
        with open(path) as f:
            early = early_scalar_reads(f)
        if early:
            raise RuntimeError("scalar registers read too early in %s: %d loads, first %s" % (base, len(early), early[0]))
    # (a profiling build carries the time stamps' registers as well: its spills are reported, not refused)
    if spilled and ("-DCUBE3D_PROFILE" in FLAGS or os.environ.get("CUBE3D_ALLOW_SPILLS")):
        sys.stderr.write("note: register spills in %s: %d kernels\n" % (base, len(set(spilled))))
    elif spilled:
        raise RuntimeError("register spills in %s: %s" % (base, sorted(set(spilled))))
    return obj


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(force: bool = True, jobs: int = 8) -> str:
    srcs = sources()
    deps = srcs + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in deps):
        return LIB
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs,
                    "-Wl,-rpath,/opt/rocm/lib"], check=True)
    os.replace(tmp, LIB)
    return LIB


def build_sanitized(outdir: str, jobs: int = 8) -> str:
    """The library with its HOST code under AddressSanitizer and UndefinedBehaviorSanitizer (the device
    code is compiled as usual), for the host-only check of the argument-validation layer.  Returns the
    path of ``libcube3d_san.so`` in `outdir`."""
    os.makedirs(outdir, exist_ok=True)
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-sanitize-recover=all", "-Xarch_host", "-fno-omit-frame-pointer", "-g"]

    def one(src):
        obj = os.path.join(outdir, os.path.basename(src) + ".o")
        res = subprocess.run([HIPCC, *FLAGS, *san, "-c", src, "-o", obj], stderr=subprocess.PIPE, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stderr)
            raise subprocess.CalledProcessError(res.returncode, HIPCC)
        return obj
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(one, sources()))
    lib = os.path.join(outdir, "libcube3d_san.so")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fsanitize=address", "-fsanitize=undefined",
                    "-fno-gpu-sanitize", "-o", lib, *objs, "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return lib


if __name__ == "__main__":
    print(build(force="--if-stale" not in sys.argv))
