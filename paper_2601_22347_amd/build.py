"""Builds libperq.so (HIP kernels + C ABI) for gfx950 with hipcc, and the Python extension module that calls it, in-tree."""
from __future__ import annotations

import hashlib
import importlib.util
import os
import shutil
import subprocess
import sysconfig
import warnings

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libperq.so")

SOURCES = ["perq_host.cpp", "perq_colabs.hip", "perq_butterfly.hip", "perq_mfma.hip", "perq_block.hip", "perq_api.hip",
           "perq_gemm.hip", "perq_qerr.hip", "perq_npo2.hip", "perq_npo2_12.hip", "perq_npo2_76.hip", "perq_npo2_32.hip"]

# -packed-fp32-ops: keep the compiler from fusing fp32 pairs into packed VALU instructions.
HIP_FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=off",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             # keep the one-lane ticket atomic of the matrix-core kernel as written: the wave-level
             # rewrite of uniform atomics reads the result back at once and stalls on it
             "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
             "-Wall", "-Wno-unused-command-line-argument"]
MODULE_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas", "-DUSE_ROCM=1",
                "-D__HIP_PLATFORM_AMD__=1"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Compile every source and link libperq.so, then the extension module where Python calls can be made at all
    (module_lacks); always recompiles."""
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc(), *HIP_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
               "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, cmd, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "not a recognized feature" not in l)
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{' '.join(cmd)}\n{out}")
        if verbose and out.strip():
            print(out)
    link = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    res = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}")
    lacks = module_lacks()
    if lacks:
        warnings.warn(f"libperq.so is built, the extension module for Python is not: no {', no '.join(lacks)}")
    else:
        module = build_module()
        for name in os.listdir(PKG):                       # modules made from earlier sources
            if name.startswith("_perq_torch") and name.endswith(".so") and name != os.path.basename(module):
                os.unlink(os.path.join(PKG, name))
    return LIB


def _torch_dir() -> str | None:
    spec = importlib.util.find_spec("torch")
    return os.path.dirname(spec.origin) if spec and spec.origin else None


def module_lacks() -> list[str]:
    """What the extension module needs beside libperq.so and is not here; the C library needs none of it."""
    where, lacks = _torch_dir(), []
    if where is None:
        lacks.append("PyTorch")
    elif not os.path.exists(os.path.join(where, "include", "c10", "hip", "HIPStream.h")):
        lacks.append("PyTorch headers for ROCm")
    if shutil.which("g++") is None:
        lacks.append("g++")
    if not os.path.exists(os.path.join(sysconfig.get_path("include"), "Python.h")):
        lacks.append("Python headers")
    return lacks


def module_path() -> str:
    """The extension module's file.  Its name stands for all it was made from, sources and the versions of PyTorch and
    Python, so that a module that no longer fits is not found, instead of loaded."""
    import torch
    made_from = hashlib.sha256(repr((MODULE_FLAGS, torch.__version__, sysconfig.get_config_var("EXT_SUFFIX"))).encode())
    for path in (os.path.join(CSRC, "perq_torch.cpp"), os.path.join(ROOT, "include", "perq.h")):
        with open(path, "rb") as f:
            made_from.update(f.read())
    return os.path.join(PKG, f"_perq_torch_{made_from.hexdigest()[:12]}.so")


def build_module() -> str:
    """Compile the extension module (host code; needs libperq.so to link against)."""
    import torch
    where, module = _torch_dir(), module_path()
    # under a name of this process's own, then renamed: another process finds the whole file or none
    made = f"{module}.{os.getpid()}.tmp"
    cmd = [shutil.which("g++") or "g++", *MODULE_FLAGS, f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(where, "include"),
           "-isystem", os.path.join(where, "include", "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_path("include"), os.path.join(CSRC, "perq_torch.cpp"), "-o", made,
           "-L", PKG, "-l:libperq.so", "-Wl,-rpath,$ORIGIN", "-L", os.path.join(where, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip"]
    try:
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"g++ failed on perq_torch.cpp:\n{' '.join(cmd)}\n{res.stdout}")
        os.replace(made, module)
    finally:
        if os.path.exists(made):
            os.unlink(made)
    return module


def _device_assembly(src: str) -> str:
    import tempfile
    with tempfile.TemporaryDirectory() as tmp:
        asm = os.path.join(tmp, os.path.splitext(src)[0] + ".s")
        flags = [f for f in HIP_FLAGS if f != "-fPIC"]
        cmd = [hipcc(), *flags, "--offload-device-only", "-S", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
               "-x", "hip", os.path.join(CSRC, src), "-o", asm]
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed:\n{res.stdout}")
        return open(asm).read()


def check_product_waits() -> set:
    """Compiler check for the counted waits of the products' tile kernels (perq_gemm.hip), about six seconds.

    A stage begins with a wait that lets the loads of the stages behind it be on their way, and requests one
    more stage.  The waits may count loads into LDS only, and every one of those has to be there: one wait of
    NBUF - 1 stages, then a wait of NBUF - 2 stages and a stage of loads each.  Returns the kernel variants
    checked, (MXFP4, MT, NT, WM, WN, NBUF, DWORDS, SHORT); raises on a mismatch."""
    import re
    text = _device_assembly("perq_gemm.hip")
    checked = set()
    for m in re.finditer(r"\n(_ZN4perq\S*gemm_tile_kernelILb(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi\dELb(\d)ELb(\d)\S*): +; @", text):
        mx, mt, nt, wm, wn, nbuf, dwords, short = (int(v) for v in m.groups()[1:])
        loads = 4 * (mt * wm + nt * wn) // (wm * wn)                 # of a wave and stage
        # scale bytes, loaded before the first stage and once in the loop over whole superstages; not counted by the waits
        scales = 2 * -(-(mt * wm + nt * wn) // (wm * wn)) if mx and dwords else 0
        body = text[m.end():text.index(".Lfunc_end", m.end())].split("\n")
        issued = sum("buffer_load_dwordx4" in l and " lds" in l for l in body)
        waits = [int(re.search(r"vmcnt\((\d+)\)", l).group(1)) for i, l in enumerate(body)
                 if "vmcnt(" in l and any("s_barrier" in k for k in body[i + 1:i + 5])]
        stages = len(waits) - 1
        # (rows of less than a superstage: the four stages of the partial one, else also whole ones with and without the next)
        if (stages != 4 if short else stages < 12) or sorted(waits) != sorted([loads * (nbuf - 1)] + [loads * (nbuf - 2)] * stages) or \
                issued != loads * (nbuf + stages) + scales:
            raise RuntimeError(f"{m.group(1)}: {loads} loads a stage, {issued} in all, waits {waits}")
        checked.add((mx, mt, nt, wm, wn, nbuf, dwords, short))
    if not checked:
        raise RuntimeError("no tile kernel found")
    return checked


def check_statistics_order() -> int:
    """Compiler check for the column statistics in one launch (perq_colabs.hip), a few seconds.

    A workgroup counts itself in when its partial sums are where the whole device sees them, and the last one reads
    all of them.  What orders this is in the instructions: partials are stored with device scope (sc1), the wave waits
    for its stores before the barrier ahead of the count, and partials are read with device scope.  Returns the number of
    kernel variants checked; raises on a mismatch."""
    import re
    text = _device_assembly("perq_colabs.hip")
    checked = 0
    for m in re.finditer(r"\n(_ZN4perq\S*colabs_partial_kernelILb\dELb0ELb\d\S*): +; @", text):
        body = [l.split(";")[0].strip() for l in text[m.end():text.index(".Lfunc_end", m.end())].split("\n")]
        at = [i for i, l in enumerate(body) if l.startswith("global_atomic_add ")]
        stores = [i for i, l in enumerate(body) if l.startswith("global_store_dwordx2 ") and l.endswith(" sc1")]
        if len(at) != 1 or len(stores) != 1 or stores[0] > at[0]:
            raise RuntimeError(f"{m.group(1)}: counts at lines {at}, device-scope stores at lines {stores}")
        before = [l for l in body[stores[0] + 1:at[0]] if re.match(r"(s_waitcnt|s_barrier|global_|flat_|buffer_)", l)]
        # (the partial of two launches and the result of a single slice, then: wait, barrier, count)
        order = [l.split()[0] for l in before if not l.startswith("s_waitcnt lgkmcnt")]
        last = [l for l in before if l.startswith("s_waitcnt") and "vmcnt(0)" in l][-1:]
        if order[-2:] != ["s_waitcnt", "s_barrier"] or not last or before.index(last[0]) < max(i for i, l in enumerate(before) if "store" in l):
            raise RuntimeError(f"{m.group(1)}: between the partial and the count {before}")
        reads = [l for l in body[at[0]:] if re.match(r"(global|flat|buffer)_load", l)]
        if len(reads) != 32 or any(not l.startswith("global_load_dwordx2 ") or not l.endswith(" sc1") for l in reads):
            raise RuntimeError(f"{m.group(1)}: partials read by {reads}")
        checked += 1
    if checked == 0:
        raise RuntimeError("no kernel with arrivals found")
    return checked


def _built_kernels(name: str):
    """(symbol, instructions) of every kernel in libperq.so whose name holds `name` (an expression), from its disassembly."""
    import re
    import tempfile
    llvm = os.path.join(os.path.dirname(os.path.dirname(hipcc())), "llvm", "bin", "llvm-objdump")
    run = lambda *args, **kw: subprocess.run([llvm, *args], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, **kw).stdout
    with tempfile.TemporaryDirectory() as tmp:
        lib = shutil.copy(LIB, tmp)
        run("--offloading", lib, cwd=tmp)
        for part in sorted(os.listdir(tmp)):
            with open(os.path.join(tmp, part), "rb") as f:
                if not part.endswith("gfx950") or not re.search(name.encode(), f.read()):
                    continue
            for m in re.finditer(rf"\n[0-9a-f]+ <(\S*{name}\S*)>:\n((?:.+\n)*)", run("-d", os.path.join(tmp, part))):
                yield m.group(1), [l.split("//")[0].strip() for l in m.group(2).split("\n") if l.startswith("\t")]


def check_ticket_register() -> int:
    """Check of the built library for the run-time row schedule's tickets (perq_block.hip, perq_mfma.hip), a few seconds.

    A ticket is on its way into a register of its own while the compiler's code runs, so no other instruction may
    name that register (as a part of a tuple neither), and every kernel has to have it.  Returns the number of kernel
    variants checked; raises on a mismatch.  `python -m paper_2601_22347_amd.build --check-ticket-register`."""
    import re
    checked = 0
    for kernel, number in (("block_kernel", 127), ("mfma_kernel", 255)):
        found = 0
        for symbol, body in _built_kernels(rf"perq\S*\d{kernel}I"):
            drawn = 0
            for line in body:
                if re.match(rf"(global_atomic_add v{number}, |v_readfirstlane_b32 s\d+, v{number}$)", line):
                    drawn += line.startswith("global_atomic_add")
                    continue
                used = [int(v) for v in re.findall(r"\bv(\d+)\b", line)] + [int(v) for v in re.findall(r"\bv\[\d+:(\d+)\]", line)]
                if any(v >= number for v in used):
                    raise RuntimeError(f"{symbol}: {line}")
            if drawn < 2:
                raise RuntimeError(f"{symbol}: {drawn} draws")
            found += 1
        if found == 0:
            raise RuntimeError(f"no {kernel} found")
        checked += found
    return checked


def check_lane_stages() -> int:
    """Check of the built library for the butterflies across lanes of block_kernel, a few seconds.

    They are instructions that the compiler does not look into: it keeps no distance between them and what it puts around
    them.  A vector instruction's result may be read through DPP, and by a swap of half-waves or rows of lanes, two wait states
    later.  Returns the number of stages' instructions and swaps checked; raises on a mismatch."""
    import re
    checked = 0
    for symbol, body in _built_kernels(r"perq\S*\d+block_kernelI"):
        for i, line in enumerate(body):
            if line.startswith("v_fmac_f32_dpp "):
                reads = {int(re.match(r"v_fmac_f32_dpp v\d+, v(\d+),", line).group(1))}
            elif line.startswith("v_permlane"):
                reads = {int(v) for v in re.findall(r"\bv(\d+)\b", line)}
            else:
                continue
            checked += 1
            states = 0
            for before in reversed(body[max(0, i - 2):i]):
                nop = re.match(r"s_nop (\d+)", before)
                if states < 2 and not nop and before.startswith("v_fmac_f32_dpp" if line.startswith("v_permlane") else "v_"):
                    first = re.match(r"\S+ v(\d+|\[\d+:\d+\])", before)
                    ends = [int(v) for v in re.findall(r"\d+", first.group(1))] if first else []
                    if ends and reads & set(range(ends[0], ends[-1] + 1)):
                        raise RuntimeError(f"{symbol}: {before} | {line}")
                states += int(nop.group(1)) + 1 if nop else 1
    if checked == 0:
        raise RuntimeError("no stage across lanes found")
    return checked


def check_table_reads() -> int:
    """Compiler check for the prepared-form reads of the matrix-core kernel (perq_mfma.hip).

    The kernel issues eight 16-byte loads as instructions, waits for them by count and only then hands
    the eight register tuples back to the compiler (a comment line in the assembly lists them).  Were the
    compiler to move one of the tuples in between, it would copy registers whose data have not arrived.
    This compiles the file to assembly (about three minutes) and checks, for every kernel variant, that
    the tuples handed back are the ones the loads were given.  Returns the number of variants checked;
    raises on a mismatch.  Run after a compiler upgrade: `python -m paper_2601_22347_amd.build --check-table-reads`."""
    import re
    text = _device_assembly("perq_mfma.hip")
    checked = 0
    for m in re.finditer(r"\n(_ZN4perq\S*mfma_kernel\S*): +; @", text):
        body = text[m.end():text.index("s_endpgm", m.end())].split("\n")
        handed = [l for l in body if "table reads have landed in" in l]
        if not handed:
            continue
        loads = [re.search(r"global_load_dwordx4 (v\[\d+:\d+\])", body[i + 1]).group(1)
                 for i, l in enumerate(body[:-1])
                 if "#ASMSTART" in l and re.search(r"global_load_dwordx4 v\[\d+:\d+\], v\[\d+:\d+\], off\s*$", body[i + 1])]
        for l in handed:
            regs = sorted(re.findall(r"v\[\d+:\d+\]", l))
            if len(loads) % 8 != 0 or regs not in (sorted(loads[:8]), sorted(loads[-8:])):
                raise RuntimeError(f"{m.group(1)}: loads into {loads}, handed back {regs}")
            checked += 1
    if checked == 0:
        raise RuntimeError("no kernel variant with the prepared-form reads found")
    return checked


if __name__ == "__main__":
    import sys
    if "--check-table-reads" in sys.argv:
        print(check_table_reads(), "kernel variants checked")
    elif "--check-ticket-register" in sys.argv:
        print(check_ticket_register(), "kernel variants checked")
    else:
        print(build(verbose=True))
