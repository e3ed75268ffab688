"""Build libvq.so (the HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

try:
    from . import check_async
except ImportError:                      # run as a script
    import check_async

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvq.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["vq_api.hip", "vq_dequant.hip", "vq_gemv.hip", "vq_gemv_fast.hip", "vq_gemv_res8.hip", "vq_gemv_mfma.hip", "vq_gemm.hip", "vq_gemm_fused.hip", "vq_gemm_dense.hip", "vq_assign.hip", "vq_gemv_down.hip", "vq_gemv_down_mfma.hip", "vq_gemv_v8.hip", "vq_colperm.hip", "vq_quantize.hip", "vq_quantize_loop.hip", "vq_gemm_v6.hip", "vq_gemv_lds.hip", "vq_gemv_rows.hip", "vq_dequant_tables.hip", "vq_gemv_down_lds.hip", "vq_gemv_products.hip"]
# packed-FP32 VALU forms are switched off for every device compile (they are not trusted on the test machines)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument"]
# Kernels in these files load registers asynchronously from inline assembly and wait for them with counted
# s_waitcnt.  The compiler does not know such a register is pending: if it spilled one, it would save the old
# contents.  Their kernels must therefore not spill at all; the build reads the compiler's resource remarks.
NO_SPILL = {"vq_gemv_mfma.hip", "vq_gemm_fused.hip", "vq_gemm_dense.hip", "vq_gemv_down.hip", "vq_gemv_down_mfma.hip", "vq_gemv_fast.hip", "vq_gemv_res8.hip", "vq_quantize.hip", "vq_gemm_v6.hip"}
# One exception, checked in the generated code of this image's compiler (ROCm 7.2): the 512-token GEMM tile saves
# five address registers at kernel entry, before its first asynchronous load, and reloads them in the epilogue.
SPILLS_ALLOWED = {"gemm_v8_kernelILi512E": 5}
REMARKS = ["-Rpass-analysis=kernel-resource-usage"]
# The same files, and the dot-product GEMV with its hand-issued LDS reads, get their device assembly audited for
# instructions that touch a register while an inline-assembly load into it is pending (check_async.py).
AUDITED = ["vq_gemv_mfma.hip", "vq_gemm_fused.hip", "vq_gemm_dense.hip", "vq_gemv_fast.hip", "vq_gemv_res8.hip", "vq_gemv_down.hip", "vq_gemv_down_mfma.hip", "vq_quantize.hip", "vq_gemm_v6.hip"]


# Files whose control-flow graphs hold paths that no run takes (two branches on the same loop-invariant value, taken
# differently) and on which the audit's queues therefore come up short: for each kernel the number of cross-block findings when
# those paths were last read.  Their single-block findings still fail the build; every other file, and every other kernel of these, must
# come out clean across blocks.
# vq_gemv_mfma.hip: the variants with two 16-row blocks per chunk, whose unrolled pass loop tests my_passes > 0 ("this wave has vectors in
# this group") and c < n_chunks ("chunks left") once per copy of its body.  A pass that is skipped in one copy and taken in the next would
# meet fewer loads in flight than its wait counts on; my_passes does not change inside the loop, and the loads of a taken pass are issued
# whether or not chunks are left.  groups, multi and parts are the same body (gemv_v6_mfma_body) in other grids: the findings of
# parts<R, 2> are, instruction by instruction and register by register, those of kernel<R, 8, 2, false, SIX>, and stand behind the same
# two tests, as a part of the columns is what a group is there; so are those of the three with activations through LDS (STAGED, 2).
CROSS_BLOCK_KNOWN = {"vq_gemv_mfma.hip": {
    "gemv_v6_mfma_kernelILi0ELi8ELi2ELb0ELi1E": 64, "gemv_v6_mfma_kernelILi0ELi8ELi2ELb0ELi0E": 20, "gemv_v6_mfma_kernelILi0ELi8ELi2ELb1ELi0E": 20,
    "gemv_v6_mfma_kernelILi8ELi8ELi2ELb0ELi0E": 16, "gemv_v6_mfma_kernelILi8ELi8ELi2ELb1ELi0E": 128, "gemv_v6_mfma_kernelILi12ELi8ELi2ELb0ELi0E": 24,
    "gemv_v6_mfma_kernelILi12ELi8ELi2ELb1ELi0E": 128, "gemv_v6_mfma_parts_kernelILi0ELi2ELi0E": 20, "gemv_v6_mfma_parts_kernelILi8ELi2ELi0E": 16,
    "gemv_v6_mfma_parts_kernelILi12ELi2ELi0E": 24, "gemv_v6_mfma_groups_kernelILi0ELi8ELi2E": 20, "gemv_v6_mfma_groups_kernelILi8ELi8ELi2E": 16,
    "gemv_v6_mfma_groups_kernelILi12ELi8ELi2E": 128, "gemv_v6_mfma_groups_kernelILi0ELi4ELi2E": 20, "gemv_v6_mfma_groups_kernelILi8ELi4ELi2E": 16,
    "gemv_v6_mfma_multi_kernelILi0ELi8ELi2ELi1E": 64, "gemv_v6_mfma_multi_kernelILi0ELi8ELi2ELi0E": 20, "gemv_v6_mfma_multi_kernelILi8ELi8ELi2ELi0E": 16,
    "gemv_v6_mfma_multi_kernelILi12ELi8ELi2ELi0E": 24,
    "gemv_v6_mfma_kernelILi0ELi8ELi2ELb0ELi2E": 20, "gemv_v6_mfma_multi_kernelILi0ELi8ELi2ELi2E": 20, "gemv_v6_mfma_parts_kernelILi0ELi2ELi2E": 20}}
# The compiler whose generated code the counted waits were last checked against (first line of `hipcc --version`).
VERIFIED_HIPCC = "HIP version: 7.2.26015-fc0010cf6a"


def hipcc_version(hipcc: str) -> str:
    try:
        return subprocess.run([hipcc, "--version"], stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout.splitlines()[0].strip()
    except (OSError, IndexError):
        return "unknown"


def check_no_spills(src: str, remarks: str) -> None:
    name = None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].strip()
        elif "VGPRs Spill:" in line:
            n = int(line.split("Spill:")[1].split()[0])
            allowed = max([v for k, v in SPILLS_ALLOWED.items() if name and k in name] + [0])
            if n > allowed:
                raise RuntimeError("%s: kernel %s spills %d vector registers; it must not (asynchronous loads)" % (src, name, n))
        elif "ScratchSize" in line and "bytes/lane" in line:
            # arrays the compiler keeps in scratch memory (a run-time choice among registers does that) travel through the same
            # counters as the asynchronous loads and cost a trip to memory each
            n = int(line.split(":")[-1].split()[0])
            allowed = max([4 * v + 4 for k, v in SPILLS_ALLOWED.items() if name and k in name] + [0])
            if n > allowed:
                raise RuntimeError("%s: kernel %s uses %d bytes of scratch memory per lane; it must not" % (src, name, n))


def build_binding() -> None:
    """_binding.so: the torch conveniences of the package in C++ (host code only)."""
    import sysconfig

    import torch
    root = os.path.join(os.path.dirname(torch.__file__))
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include",
               sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
    cmd += [flag for d in include for flag in ("-isystem", d)] + [os.path.join(CSRC, "binding.cpp"), "-o", BINDING]
    # (torch's own libraries are in the process before this one is imported, so no path to them is recorded)
    cmd += ["-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    subprocess.check_call(cmd)


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    binding = ThreadPoolExecutor(max_workers=1).submit(build_binding)
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        cmd = [hipcc] + FLAGS + (REMARKS if src in NO_SPILL else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if src in NO_SPILL:
            check_no_spills(src, out)
            out = "\n".join(l for l in out.splitlines() if "remark:" not in l)
        if verbose and out.strip():
            print(out)
    def audit(src):
        asm = check_async.device_asm(hipcc, FLAGS, os.path.join(CSRC, src))
        return src, check_async.audit_blocks(asm), check_async.audit(asm)
    with ThreadPoolExecutor(max_workers=len(AUDITED)) as pool:
        for src, in_block, cross_block in pool.map(audit, AUDITED):
            known = CROSS_BLOCK_KNOWN.get(src, {})
            findings = in_block + [f for f in cross_block if not any(k in f[0] for k in known)]
            if findings:
                name, label, text, regs = findings[0]
                raise RuntimeError("%s: %d instruction(s) touch a register with an asynchronous load pending, e.g. in %s %s: %s"
                                   % (src, len(findings), name, label, text))
            for kernel, n in known.items():
                found = sum(kernel in f[0] for f in cross_block)
                if found != n:
                    print("note: %s: %d cross-block findings of the asynchronous-load audit in %s, %d when its paths were last read; "
                          "read the new ones (python check_async.py on the device assembly)" % (src, found, kernel, n))
    if hipcc_version(hipcc) != VERIFIED_HIPCC:
        print("note: hipcc is '%s'; the counted waits of the kernels in %s were read against the code generated by '%s': "
              "run the GPU tests before relying on this build" % (hipcc_version(hipcc), ", ".join(AUDITED), VERIFIED_HIPCC))
    # no rpath: inside a PyTorch process the already-loaded HIP runtime (same soname) is the one used
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    binding.result()
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
