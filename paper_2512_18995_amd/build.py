"""Build libdq.so (the gfx950 HIP library) in-tree with hipcc.

    python -m paper_2512_18995_amd.build

Every HIP source is compiled for gfx950 only, with packed-FP32 instructions
disabled (``-packed-fp32-ops``): hipcc would otherwise form v_pk_* FP32
operations from ordinary float code.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdq.so")
# helper program that compiles one tile pass per process (next to the library)
JITC = os.path.join(HERE, "dq_jitc")
# (source, object name, extra flags); the interpreted tile passes are built
# once per direction and precision so that the slow units compile in parallel
UNITS = [
    ("runtime.cpp", "runtime", []),
    ("jit.cpp", "jit", []),
    ("jit_rtc.cpp", "jit_rtc", []),
    ("kernels.hip", "kernels", []),
    ("tiles.hip", "tiles_fwd_c64", []),
    ("tiles.hip", "tiles_fwd_c128", ["-DDQ_TILES_F64"]),
    ("tiles.hip", "tiles_adj_c64", ["-DDQ_TILES_ADJ"]),
    ("tiles.hip", "tiles_adj_c128", ["-DDQ_TILES_ADJ", "-DDQ_TILES_F64"]),
    ("wg.hip", "wg_fwd", []),
    ("wg.hip", "wg_adj", ["-DDQ_WG_ADJ"]),
]
ARCH = "gfx950"
ROCM_LIB = "/opt/rocm/lib"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def flags():
    return ["-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-mllvm", "-simplifycfg-sink-common=false",
            "-Wall", "-Wno-unused-result", "-I" + os.path.join(HERE, "..", "include"),
            "-I" + os.path.join(HERE, "_build")]


def embed_tile_header(build_dir: str) -> None:
    """The runtime compiles tile passes with hipRTC against the text of
    tile_dev.h; write it as a raw string literal for jit.cpp."""
    text = open(os.path.join(CSRC, "tile_dev.h")).read()
    if ")DQSRC\"" in text:
        raise RuntimeError("tile_dev.h contains the raw-string delimiter")
    out = ("// generated by build.py from csrc/tile_dev.h\n"
           "static const char kTileDevSrc[] = R\"DQSRC(" + text + ")DQSRC\";\n")
    path = os.path.join(build_dir, "tile_dev_src.inc")
    if not os.path.exists(path) or open(path).read() != out:
        with open(path, "w") as f:
            f.write(out)


# the compiler's per-kernel resource report (registers, scratch, occupancy)
RESOURCE_REMARK = "-Rpass-analysis=kernel-resource-usage"
# kernels that stream the state through registers: none of them may keep
# registers in scratch memory (such tile kernels ran for minutes on states
# of a few thousand amplitudes)
NO_SCRATCH = ("k_tile_", "k_wg_", "k_dense_", "k_gate", "k_cnot", "k_cz", "k_init", "k_expval", "k_zdiag", "k_xtile", "k_lambda")


def parse_resources(text: str) -> dict:
    """{kernel: {"vgpr", "agpr", "scratch", "occupancy"}} from the compiler's
    kernel-resource-usage remarks."""
    import re
    out, cur = {}, None
    keys = (("VGPRs", "vgpr"), ("AGPRs", "agpr"), ("ScratchSize [bytes/lane]", "scratch"),
            ("Occupancy [waves/SIMD]", "occupancy"))
    for line in text.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            cur = m.group(1)
            out[cur] = {}
            continue
        if cur is None:
            continue
        for k, short in keys:
            m = re.search(r"remark:\s+" + re.escape(k) + r": (\d+)", line)
            if m:
                out[cur][short] = int(m.group(1))
    return out


def demangled_base(name: str) -> str:
    """The kernel's own identifier inside an Itanium-mangled name."""
    import re
    m = re.search(r"(k_[a-z0-9_]+?)(?:I|E|v|P)", name.split("GLOBAL__N_1")[-1])
    return m.group(1) if m else name


def build(verbose: bool = False, jobs: int = 0) -> str:
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    embed_tile_header(build_dir)
    cmds, objs = [], []
    for src, name, extra in UNITS:
        obj = os.path.join(build_dir, name + ".o")
        rem = [RESOURCE_REMARK, "-fno-caret-diagnostics"] if src.endswith(".hip") else []
        cmds.append([hipcc()] + flags() + extra + rem + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    jobs = jobs or min(len(cmds), max(1, os.cpu_count() or 1), 8)

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        return cmd, r

    failed, resources = [], {}
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        for cmd, r in ex.map(run, cmds):
            resources.update(parse_resources(r.stdout))
            # hipcc's host pass reports the device-only feature flag: not an error
            out = "\n".join(l for l in r.stdout.splitlines()
                            if "packed-fp32-ops" not in l and "kernel-resource-usage" not in l)
            if out.strip():
                print(out, file=sys.stderr)
            if r.returncode != 0:
                failed.append(cmd[-3])
    if failed:
        raise RuntimeError("compilation failed: " + ", ".join(failed))
    import json
    with open(os.path.join(build_dir, "kernel_resources.json"), "w") as f:
        json.dump(resources, f, indent=0, sort_keys=True)
    spilled = sorted(k for k, v in resources.items()
                     if v.get("scratch", 0) > 0 and demangled_base(k).startswith(NO_SCRATCH))
    if spilled:
        raise RuntimeError("kernels keep registers in scratch memory: " + ", ".join(spilled))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + objs + \
          ["-L" + ROCM_LIB, "-lhiprtc", "-Wl,-rpath," + ROCM_LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    build_helper(build_dir, verbose)
    return LIB


def build_helper(build_dir: str, verbose: bool = False) -> str:
    """dq_jitc: host-only C++ (hipRTC), built with the system C++ compiler."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        raise RuntimeError("no host C++ compiler for dq_jitc")
    tmp = JITC + ".tmp%d" % os.getpid()
    cmd = [cxx, "-O2", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + build_dir,
           os.path.join(CSRC, "jitc_main.cpp"), os.path.join(CSRC, "jit_rtc.cpp"), "-o", tmp,
           "-L" + ROCM_LIB, "-lhiprtc", "-Wl,-rpath," + ROCM_LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, JITC)
    return JITC


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
