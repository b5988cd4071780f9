"""Build libvegas for gfx950 with hipcc (in-tree: the shared library is
written next to this file)."""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libvegas_gfx950.so")
# the event kernels of one precision and integrand kind are a compilation each
# of the same file (source, defines); the longest compilations come first
PARTS = [(f"k_{w}.hip", [f"-DVEGAS_{w.upper()}_PREC={p}", f"-DVEGAS_{w.upper()}_KIND={k}"])
         for w in ("batch", "sample") for p in (64, 32) for k in range(4)]
SOURCES = PARTS + [(f, []) for f in ("k_sample.hip", "k_merge.hip", "k_batch.hip", "capi.cpp", "batch.cpp", "rtc.cpp",
                                     "noalloc.cpp", "probe.hip")]
# device sources the library hands to the runtime compiler for user integrands
RTC_HEADERS = [("kRtcInternal", "vegas_internal.hpp"), ("kRtcCommon", "device_common.hpp"),
               ("kRtcUser", "k_user_rtc.hpp")]
RTC_INC = "vegas_rtc_sources.inc"
ARCH = "gfx950"


def hipcc() -> str:
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def flags(objdir: str) -> list[str]:
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
            # no packed-FP32 instructions in generated code
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", INCLUDE, "-I", CSRC, "-I", objdir, "-Wall", "-Wno-unused-function"]


def write_rtc_sources(objdir: str) -> None:
    """Embed the device headers the runtime compiler needs as C++ raw strings."""
    delim = "vegas_rtc"
    out = ["// generated by build.py from csrc/ (do not edit)\n"]
    for name, fname in RTC_HEADERS:
        with open(os.path.join(CSRC, fname)) as f:
            text = f.read()
        if f"){delim}\"" in text:
            raise RuntimeError(f"{fname} contains the raw-string delimiter")
        out.append(f'static const char {name}[] = R"{delim}({text}){delim}";\n')
    path = os.path.join(objdir, RTC_INC)
    tmp = path + f".tmp{os.getpid()}"
    with open(tmp, "w") as f:
        f.write("".join(out))
    os.replace(tmp, path)


def build(verbose: bool = False, jobs: int = 8, out: str = LIB, objdir: str | None = None,
          extra: list[str] | None = None, link_extra: list[str] | None = None) -> str:
    """Compile every source for gfx950 and link the shared library `out`
    (extra / link_extra: more hipcc flags, e.g. host-pass sanitizers)."""
    objdir = objdir or os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    write_rtc_sources(objdir)

    def compile_one(unit) -> str:
        src, defines = unit
        obj = os.path.join(objdir, os.path.splitext(src)[0] + "".join(d.split("=")[1].rjust(3, "_") for d in defines) + ".o")
        cmd = [hipcc(), *flags(objdir), *defines, *(extra or []), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
        if verbose and r.stderr.strip():
            print(r.stderr, file=sys.stderr)
        return obj

    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = out + f".tmp{os.getpid()}"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *(link_extra or []), "-o", tmp, *objs, "-lhiprtc", "-lrocprofiler-sdk-roctx"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
