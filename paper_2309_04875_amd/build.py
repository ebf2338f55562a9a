"""Build paper_2309_04875_amd/libhb.so (the library), the _binding module (the native part of hb.py) and libhb_probes.so (bench.py's
measurement aids, a separate library that the product does not load) from csrc/ with hipcc for gfx950 (cross-compiles without a
GPU; the binding is host code, left out where torch or Python's headers are missing).

The group kernels exist once per (mode, slice width); hb_launch_part.hip is compiled once per mode and
width range so that the parts build in parallel.  Objects go to a temporary directory; only the
libraries are left in the tree.  Run as `python -m paper_2309_04875_amd.build`.
"""
import os
import shutil
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIBRARY = os.path.join(HERE, "libhb.so")
PROBES_LIBRARY = os.path.join(HERE, "libhb_probes.so")
BINDING = os.path.join(HERE, "_binding" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))     # the name says which Python it is for

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-fvisibility=hidden",
    "-Wall",
    # packed FP32 instructions are not to be generated on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

MODES = (0, 1, 2, 3, 4)                                 # DReLU, ReLU, sign shares; DReLU, ReLU on the shared-mask layout
WIDTH_RANGES = ((1, 16), (17, 32), (33, 48), (49, 64))
MP_PARTIES = (3, 4)                                     # multi-party kernels (two parties: the kernels above)
PARTY_WIDTH_RANGES = ((1, 4), (5, 8), (9, 16), (17, 32), (33, 48), (49, 64))   # party-faithful kernels
MP_WIDTH_RANGES = tuple((w, w + 3) for w in range(1, 33, 4)) + ((33, 48), (49, 64))


def _hipcc():
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(args):
    src, obj, defines = args
    cmd = [_hipcc()] + HIPCC_FLAGS + ["-D%s=%s" % kv for kv in defines] + ["-c", src, "-o", obj]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "not a recognized feature for this target" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed: %s\n%s" % (" ".join(cmd), out))
    return out


def _build_binding():
    """The native part of hb.py: host code against Python, torch and libhb.so beside it.  Without torch or Python's headers there is
    none, and hb.py does without.  (DT_RPATH: the libhb.so beside it, whatever LD_LIBRARY_PATH says, for hb.py loads that one.)"""
    headers = sysconfig.get_paths()["include"]
    try:
        import torch
    except ImportError:
        torch = None
    if torch is None or not os.path.exists(os.path.join(headers, "Python.h")):
        print("no _binding: %s" % ("torch cannot be imported" if torch is None else "Python.h is missing"))
        if os.path.exists(BINDING):
            os.remove(BINDING)                  # an older one would go on with the new library
        return
    inside = os.path.dirname(torch.__file__)
    lib = os.path.join(inside, "lib")
    tmp = BINDING + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DHB_TORCH_VERSION="%s"' % torch.__version__, "-I" + headers]
    for path in (os.path.join(inside, "include"), os.path.join(inside, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include"):
        cmd += ["-isystem", path]
    cmd += [os.path.join(CSRC, "hb_binding.cpp"), "-o", tmp, "-L" + HERE, "-l:" + os.path.basename(LIBRARY), "-L" + lib,
            "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10", "-Wl,--disable-new-dtags,-rpath,$ORIGIN"]
    subprocess.run(cmd, check=True)
    os.replace(tmp, BINDING)


def build(verbose: bool = False, jobs: int = 0) -> str:
    jobs = jobs or min(8, os.cpu_count() or 1)
    work = tempfile.mkdtemp(prefix="hb_build_")
    try:
        probes = (os.path.join(CSRC, "hb_probes.hip"), os.path.join(work, "hb_probes.o"), [])
        units = [(os.path.join(CSRC, "hb_api.hip"), os.path.join(work, "hb_api.o"), [])]
        for mode in MODES:
            for lo, hi in WIDTH_RANGES:
                units.append((os.path.join(CSRC, "hb_launch_part.hip"),
                              os.path.join(work, "part_m%d_w%d.o" % (mode, lo)),
                              [("HB_PART_MODE", mode), ("HB_PART_LO", lo), ("HB_PART_HI", hi)]))
        for parties in MP_PARTIES:
            for lo, hi in MP_WIDTH_RANGES:
                units.append((os.path.join(CSRC, "hb_mp_part.hip"),
                              os.path.join(work, "mp_p%d_w%d.o" % (parties, lo)),
                              [("HB_PART_PARTIES", parties), ("HB_PART_LO", lo), ("HB_PART_HI", hi)]))
        for lo, hi in PARTY_WIDTH_RANGES:
            units.append((os.path.join(CSRC, "hb_party_part.hip"), os.path.join(work, "party_w%d.o" % lo),
                          [("HB_PART_LO", lo), ("HB_PART_HI", hi)]))
        # the multi-party units take longest, those of four parties twice as long as those of three: started first, so that none
        # of them is left to compile alone at the end
        longest_first = sorted([probes] + units, key=lambda unit: ("hb_mp_part" not in unit[0], ("HB_PART_PARTIES", 4) not in unit[2]))
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            for out in pool.map(_compile, longest_first):
                if verbose and out.strip():
                    print(out)
        for objects, library in (([u[1] for u in units], LIBRARY), ([probes[1]], PROBES_LIBRARY)):
            tmp = library + ".tmp.%d" % os.getpid()
            cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC"] + objects + ["-o", tmp]
            subprocess.run(cmd, check=True)
            os.replace(tmp, library)
        _build_binding()
    finally:
        shutil.rmtree(work, ignore_errors=True)
    return LIBRARY


if __name__ == "__main__":
    print(build(verbose=True))
