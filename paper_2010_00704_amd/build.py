"""Builds libbcnn.so (HIP, gfx950, with hipcc) and _marshal.so (argument marshalling for Python, with g++) next to this file."""
import glob
import os
import subprocess

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
LIB_PATH = os.path.join(_HERE, "libbcnn.so")
MARSHAL_PATH = os.path.join(_HERE, "_marshal.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    # packed-fp32 instruction forms are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a*b + c is fused only where the source says fma: float results are part of the interface
    "-ffp-contract=off",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(_HERE, "csrc", "*.hip")))


def _run(cmd):
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature name and says so; harmless
    log = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    return proc.returncode, log


def build_marshal(path=MARSHAL_PATH, torch_version=None):
    """Compile csrc/marshal.cpp, a Python extension on torch's C++ headers, into _marshal.so.  It loads under this Python
    and this torch only (torch's C++ layouts differ between versions)."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    libs = os.path.join(root, "lib")
    tmp = path + ".tmp.%d" % os.getpid()
    rc, log = _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                    '-DBCNN_TORCH_VERSION="%s"' % (torch_version or torch.__version__),
                    "-I", os.path.join(_ROOT, "include"), "-I", sysconfig.get_paths()["include"],
                    "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
                    "-isystem", "/opt/rocm/include", os.path.join(_HERE, "csrc", "marshal.cpp"), "-o", tmp,
                    "-L", libs, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath," + libs])
    if rc != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("building _marshal.so failed:\n" + log)
    os.replace(tmp, path)
    return path


def build_library(verbose=False):
    """Compile every .hip file under csrc/ (one hipcc process per file, in
    parallel) and link them into libbcnn.so; build _marshal.so (a warning where that cannot be built: the
    binding then marshals by ctypes).  Always compiles."""
    import shutil
    import tempfile
    from concurrent.futures import ThreadPoolExecutor

    srcs = sources()
    tmpdir = tempfile.mkdtemp(prefix="bcnn_build_")
    try:
        common = [f for f in FLAGS if f != "-shared"] + ["-I", os.path.join(_ROOT, "include"),
                                                         "-I", os.path.join(_HERE, "csrc")]
        objs = [os.path.join(tmpdir, os.path.basename(src) + ".o") for src in srcs]
        jobs = min(len(srcs), max(1, min(8, os.cpu_count() or 1)))
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            marshal = pool.submit(build_marshal)
            results = list(pool.map(lambda so: _run([HIPCC] + common + ["-c", so[0], "-o", so[1]]), zip(srcs, objs)))
        logs = []
        for src, (rc, log) in zip(srcs, results):
            if rc != 0:
                raise RuntimeError("hipcc failed on %s:\n%s" % (os.path.basename(src), log))
            if log.strip():
                logs.append(log)
        tmp = LIB_PATH + ".tmp.%d" % os.getpid()
        rc, log = _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
        if rc != 0:
            if os.path.exists(tmp):
                os.remove(tmp)
            raise RuntimeError("link failed:\n" + log)
        if verbose and (logs or log.strip()):
            print("\n".join(logs + [log]))
        os.replace(tmp, LIB_PATH)
        try:
            marshal.result()
        except Exception as e:                       # no host compiler, no C++ headers of torch's or Python's, ...
            import warnings
            if os.path.exists(MARSHAL_PATH):         # of another build
                os.remove(MARSHAL_PATH)
            warnings.warn("the binding marshals by ctypes, some microseconds a call slower: %s" % e, RuntimeWarning)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB_PATH


def resource_usage(jobs=None):
    """Device-only compile of every source with the compiler's per-kernel
    resource remarks switched on.  Returns {kernel symbol: {"scratch": bytes
    per lane, "vgpr_spills": n, "sgpr_spills": n, "vgprs": n, "agprs": n,
    "occupancy": waves per SIMD}}; nothing is linked or written."""
    import re
    import shutil
    import tempfile
    from concurrent.futures import ThreadPoolExecutor

    srcs = sources()
    tmpdir = tempfile.mkdtemp(prefix="bcnn_usage_")
    common = [f for f in FLAGS if f not in ("-shared", "-fPIC")] + [
        "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
        "-I", os.path.join(_ROOT, "include"), "-I", os.path.join(_HERE, "csrc")]
    fields = {"ScratchSize [bytes/lane]": "scratch", "VGPRs Spill": "vgpr_spills", "SGPRs Spill": "sgpr_spills",
              "VGPRs": "vgprs", "AGPRs": "agprs", "Occupancy [waves/SIMD]": "occupancy"}
    out = {}
    try:
        jobs = jobs or min(len(srcs), max(1, min(8, os.cpu_count() or 1)))
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            results = list(pool.map(
                lambda src: _run([HIPCC] + common + ["-c", src, "-o", os.path.join(tmpdir, os.path.basename(src) + ".o")]),
                srcs))
        for src, (rc, log) in zip(srcs, results):
            if rc != 0:
                raise RuntimeError("hipcc failed on %s:\n%s" % (os.path.basename(src), log))
            cur = None
            for line in log.splitlines():
                m = re.search(r"remark:\s+(.*?):\s+(\S+) \[-Rpass-analysis", line)
                if not m:
                    continue
                key, val = m.group(1).strip(), m.group(2)
                if key == "Function Name":
                    cur = out.setdefault(val, {"source": os.path.basename(src)})
                elif cur is not None and key in fields:
                    cur[fields[key]] = int(val)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return out


if __name__ == "__main__":
    print(build_library(verbose=True))
