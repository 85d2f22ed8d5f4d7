"""Builds libmtsched.so (gfx950 only) in-tree with hipcc.  No fallback: a missing compiler is an error."""
import hashlib
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmtsched.so")

DEVICE_SOURCES = ["kernels_direct.hip", "kernels_igemm.hip", "kernels_stem.hip", "kernels_rowb.hip", "kernels_tile.hip", "kernels_dconv.hip"]
HOST_SOURCES = ["sched_core.cpp", "lanes.cpp", "runtime.cpp"]
COMMON = ["-O3", "-fPIC", "-std=c++20", "-Wall", "-Wno-unused-function"]
# packed-fp32 code generation is switched off for all device code
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
HOST_FLAGS = ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include"]


def _hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src, extra, obj_dir=None):
    out = os.path.join(obj_dir or OBJ, os.path.basename(src) + ".o")
    cmd = [_hipcc(), "-c", os.path.join(CSRC, src), "-o", out] + COMMON + extra
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return out


def source_digest():
    """What a library is built from: names and contents of the sources and headers, and the flags.  The library carries the digest (mt_source_digest),
    so that one of other sources is not mistaken for theirs."""
    h = hashlib.sha256(repr((COMMON, DEVICE_FLAGS, HOST_FLAGS)).encode())
    for folder in (CSRC, INCLUDE):
        for name in sorted(os.listdir(folder)):
            if name.endswith((".h", ".hip", ".cpp")):
                data = open(os.path.join(folder, name), "rb").read()
                h.update(b"%s %d " % (name.encode(), len(data)) + data)
    return h.hexdigest()


# host-side sanitizers (address + undefined behaviour) for the two host sources; device code is never instrumented
SANITIZE_HOST = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-omit-frame-pointer", "-g"]


def build(verbose=False, lib=None, sanitize=False):
    """sanitize=True builds the host objects with AddressSanitizer and UBSan into `lib` (give another path than the
    product library's): the CPU-only tests can then run against it with the sanitizer runtime preloaded, e.g.
    MTSCHED_LIB=<lib> LD_PRELOAD="$LD_PRELOAD:$(clang -print-file-name=libclang_rt.asan-x86_64.so)" pytest -m "not gpu"."""
    global LIB
    out = lib or LIB
    if not sanitize and lib:
        LIB = lib
    obj_dir = OBJ + ("_asan" if sanitize else "")
    os.makedirs(obj_dir, exist_ok=True)
    if os.path.exists(out):
        os.remove(out)                                       # a build that fails leaves no library of older sources behind
    digest = os.path.join(obj_dir, "source_digest.cpp")
    with open(digest, "w") as f:
        f.write('extern "C" const char mt_source_digest[];\nconst char mt_source_digest[] = "%s";\n' % source_digest())
    host_extra = HOST_FLAGS + (SANITIZE_HOST if sanitize else [])
    jobs = [(s, DEVICE_FLAGS, obj_dir) for s in DEVICE_SOURCES] + [(s, host_extra, obj_dir) for s in HOST_SOURCES] + [(digest, [], obj_dir)]
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(lambda j: _compile(*j), jobs))
    cmd = [_hipcc(), "-shared", "-fPIC", "-o", out + ".new"] + objs + ["--offload-arch=gfx950", "-lhsa-runtime64"]
    if sanitize:
        cmd += ["-fsanitize=address", "-fsanitize=undefined", "-fno-gpu-sanitize", "-shared-libsan"]
    subprocess.check_call(cmd)
    os.replace(out + ".new", out)
    if sanitize:
        return out
    if verbose:
        print("built", LIB)
    return LIB


def lib_path():
    return LIB


if __name__ == "__main__":
    if "--sanitize" in sys.argv:
        print("built", build(lib=os.path.join(HERE, "libmtsched_asan.so"), sanitize=True))
    else:
        build(verbose=True)
