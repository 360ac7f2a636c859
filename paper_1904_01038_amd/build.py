"""Builds libtfm.so (the HIP kernels and the C boundary) for gfx950 with hipcc, in-tree."""
import hashlib
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtfm.so")
HEADERS = [os.path.join(os.path.dirname(HERE), "include", "tfm.h")]
SOURCES = ["tfm.hip", "dispatch.hip", "gemm_naive.hip", "gemm_f32.hip", "gemm_mfma.hip", "gemm_thin.hip", "attention_naive.hip", "attention_mfma.hip", "norm.hip", "loss.hip", "embed.hip",
           "optim.hip", "batching.hip", "decode.hip", "adaptive.hip", "probe.hip"]
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-Wno-unused-result", "-Wno-unused-value",
         "-Wno-inline-asm"]      # (the direct-to-LDS load names m0 in its clobber list, which clang reports as a reserved register)


def _compile(src):
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr[-6000:]))
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    return obj, err


def fingerprint():
    """Of everything the library is made from: the sources and headers, their list, and the compiler's flags."""
    h = hashlib.sha256(repr((SOURCES, FLAGS)).encode())
    for path in [os.path.join(CSRC, n) for n in sorted(os.listdir(CSRC)) if n.endswith((".hip", ".h"))] + HEADERS:
        with open(path, "rb") as f:
            text = f.read()
        h.update(b"%s %d\n" % (os.path.basename(path).encode(), len(text)))
        h.update(text)
    return h.hexdigest()


def _compile_fingerprint(digest):
    """The library carries it as `tfm_built_from`: a library of other sources is recognised wherever it was copied (binding.lib)."""
    src, obj = os.path.join(OBJ, "built_from.cpp"), os.path.join(OBJ, "built_from.o")
    with open(src, "w") as f:
        f.write('extern "C" { extern const char tfm_built_from[65]; const char tfm_built_from[65] = "%s"; }\n' % digest)
    r = subprocess.run(["hipcc", "-x", "c++", "-fPIC", "-c", src, "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr[-4000:]))
    return obj


def build(verbose=True, jobs=8):
    """Compiles everything.  What an earlier build left is removed first, so that a build that fails leaves nothing to load."""
    if os.path.exists(LIB):
        os.remove(LIB)
    shutil.rmtree(OBJ, ignore_errors=True)
    os.makedirs(OBJ)
    digest = fingerprint()
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(_compile, SOURCES))
    objs = [o for o, _ in results] + [_compile_fingerprint(digest)]
    if verbose:
        for (_, err), src in zip(results, SOURCES):
            if err.strip():
                print("[%s]\n%s" % (src, err), file=sys.stderr)
    r = subprocess.run(["hipcc", "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", LIB],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr[-4000:])
    return LIB


if __name__ == "__main__":
    print(build())
