"""Build the gfx950 shared library libterra_swin.so in-tree with hipcc.

Every HIP source under csrc/ is compiled for gfx950 only, with packed-fp32
instruction selection switched off, and linked into one shared library next
to this file.  Object files go to _build/ at the repository root.
"""

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libterra_swin.so")
# attn.hip holds one element type's kernels per compilation (0 float, 1
# bfloat16, 2 float16), so that they build in parallel.
SOURCES = [("attn.hip", ["-DTERRA_ATTN_T=1"]), ("attn.hip", ["-DTERRA_ATTN_T=2"]), ("attn.hip", ["-DTERRA_ATTN_T=0"]),
           ("route.hip", []), ("attn_win.hip", []), ("dtab.hip", []), ("plan.hip", []), ("block.hip", []),
           ("abi.hip", [])]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-result", "-Wno-unused-command-line-argument",
    "-I" + os.path.join(ROOT, "include"),
]


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature; drop that note.
    out = "\n".join(l for l in p.stdout.splitlines()
                    if "packed-fp32-ops' is not a recognized feature" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def build(verbose=False):
    """Compile every source and link libterra_swin.so.  Always rebuilds."""
    bdir = os.path.join(ROOT, "_build")
    os.makedirs(bdir, exist_ok=True)
    objs = [os.path.join(bdir, s.replace(".hip", "") + "".join(d[-1] for d in defs) + ".o") for s, defs in SOURCES]

    def comp(pair):
        (src, defs), obj = pair
        return _run([HIPCC] + FLAGS + defs + ["-c", os.path.join(CSRC, src), "-o", obj])

    with ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        outs = list(ex.map(comp, zip(SOURCES, objs)))
    tmp = LIB + ".tmp"
    outs.append(_run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs))
    os.replace(tmp, LIB)
    if verbose:
        for o in outs:
            if o.strip():
                print(o, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
