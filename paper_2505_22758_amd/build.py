"""Builds libflashformer.so (hipcc, gfx950) next to this file.  Run on the CPU container; the
built library travels with the tree to the GPU machine."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libflashformer.so")
SOURCES = ["flashformer.hip"] + [f"ff_{k}_{w}_hd{h}_g{g}.hip" for k in ("fused", "solo") for w in ("bf16", "int8", "int4")
                               for h, g in ((64, 4), (128, 4), (128, 8))]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"] + os.environ.get("FF_EXTRA_FLAGS", "").split()

# The int8 kernels' loops start on whole 128-byte instruction-cache lines.  Where the row-partitioned kernel's stream happens to
# lie is worth up to 0.9 %: 8B int8, eight layers, context 4096 / 1024, us per step 600 / 559 and 597 / 556 by chance,
# 593 / 552 aligned; bf16 does not change (734 / 734), int4 is slower aligned (594 / 598).
def source_flags(src):
    return ["-falign-loops=128"] if "int8" in os.path.basename(src) else []


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", "flashformer.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every translation unit (in parallel) and link libflashformer.so."""
    if not force and not is_stale():
        return LIB
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]
    procs = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        procs.append((src, obj, subprocess.Popen([HIPCC] + compile_flags + source_flags(src) + ["-c", "-o", obj, src],
                                                 stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    objs = []
    for src, obj, p in procs:
        out, _ = p.communicate()
        msgs = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n" + msgs)
        if verbose and msgs.strip():
            print(msgs)
        objs.append(obj)
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stdout + res.stderr)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
