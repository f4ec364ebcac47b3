"""Builds libtdf.so (the C-ABI library) for gfx950 with hipcc, in-tree, and beside it
libtdf_hooks.so: the same objects except that eval.hip is compiled with TDF_TEST_HOOKS, which lets
the tests make the host take its repeat paths.  The product library has no such switch."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtdf.so")
LIB_HOOKS = os.path.join(HERE, "libtdf_hooks.so")
SOURCES = ["graph_build.cpp", "tag_machine.hip", "forest_walk.hip", "cells.hip", "eval.hip", "jit.cpp"]
# headers the run-time compiler needs, embedded into the library as string literals
EMBEDDED = [("tdf.h", os.path.join(ROOT, "include", "tdf.h")), ("tdf_tables.h", os.path.join(CSRC, "tdf_tables.h")),
            ("engine.h", os.path.join(CSRC, "engine.h")), ("die_sync.h", os.path.join(CSRC, "die_sync.h")), ("step_device.h", os.path.join(CSRC, "step_device.h")),
            ("lane_device.h", os.path.join(CSRC, "lane_device.h"))]


def write_embedded_headers():
    out = ["// generated by build.py from the headers of the device code; do not edit"]
    for i, (name, path) in enumerate(EMBEDDED):
        text = open(path).read()
        assert ')TDFHDR"' not in text
        # string literals are limited in length by some compilers: split into pieces
        pieces = [text[k:k + 8000] for k in range(0, len(text), 8000)]
        out.append("static const char kEmbedded%d[] =" % i)
        out.extend('R"TDFHDR(%s)TDFHDR"' % p for p in pieces)
        out.append(";")
    out.append("static const char* const kEmbeddedSources[] = {%s};" % ", ".join("kEmbedded%d" % i for i in range(len(EMBEDDED))))
    out.append("static const char* const kEmbeddedNames[] = {%s};" % ", ".join('"%s"' % n for n, _ in EMBEDDED))
    out.append("static const int kEmbeddedCount = %d;" % len(EMBEDDED))
    path = os.path.join(CSRC, "embedded_headers.inc")
    text = "\n".join(out) + "\n"
    if not os.path.exists(path) or open(path).read() != text:
        open(path, "w").write(text)


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    write_embedded_headers()
    objs = []
    procs = []
    hooks_obj = os.path.join(CSRC, "eval_hooks.o")
    for src, obj, defs in [(s, os.path.join(CSRC, os.path.splitext(s)[0] + ".o"), []) for s in SOURCES] + \
            [("eval.hip", hooks_obj, ["-DTDF_TEST_HOOKS"])]:
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"] + defs + \
              ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if not defs:
            objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l]
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, "\n".join(lines)))
        if verbose and lines:
            print("\n".join(lines))
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs + ["-ldl"])
    eval_obj = os.path.join(CSRC, "eval.o")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_HOOKS] +
                          [hooks_obj if o == eval_obj else o for o in objs] + ["-ldl"])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
