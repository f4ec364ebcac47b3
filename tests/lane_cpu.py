"""The depth-first lanes on the CPU: the library prints the code that it generates for a program (no GPU is needed for
that), tests/lane_driver.cpp is compiled with it, and the waves run as fibers that take turns at random places."""
import concurrent.futures
import json
import os
import platform
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_20225_amd", "csrc")

needs_host_lanes = pytest.mark.skipif(not shutil.which("g++") or platform.machine() != "x86_64", reason="needs g++ on x86-64")

_DUMP = """
import json, sys
sys.path.insert(0, %r)
from paper_2410_20225_amd import tdf
fns, r, grad = json.load(sys.stdin)
fns = [(n, p, [(op, [tuple(i) for i in ins], imm) for op, ins, imm in nodes]) for n, p, nodes in fns]
tdf.graph_precompile(tdf.graph_build(fns, r, want_grad=grad))
"""


def _lane_source(job):
    res = subprocess.run([sys.executable, "-c", _DUMP % ROOT], input=job, capture_output=True, text=True, env=dict(os.environ, TDF_JIT_DUMP="1"))
    assert res.returncode == 0, res.stderr[-2000:]
    return res.stderr[res.stderr.index('#include "lane_device.h"'):]


_pool = concurrent.futures.ThreadPoolExecutor(6)
_sources = {}   # by program: the library compiles what it prints, which takes some seconds a program


def prefetch(prog, want_grad=False):
    job = json.dumps([*prog, want_grad])
    if job not in _sources:
        _sources[job] = _pool.submit(_lane_source, job)
    return _sources[job]


def lane_source(prog, want_grad=False):
    """The generated lanes of a program, as the library compiles them."""
    return prefetch(prog, want_grad).result()


class Lanes:
    def __init__(self, prog, folder, defines=()):
        self.source = lane_source(prog)
        with open(os.path.join(folder, "generated.inc"), "w") as f:
            f.write(self.source)
        self.exe = os.path.join(folder, "lanes")
        subprocess.run(["g++", "-std=c++17", "-O1", "-w", *("-D" + d for d in defines), "-I", str(folder), "-I", CSRC,
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "tests"),
                        os.path.join(ROOT, "tests", "lane_driver.cpp"), "-o", self.exe], check=True)

    def run(self, args, **job):
        """args: one tuple per instance.  Numbers and lists of `job` go to the driver as they are."""
        job = dict(job, args=[v for t in args for v in t], n_args=len(args[0]), n_inst=len(args))
        text = "".join("%s %d %s\n" % (k, len(v), " ".join(map(str, v))) for k, v in
                       ((k, list(v) if hasattr(v, "__len__") else [v]) for k, v in job.items()))
        res = subprocess.run([self.exe], input=text, capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, "the lanes ended with status %d: %s" % (res.returncode, res.stderr[-500:])
        out = {}
        for line in res.stdout.splitlines():
            key, _, *v = line.split()
            out[key] = [int(x) for x in v]
        for k in ("status", "tags", "tokens", "leaves", "cells", "depth", "level", "sweeps", "records", "turns", "hung"):
            if k in out:
                out[k] = out[k][0]
        assert "hung" not in out, "the lanes do not come to an end"
        return out
