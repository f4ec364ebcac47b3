"""The depth-first lanes on the CPU: tests/lane_source.cpp prints the code that the library generates for a program,
tests/lane_driver.cpp is compiled with it, and the waves run as fibers that take turns at random places."""
import atexit
import functools
import os
import platform
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_20225_amd", "csrc")

needs_host_lanes = pytest.mark.skipif(not shutil.which("g++") or platform.machine() != "x86_64", reason="needs g++ on x86-64")

@functools.lru_cache(maxsize=None)
def _generator():
    """tests/lane_source.cpp, built once."""
    folder = tempfile.mkdtemp(prefix="lane_source")
    atexit.register(shutil.rmtree, folder, ignore_errors=True)
    exe = os.path.join(folder, "lane_source")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "lane_source.cpp"), os.path.join(CSRC, "graph_build.cpp"),
                    "-L/opt/rocm/lib", "-lamdhip64", "-ldl", "-Wl,-rpath,/opt/rocm/lib", "-o", exe], check=True)
    return exe


def lane_source(prog):
    """The generated lanes of a program, as the library compiles them; None if it is no program or none of the lanes'."""
    fns, result = prog
    text = "%d %d\n" % (len(fns), result)
    for _, n_params, nodes in fns:
        text += "%d %d\n" % (n_params, len(nodes))
        text += "".join("%d %d %d %s\n" % (op, imm, len(ins), " ".join("%d %d" % tuple(r) for r in ins)) for op, ins, imm in nodes)
    res = subprocess.run([_generator()], input=text, capture_output=True, text=True)
    assert res.returncode in (0, 2, 3), res.stderr[-500:]
    return res.stdout if res.returncode == 0 else None


class Lanes:
    def __init__(self, prog, folder, optimise="-O1", source=None):
        with open(os.path.join(folder, "generated.inc"), "w") as f:
            f.write(source or lane_source(prog))
        self.exe = os.path.join(folder, "lanes")
        subprocess.run(["g++", "-std=c++17", optimise, "-w", "-I", str(folder), "-I", CSRC,
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
