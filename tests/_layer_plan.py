"""Runs layer_plan_probe.cpp (the layer's host rules, compiled with g++)."""
import atexit
import functools
import os
import shutil
import subprocess
import tempfile
from collections import namedtuple

HERE = os.path.dirname(os.path.abspath(__file__))
Plan = namedtuple("Plan", "slots W ns parts room fit_W fit_ns fit_parts workspace")


@functools.lru_cache(maxsize=None)
def _probe():
    d = tempfile.mkdtemp(prefix="layer_plan_")
    atexit.register(shutil.rmtree, d, ignore_errors=True)
    exe = os.path.join(d, "probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", os.path.join(HERE, "..", "paper_2608_02438_amd", "csrc"),
                    os.path.join(HERE, "layer_plan_probe.cpp"), "-o", exe], check=True)
    return exe


def _ask(lines):
    r = subprocess.run([_probe()], input="\n".join(lines) + "\n", capture_output=True, text=True,
                       check=True)
    out = r.stdout.split("\n")[:-1]
    assert len(out) == len(lines)
    return out


def plans(cases):
    """Plan of every (H, heads, kv, ffn, batch, B, C_max)."""
    return [Plan(*map(int, s.split())) for s in
            _ask(["plan " + " ".join(map(str, c)) for c in cases])]


def walks(cases):
    """Whether the parts of every (nkv, B, W, ns, contexts) fit together."""
    return [s == "1" for s in
            _ask(["walk %d %d 0 %d %d %d %s" % (nkv, B, W, ns, len(ctx), " ".join(map(str, ctx)))
                  for nkv, B, W, ns, ctx in cases])]


def gemm_plans(cases):
    """(tile size, k parts, stages, part boundaries) of every projection (n0, n1, N,
    K, M, slab floats)."""
    out = [list(map(int, s.split())) for s in
           _ask(["gemm " + " ".join(map(str, c)) for c in cases])]
    return [(o[0], o[1], o[2], o[3:]) for o in out]
