"""The kernels' sources compiled for the CPU (tests/wave_cpu: one wave of 64
lanes, LDS blocks of exactly the launch's length) and run against the oracle
at small sizes: a store past a launch's LDS, LDS that one lane overwrites
before another has read it (the lanes run one after the other between two
synchronisations, lowest first and highest first), or LDS read before it is
written ends the run or changes a result.  Every run is a process of its own.
The comparison is tests/parity.py's."""

import json
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_14611_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

CHILD = r"""
import json, sys
sys.path.insert(0, __ROOT__)
import numpy as np
import oracle
from paper_2504_14611_amd import jdob
from paper_2504_14611_amd import workloads as W
from tests.parity import compare
from tests.test_gpu_grouped import compare_grouped
lib = jdob.load(__SO__)

def joint(d, **k):
    return jdob.eval_joint(d, jdob.eval_user_tables(d, stream=0), **k)

for n, c in enumerate(json.loads(sys.stdin.read())):
    print(c, flush=True)
    p = W.generate(W.WORKLOADS[c["base"]].replace(name="cpu", stream=c.get("stream", 8600), num_instances=c.get("I", 2),
                                                  dtype=c.get("dtype", "f32"), **c["kw"]))
    p["mode"] = int(p["mode"]) | c.get("mode", 0) if c.get("keep_mode", True) else c.get("mode", 0)
    for k, f in c.get("scale", {}).items():
        p[k] = float(p[k] * f) if np.isscalar(p[k]) else (p[k] * p[k].dtype.type(f)).astype(p[k].dtype)
    for k, v in c.get("fill", {}).items():
        p[k] = np.full_like(p[k], v)
    if c.get("busy"):
        p["t_free"] = (c["busy"] * p["deadline"].min(axis=1)).astype(p["t_free"].dtype)
    grouped = c.get("grouped", False)
    ora = oracle.solve_grouped(p, threads=4) if grouped else oracle.solve(p, threads=4)
    d = jdob.to_device(p, "cpu")
    calls = [jdob.solve_grouped] if grouped else [jdob.solve_batch]
    if not grouped and p.get("user_zeta") is None:
        calls.append(joint)
    for down in (0, 1):
        lib.wave_cpu_descending(down)
        for call in calls:
            for counters in (False, True):
                got = jdob.to_host(call(d, stream=0, counters=counters, freq=True))
                label = f"{call.__name__} counters={counters} descending={down}"
                if c.get("overflow"):
                    same = [k for k in got if got[k] is not None and (counters or k[:4] != "num_")]
                    ok = ~np.isnan(ora["energy"])
                    for k in same:
                        assert np.array_equal(got[k][ok], ora[k][ok]), (label, k, got[k], ora[k])
                    continue
                compare_grouped(p, got, ora, label) if grouped else compare(p, got, ora, label=label)
print("RUN COMPLETE", flush=True)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    """Builds the library once; returns a function that runs a list of cases."""
    tmp = tmp_path_factory.mktemp("wave_cpu")
    for f in os.listdir(CSRC):
        src = open(os.path.join(CSRC, f)).read()
        # what a header cannot define away: LDS, address spaces, empty asm that pins registers
        src = re.sub(r"extern __shared__[^;]*?(\w+)\[\];", r"unsigned char *const \1 = wave_cpu::lds();", src)
        src = re.sub(r'asm volatile\("" :[^;]*\);', "", src).replace("__attribute__((address_space(4)))", "")
        (tmp / f.replace(".hip", ".cpp")).write_text(src)
    objs = [str(f) for f in sorted(tmp.glob("*.cpp"))]
    flags = ["-O1", "-std=c++17", "-fPIC", "-ffp-contract=off", "-w", "-I", os.path.join(ROOT, "tests", "wave_cpu"),
             "-I", os.path.join(ROOT, "include")]
    procs = [subprocess.Popen([CLANG, *flags, "-c", f, "-o", f + ".o"]) for f in objs]
    assert all([p.wait() == 0 for p in procs])
    so = str(tmp / "libjdob_cpu.so")
    subprocess.run([CLANG, "-shared", "-o", so, *[f + ".o" for f in objs]], check=True)
    code = CHILD.replace("__ROOT__", repr(ROOT)).replace("__SO__", repr(so))

    def go(cases):
        r = subprocess.run([sys.executable, "-c", code], input=json.dumps(cases), capture_output=True, text=True,
                           timeout=600)
        assert r.returncode == 0 and "RUN COMPLETE" in r.stdout, \
            f"exit {r.returncode}\n{r.stdout[-600:]}\n{r.stderr[-3000:]}"
    return go


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_few_users_stay_in_the_launch(run, dtype):
    """The rows of few users are the shortest: at 1 to 17 users and GPU levels
    on both sides of every count of batch records."""
    run([dict(base="c2", mode=mode, dtype=dtype, kw=dict(N=N, L=1 + N % 4, K=4, J=J))
         for mode in (0, 1, 2, 8) for N in (1, 2, 3, 4, 5, 6, 9, 10, 12, 13, 16, 17)
         for J in (1, 2, 5, 8, 16, 31, 33, 48, 64, 65)])


SHAPES = [dict(base="p4a", kw=dict(N=10, L=22, K=4, J=32)), dict(base="c2b", kw=dict(N=20, L=22, K=8, J=9)),
          dict(base="c3", kw=dict(N=32, L=22, K=16, J=32)), dict(base="c4b", kw=dict(N=64, L=63, K=8, J=16)),
          dict(base="c4b", kw=dict(N=70, L=20, K=8, J=40)), dict(base="p4b", kw=dict(N=130, L=9, J=65)),
          dict(base="p4b", kw=dict(N=9, L=70, J=5)),
          dict(base="g10", grouped=True, kw=dict(N=7, L=6, K=5, J=9)),
          dict(base="p5", grouped=True, kw=dict(N=5, L=3, J=33))]


def test_shapes(run):
    run([dict(s, mode=mode, dtype=dtype) for s in SHAPES for mode in (0, 1, 2, 4) for dtype in ("f32", "f64")])


HETERO = [dict(base="h1", kw=dict(N=12, L=6, K=5, J=9)), dict(base="h1", kw=dict(N=16, L=66, K=3, J=4)),
          dict(base="h2", kw=dict(N=30, L=7, J=33)), dict(base="h2", kw=dict(N=63, L=5, J=12)),
          dict(base="h5", grouped=True, kw=dict(N=6, L=5, J=8)),
          dict(base="h1", grouped=True, I=1, kw=dict(N=10, L=60, K=5, J=8))]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_heterogeneous_users(run, dtype):
    """Several partition points' gamma orders are formed in one room: keys,
    then records."""
    run([dict(h, mode=mode, dtype=dtype) for h in HETERO for mode in (0, 1, 4, 8)])


QUEUED = [dict(base="c4b", kw=dict(N=33, L=9, K=8, J=16)), dict(base="c4b", kw=dict(N=100, L=22, K=8, J=64), I=1),
          dict(base="c2b", kw=dict(N=33, L=9, K=8, J=8)), dict(base="c2b", kw=dict(N=20, L=22, K=16, J=65)),
          dict(base="c2b", kw=dict(N=70, L=9, K=8, J=16))]


def test_queue_of_candidates(run):
    """A full queue of candidates is evaluated in the pass that filled it.
    (Cheap uploads and GPU levels leave many candidates to evaluate.)"""
    run([dict(q, dtype=dtype, mode=0, stream=8700 + n, scale=dict(deadline=a, p_tx=b, gpu_c=b, gpu_p_static=b))
         for q in QUEUED for dtype in ("f32", "f64") for n in range(3) for a in (0.7, 1.0, 1.5) for b in (0.01, 0.1)])


def test_heterogeneous_energies_that_overflow(run):
    """Frequencies whose squares are past binary32 make energies infinite.
    Feasibility and the counters do not depend on them, and with none finite
    the first candidate of the order wins.  (Instances whose energy is no
    number, infinity times no work, are left out.)"""
    run([dict(base=base, mode=mode, kw=kw, I=12, stream=8800 + f, keep_mode=False, overflow=True,
              scale=dict(cycles=f * 1e9, user_local_freq=f * 1e9, local_freq=f * 1e9, user_kappa=1e-8, kappa=1e-8))
         for base in ("h1", "h2") for kw in (dict(N=7, L=8, K=5, J=5), dict(N=20, L=6, K=4, J=12), dict(N=40, L=5, K=3, J=4))
         for mode in (0, 1, 2) for f in (5, 10, 12, 16)])


def test_rates_without_a_reciprocal(run):
    """Nothing to upload over links whose rates are denormal numbers: the
    upload takes no time, and offloading is feasible."""
    run([dict(base=base, kw=dict(N=N, L=9, K=4, J=8), I=32, stream=7001, keep_mode=False, mode=mode,
              fill=dict(bits=0.0, rate=1e-40)) for base in ("c2b", "p4b") for N in (3, 8, 20) for mode in (0, 1, 8)])


@pytest.mark.parametrize("L", [1, 2, 3, 4])
def test_grouping_over_few_partition_points(run, L):
    """Partition points searched as they come, with counting passes: winners
    and counters are the oracle's, on an idle and on a busy GPU.  Passes of
    several batch sizes, of one, and of two chunks of GPU levels."""
    run([dict(base=base, grouped=True, mode=mode, dtype=dtype, stream=8900 + n, kw=dict(N=N, L=L, K=5, J=J), busy=busy)
         for base in ("g20", "p5") for mode in (0, 1, 2, 4) for J in (1, 9, 33, 70) for n, (N, dtype, busy) in
         enumerate(((2, "f32", 0.0), (7, "f32", 0.4), (6, "f64", 0.2)))])


def test_gpu_power_at_the_ends(run):
    """The bound of the GPU energy without static or dynamic power, and with
    the cheapest frequency below and above the levels."""
    run([dict(base=base, kw=dict(N=N, L=9, J=J), I=4, scale=scale, stream=8950)
         for J in (2, 3, 4, 5, 16) for base, N in (("p4a", 10), ("p4b", 70), ("h2", 9)) for scale in
         (dict(gpu_p_static=0.0), dict(gpu_c=0.0), dict(gpu_p_static=1e-4), dict(gpu_p_static=1e4))])
