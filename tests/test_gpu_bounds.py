"""GPU parity where partition points and batches are dropped by energy bounds.

The launches without work counters search only what a lower bound of the
energy leaves, and the counters come from a walk of their own: both launches
are compared with the oracle, at the sizes where the bounds' layout changes
(one to three partition points, more than 64 of them, lanes per partition
point from 1 to 64, batch sizes beyond one wave, GPU levels beyond one wave),
with and without local computing as the energy to beat, on a busy GPU, and
with users who are all alike.  The comparison is tests/parity.py's: the
winner, its levels, energy and release time are the oracle's bit for bit,
near-ties aside.
"""

import numpy as np
import pytest

import oracle
from paper_2504_14611_amd import jdob
from paper_2504_14611_amd import workloads as W
from tests.parity import compare
from tests.test_gpu_grouped import compare_grouped

pytestmark = pytest.mark.gpu

# base (c2b: some users gain by offloading; p4a, p4b: all do; c4b: no local
# computing; c3: local computing wins), instances, sizes
SHAPES = [
    ("c2b", 192, dict(N=12, L=1, K=8, J=8)),
    ("c2b", 192, dict(N=12, L=2, K=8, J=8)),
    ("c2b", 192, dict(N=12, L=3, K=8, J=8)),
    ("p4a", 128, dict(N=10, L=16, J=33)),
    ("p4b", 128, dict(N=10, L=17, J=64)),
    ("c4b", 48, dict(N=64, L=33, K=16, J=48)),
    ("c4b", 24, dict(N=130, L=63, K=8, J=70)),
    ("p4b", 48, dict(N=65, L=64, J=12)),
    ("c2b", 64, dict(N=20, L=65, K=5, J=65, cycles=("lu", 1e5, 1e7))),
    ("c3", 256, dict(N=32, L=130, K=4, J=9, cycles=("lu", 1e5, 1e6))),
    ("p4b", 12, dict(N=9, L=255, J=5)),
    ("c2b", 96, dict(N=17, L=21, K=16, J=1)),
]


def both(prob, call):
    """The policy without the work counters and with them, on the host."""
    import torch
    d = jdob.to_device(prob)
    out = [jdob.to_host(call(d, counters=c, freq=True)) for c in (False, True)]
    torch.cuda.synchronize()
    return out


def joint(d, **kw):
    return jdob.eval_joint(d, jdob.eval_user_tables(d), **kw)


def problem(base, n, mode, busy, dtype, seed, **kw):
    p = W.generate(W.WORKLOADS[base].replace(name="bounds", stream=seed, num_instances=n, dtype=dtype, **kw))
    p["mode"] = int(p["mode"]) | mode
    if busy:
        p["t_free"] = (0.4 * p["deadline"].min(axis=1)).astype(p["t_free"].dtype)
    return p


@pytest.mark.parametrize("mode", [0, 1, 2, 8])
@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_bounds_solve(k, mode):
    base, n, kw = SHAPES[k]
    dtype = "f64" if k % 5 == 4 and kw["N"] <= 64 else "f32"
    prob = problem(base, n, mode, k % 2, dtype, 8000 + k, **kw)
    label = f"bounds {base} {kw} mode={prob['mode']} {dtype}"
    print(f"[gpu] {label}", flush=True)
    ora = oracle.solve(prob, threads=16)
    for gpu in both(prob, jdob.solve_batch):
        compare(prob, gpu, ora, label=label)


@pytest.mark.parametrize("mode", [0, 1, 4, 8])
@pytest.mark.parametrize("base,n,kw", [("c2b", 48, dict(N=9, L=7, K=8, J=12)), ("g10", 48, dict(N=7, L=66, K=4, J=8)),
                                       ("p5", 48, dict(N=8, L=3, J=65)), ("g20", 24, dict(N=13, L=32, K=16, J=7))])
def test_bounds_grouped(base, n, kw, mode):
    prob = problem(base, n, mode, mode == 4, "f32", 8100, **kw)
    label = f"bounds grouped {base} {kw} mode={prob['mode']}"
    print(f"[gpu] {label}", flush=True)
    ora = oracle.solve_grouped(prob, threads=16)
    for gpu in both(prob, jdob.solve_grouped):
        compare_grouped(prob, gpu, ora, label)


def test_bounds_joint_takes_upload_times_from_its_tables():
    """The joint call reads the upload times of its tables, not the rates:
    with the times of another problem it answers that problem."""
    import torch
    p = problem("c2b", 96, 0, False, "f32", 8200, N=20, L=22, K=16, J=16)
    q = dict(p)
    q["bits"] = (p["bits"] * np.float32(0.25)).astype(np.float32)
    dp, dq = jdob.to_device(p), jdob.to_device(q)
    want = jdob.to_host(jdob.solve_batch(dq, counters=False))
    got = jdob.to_host(jdob.eval_joint(dp, jdob.eval_user_tables(dq), counters=False))
    torch.cuda.synchronize()
    for k in want:
        if want[k] is not None:
            assert np.array_equal(want[k], got[k]), k


# Heterogeneous users: one, two and four partition points' orders at a time
# (64, 32 and 16 lanes each), fewer partition points than that, and more than
# 64 of them; both precisions.
HETERO = [("h1", 96, dict(N=16, L=3, K=8, J=12)), ("h2", 96, dict(N=15, L=66, J=9)),
          ("h1", 64, dict(N=17, L=21, K=5, J=65)), ("h2", 64, dict(N=32, L=6, J=16)),
          ("h1", 48, dict(N=33, L=9, K=9, J=7)), ("h2", 32, dict(N=64, L=5, J=33)),
          ("h2", 96, dict(N=9, L=2, J=64)), ("h1", 64, dict(N=1, L=30, K=4, J=1))]


@pytest.mark.parametrize("mode", [0, 1, 2, 4, 8])
@pytest.mark.parametrize("k", range(len(HETERO)))
def test_bounds_hetero(k, mode):
    base, n, kw = HETERO[k]
    prob = problem(base, n, mode, k % 2 == 0, "f64" if k % 3 == 2 else "f32", 8300 + k, **kw)
    label = f"bounds {base} {kw} mode={prob['mode']}"
    print(f"[gpu] {label}", flush=True)
    ora = oracle.solve(prob, threads=16)
    for gpu in both(prob, jdob.solve_batch):
        compare(prob, gpu, ora, label=label)


# with the orders kept per partition point, and where they do not fit
@pytest.mark.parametrize("mode", [0, 1, 4])
@pytest.mark.parametrize("base,n,kw", [("h5", 48, dict(N=9, L=11, J=12)), ("h1", 16, dict(N=17, L=66, K=5, J=8)),
                                       ("h1", 24, dict(N=8, L=255, K=3, J=5))])
def test_bounds_hetero_grouped(base, n, kw, mode):
    prob = problem(base, n, mode, mode == 1, "f32", 8400, **kw)
    label = f"bounds grouped {base} {kw} mode={prob['mode']}"
    print(f"[gpu] {label}", flush=True)
    ora = oracle.solve_grouped(prob, threads=16)
    for gpu in both(prob, jdob.solve_grouped):
        compare_grouped(prob, gpu, ora, label)


# Two to four GPU levels are tried one by one in the bound of the GPU energy,
# from five on it takes the frequency at which a second of work costs least:
# with neither kind of power (at the lowest level, at the highest) and with that
# frequency below and above the levels.
POWERS = [dict(), dict(gpu_p_static=0.0), dict(gpu_c=0.0), dict(gpu_p_static=1e-4), dict(gpu_p_static=1e4)]


@pytest.mark.parametrize("power", range(len(POWERS)))
@pytest.mark.parametrize("base,n,kw", [("p4a", 64, dict(N=10, L=16)), ("p4b", 64, dict(N=7, L=9)),
                                       ("c4b", 32, dict(N=40, L=22, K=8))])
def test_bounds_gpu_levels(base, n, kw, power):
    for J in (2, 3, 4, 5, 16):
        prob = problem(base, n, 0, J == 3, "f32", 8500 + J, J=J, **kw)
        for k, f in POWERS[power].items():
            prob[k] = float(prob[k] * f)
        label = f"bounds {base} {kw} J={J} {POWERS[power]}"
        print(f"[gpu] {label}", flush=True)
        ora = oracle.solve(prob, threads=16)
        for gpu in both(prob, jdob.solve_batch) + both(prob, joint):
            compare(prob, gpu, ora, label=label)


# the shortest rows of an instance, whose preparation keeps values in the room of the batch records
@pytest.mark.parametrize("J", [2, 16, 32, 64])
def test_bounds_few_users(J):
    for N in (1, 2, 3, 5, 9, 12):
        for mode, dtype in ((0, "f32"), (0, "f64"), (1, "f32"), (8, "f32")):
            prob = problem("c2b", 96, mode, False, dtype, 8600 + N, N=N, L=6, K=8, J=J)
            label = f"bounds few users N={N} J={J} mode={prob['mode']} {dtype}"
            print(f"[gpu] {label}", flush=True)
            ora = oracle.solve(prob, threads=16)
            for gpu in both(prob, jdob.solve_batch) + both(prob, joint):
                compare(prob, gpu, ora, label=label)


# one to four partition points, searched as they come where they are few, with
# counting passes, and by bounds where they or their passes are many
@pytest.mark.parametrize("mode", [0, 1, 4, 8])
@pytest.mark.parametrize("L", [1, 2, 3, 4])
def test_bounds_grouped_over_few_partition_points(L, mode):
    for n, N, J, dtype in ((48, 2, 1, "f32"), (48, 7, 9, "f32"), (32, 6, 33, "f64"), (16, 20, 70, "f32")):
        prob = problem("g20" if mode != 8 else "p5", n, mode, N == 7, dtype, 8700 + N, N=N, L=L, K=2 if mode == 8 else 8, J=J)
        label = f"bounds grouped N={N} L={L} J={J} mode={prob['mode']} {dtype}"
        print(f"[gpu] {label}", flush=True)
        ora = oracle.solve_grouped(prob, threads=16)
        for gpu in both(prob, jdob.solve_grouped):
            compare_grouped(prob, gpu, ora, label)
