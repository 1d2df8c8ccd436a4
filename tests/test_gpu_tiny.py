"""GPU parity of the kernel that gives every tiny instance a lane (64 instances to
a wave; batches of instances of at most two requests, and large ones of at most
eight, how large being a matter of the policy) with the CPU oracle, at its edges: instances of 0 to 8 requests in one
wave, batches that do not fill a wave, invalid instances among valid ones,
arrivals, tie keys, step caps, long runs, and the wave-per-instance kernels on the
same batch (an option that only they read selects them)."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_14544_amd import workloads as W
from test_gpu_parity import assert_parity, gpu_run, oracle_run

pytestmark = pytest.mark.gpu

POLICIES = [O.AMAX, O.AMIN, O.HSF, O.AELL, O.ADAPTIVE, O.ARANDOM]
# an LDS limit far above what a small instance's cancelled set can reach
WAVE = dict(evicted_lds_limit=4096)
# more instances than twelve rounds of 16 waves on each of 256 CUs, from which on every
# policy gives them a lane each, and the rounds from which some do; no multiples of 64
MANY = 12 * 16 * 256 + 37
LINES = {1: (3,), 2: (3,), 3: (5,), 4: (5,), 5: (5, 6), 6: (5, 8), 7: (5, 8, 12), 8: (5, 6, 8, 12)}


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_14544_amd import binding
    binding.load_library()
    return binding


def batch_of(n_max, count, seed, *, o_max=9, s_max=7, M=40, arrivals=True):
    b = W.random_small(seed, count, n_max, s_max=s_max, o_max=o_max, M=M, arrivals=arrivals)
    return W.with_random_order(b, seed)


def many_of(b, count=MANY):
    """`count` instances, those of b over and over."""
    K, reps = b.num_instances, count // b.num_instances + 1
    cat = lambda v: None if v is None else np.tile(v, reps)
    sizes = np.tile(np.diff(b.offsets), reps)[:count]
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    cut = lambda v: None if v is None else np.ascontiguousarray(cat(v)[:offs[-1]])
    return dataclasses.replace(b, offsets=offs, instance_ids=np.arange(count) % K,
                               **{f: cut(getattr(b, f)) for f in ("arrival", "prompt", "output", "lower", "upper",
                                                                  "priority", "tie_key")})


@pytest.mark.parametrize("algo", POLICIES)
@pytest.mark.parametrize("n_max", [1, 2, 3, 8])
def test_sizes_and_partial_waves(B, algo, n_max):
    for count in (1, 63, 64, 65) if n_max <= 2 else (MANY,):
        b = batch_of(n_max, min(count, 700), 10 * n_max + count, arrivals=count != 64)
        b = many_of(b, count) if count == MANY else b
        g = gpu_run(B, b, algo)
        assert_parity(b, g, oracle_run(b, algo))
        w = gpu_run(B, b, algo, **WAVE)
        assert all(np.array_equal(g[f], w[f]) for f in g if g[f] is not None)


@pytest.mark.parametrize("algo", POLICIES)
@pytest.mark.parametrize("n_max", sorted(LINES))
def test_both_sides_of_the_lines(B, algo, n_max):
    few = W.random_small(n_max, 500, n_max, s_max=7, o_max=9, M=40, arrivals=True)
    few = W.with_random_order(few, n_max)
    ref = oracle_run(few, algo)
    for rounds in LINES[n_max]:
        for count in (rounds * 16 * 256, rounds * 16 * 256 + 1):
            b = many_of(few, count)
            assert b.max_requests == n_max
            g = gpu_run(B, b, algo, no_alloc=count % 2 == 0)
            at = np.arange(count) % few.num_instances
            for f in ("status", "tel", "makespan", "request_steps", "total_evictions"):
                assert np.array_equal(g[f], ref[f][at]), f
            for f in ("completion", "evictions"):
                assert np.array_equal(g[f], np.resize(ref[f], b.total_requests)), f


@pytest.mark.parametrize("algo", POLICIES)
def test_tie_keys_caps_and_no_allocation(B, algo):
    b = W.with_tie_keys(batch_of(8, 150, 77, o_max=4), 5)
    b = many_of(dataclasses.replace(b, tie_key=(b.tie_key // 3 - 2).astype(np.int32)))   # repeated and negative
    assert_parity(b, gpu_run(B, b, algo), oracle_run(b, algo))
    for cap in (1, 3, 8):
        g, ref = gpu_run(B, b, algo, step_cap=cap, no_alloc=True), oracle_run(b, algo, step_cap=cap)
        assert_parity(b, g, ref)
    assert (g["status"] == O.E_STEP_CAP).any()


@pytest.mark.parametrize("algo", POLICIES)
def test_statuses_among_valid_instances(B, algo):
    ok = {"arrival": [0, 1, 4], "prompt": [2, 0, 3], "output": [3, 2, 5], "lower": [1, 2, 4], "upper": [4, 3, 8],
          "priority": [2, 0, 1]}
    bad = [dict(ok, arrival=[2, 1, 4]), dict(ok, output=[0, 2, 5]), dict(ok, prompt=[-1, 0, 3]),
           dict(ok, prompt=[30, 0, 3]), dict(ok, lower=[1, 3, 4]), dict(ok, upper=[4, 1, 8]),
           dict(ok, priority=[1 << 15, 0, 1]), {f: [] for f in ok}]
    b = many_of(W.from_lists(24, [x for y in bad for x in (y, ok)], name="tiny_statuses"))
    g, w = gpu_run(B, b, algo), gpu_run(B, b, algo, **WAVE)
    assert all(np.array_equal(g[f], w[f]) for f in g if g[f] is not None)
    ok_at = list(range(1, 161, 2))
    assert (g["status"][ok_at] == 0).all() and (g["status"] != 0).any()
    assert_parity(b, g, oracle_run(b, algo, instances=ok_at), instances=ok_at)


@pytest.mark.parametrize("algo", POLICIES)
def test_long_runs_and_late_arrivals(B, algo):
    # steps far apart: runs of up to 2^15 - 1 steps, arrivals up to 2^28, memory near 2^30
    rng = np.random.default_rng(3)
    insts = []
    for _ in range(70):
        n = int(rng.integers(1, 9))
        o = rng.integers(1, 1 << 14, n)
        l, u = np.maximum(1, (o * rng.random(n)).astype(np.int64)), o + rng.integers(0, 1 << 14, n)
        insts.append({"arrival": np.sort(rng.integers(0, 1 << 28, n)) // (1 if rng.random() < 0.5 else 1 << 16),
                      "prompt": rng.integers(0, 60000, n), "output": o, "lower": l, "upper": u,
                      "priority": rng.permutation(n)})
    for M in (100000, (1 << 30) - 1):
        few = W.from_lists(M, insts, name="tiny_long")
        b = many_of(few)
        g, ref = gpu_run(B, b, algo), oracle_run(few, algo)
        assert_parity(few, {f: None if v is None else v[:len(ref["completion"])] for f, v in g.items()}, ref)
        w = gpu_run(B, b, algo, **WAVE)
        assert all(np.array_equal(g[f], w[f]) for f in g if g[f] is not None)
