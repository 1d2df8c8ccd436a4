"""GPU parity of the hindsight optimum's two searches at the line between them: a
memory profile of 64 steps where the horizon (max a + sum(o + 1) + 1) plus the
longest output is at most 63, the placed runs' tests above.  Against the oracle's
independent search, with late arrivals, runs that fill the profile, identical
requests, and both kinds in one batch under a budget that leaves some of them to
the second launch."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_14544_amd import workloads as W
from opt_search import one_wave_search
from test_gpu_optimum import B, gpu_opt  # noqa: F401  (B: the module's fixture)

pytestmark = pytest.mark.gpu


def reaching(steps, n, rng, M=14):
    """A random instance of n requests whose horizon plus longest output is `steps`."""
    while True:
        o = rng.integers(1, 9, n)
        if rng.random() < 0.3:
            o[:] = o[0]
        s = rng.integers(0, 4, n)
        late = steps - int((o + 1).sum()) - 1 - int(o.max())
        if late >= 0:
            a = np.sort(rng.integers(0, min(late, 4) + 1, n))
            a[-1] = late
            return {"arrival": a.tolist(), "prompt": np.minimum(s, M - o).tolist(), "output": o.tolist()}


@pytest.mark.parametrize("steps", [62, 63, 64, 65])
def test_edge_of_the_profile(B, steps):  # noqa: F811
    rng = np.random.default_rng(steps)
    b = W.from_lists(14, [reaching(steps, n, rng) for n in (1, 2, 3, 4, 4, 5, 5)] * 2, name=f"opt_reach{steps}")
    r = gpu_opt(B, b)
    assert (r["status"] == 0).all()
    assert r["tel"].tolist() == [O.opt_tel(b.instance(k), b.M) for k in range(b.num_instances)]


def test_one_long_run_fills_the_profile(B):  # noqa: F811
    # o = 30: horizon 32, 62 steps; o = 31: 64
    insts = [{"prompt": [2], "output": [o]} for o in (29, 30, 31, 32)]
    insts += [{"prompt": [1, 1], "output": [o, 1]} for o in (28, 29, 30)]
    b = W.from_lists(34, insts, name="opt_long_run")
    r = gpu_opt(B, b)
    assert (r["status"] == 0).all()
    assert r["tel"].tolist() == [O.opt_tel(b.instance(k), b.M) for k in range(b.num_instances)]


def test_both_searches_in_the_second_launch(B):  # noqa: F811
    # the same eight requests with and without a late ninth step count: the
    # optimum of a batch that mixes both searches equals the one-instance calls'
    rng = np.random.default_rng(8)
    insts = []
    for _ in range(6):
        o = rng.integers(4, 7, 7)
        insts.append({"arrival": [0] * 7, "prompt": rng.integers(1, 4, 7).tolist(), "output": o.tolist()})
        insts.append(dict(insts[-1], arrival=[0] * 6 + [40]))
    b = W.from_lists(12, insts, name="opt_mixed")
    steps = [max(i["arrival"]) + sum(i["output"]) + 7 + 1 + max(i["output"]) for i in insts]
    assert min(steps) <= 63 < max(steps)
    r = gpu_opt(B, b)
    assert (r["status"] == 0).all()
    assert (r["nodes"] > 1 << 12).any()      # beyond the first launch's budget of so small a batch
    one = [gpu_opt(B, W.from_lists(12, [i], name="opt_one")) for i in insts]
    assert r["tel"].tolist() == [int(x["tel"][0]) for x in one]
    hsf = O.simulate_batch(b, O.HSF)["tel"]
    assert (r["tel"] <= hsf).all()


def late_instances(count, late, seed, least, most):
    """Instances of seven requests, six at step 0 and one at step `late`, that the
    one-wave search ends after `least` to `most` start steps, with their optimum and
    that number."""
    rng = np.random.default_rng(seed)
    found = []
    while len(found) < count:
        inst = {"arrival": [0] * 6 + [late], "prompt": rng.integers(0, 4, 7).tolist(),
                "output": rng.integers(1, 7, 7).tolist()}
        best, nodes, ended = one_wave_search(inst, 12, most)
        if ended and nodes > least:
            found.append((inst, best, nodes))
    return found


def test_late_arrivals_end_in_the_first_launch(B):  # noqa: F811
    # beyond the profile a small batch has the whole first budget: every start step
    # is one of the one-wave search's, also where node_cap allows few more.  (The
    # six alone are over before the seventh comes, so the optima add up.)
    found = late_instances(20, 300, 3, 1 << 12, 1 << 17)
    b = W.from_lists(12, [i for i, _, _ in found], name="opt_late")
    for cap in (0, (1 << 17) + 1):
        r = gpu_opt(B, b, node_cap=cap)
        assert (r["status"] == 0).all()
        assert r["tel"].tolist() == [t for _, t, _ in found]
        assert r["nodes"].tolist() == [c for _, _, c in found]
    for inst, t, _ in found[:3]:
        six = {f: inst[f][:6] for f in inst}
        assert t == O.opt_tel(six, 12) + inst["output"][6]
