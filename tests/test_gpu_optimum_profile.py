"""GPU parity of the hindsight optimum's two searches at the line between them: a
memory profile of 64 steps where the horizon (max a + sum(o + 1) + 1) plus the
longest output is at most 63, the placed runs' tests above.  Against the oracle's
independent search and a plain model of the one-wave one, with late arrivals, runs
that fill the profile, identical requests, and instances of both kinds that the first
launch ends and that it leaves to the second."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_14544_amd import workloads as W
from opt_search import one_wave_search
from test_gpu_optimum import B, gpu_opt  # noqa: F401  (B: the module's fixture)
from test_oracle_pins import spt_single_machine_tel

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


def late_instances(count, late, seed, least, most, n=7, o=(1, 6)):
    """Instances of n requests, the last one at step `late` and the others at step 0,
    that the one-wave search ends after `least` to `most` start steps, with their
    optimum and that number."""
    rng = np.random.default_rng(seed)
    found = []
    while len(found) < count:
        inst = {"arrival": [0] * (n - 1) + [late], "prompt": rng.integers(0, 4, n).tolist(),
                "output": rng.integers(o[0], o[1] + 1, n).tolist()}
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


@pytest.mark.parametrize("late", [300, 2000, 1 << 20])
def test_late_arrivals_in_the_second_launch(B, late):  # noqa: F811
    # beyond the profile and the first budget: what the waves go through to find their
    # pieces is a matter of the bound, not of the horizon, so the nodes stay within a
    # few of the one-wave search's for each of the device's waves
    import torch
    found = late_instances(3, late, 4, 1 << 17, 1 << 20, n=8, o=(2, 6))
    b = W.from_lists(12, [i for i, _, _ in found], name="opt_late_pool")
    r = gpu_opt(B, b)
    assert (r["status"] == 0).all()
    assert r["tel"].tolist() == [t for _, t, _ in found]
    assert (r["nodes"] > 1 << 17).all()
    waves = 32 * torch.cuda.get_device_properties(0).multi_processor_count
    assert (r["nodes"] < [4 * c + 100 * waves for _, _, c in found]).all()


def test_long_runs_in_the_second_launch(B):  # noqa: F811
    # two requests (pieces are starts of the first one), three and four, one at a time
    outs = [[900, 700], [600, 611], [300, 200, 250], [150, 150, 150], [60, 50, 40, 30]]
    insts = [{"prompt": [1000] * len(o), "output": o} for o in outs]
    assert all(one_wave_search(i, 1999, 1 << 17)[2] is False for i in insts)
    r = gpu_opt(B, W.from_lists(1999, insts, name="opt_long_pool"))
    assert (r["status"] == 0).all()
    assert r["tel"].tolist() == [spt_single_machine_tel(o) for o in outs]
    # a budget that the walk over the pieces uses up ends the search, with a bound
    o = [30000, 30000, 30000]
    r = gpu_opt(B, W.from_lists(1 << 16, [{"prompt": [1 << 15] * 3, "output": o}], name="opt_long_cap"),
                node_cap=(1 << 17) + 64)
    assert r["status"].tolist() == [O.E_STEP_CAP] and r["tel"][0] >= spt_single_machine_tel(o)


def test_both_searches_in_the_second_launch(B):  # noqa: F811
    # a batch with instances of both kinds beyond their first budgets
    rng = np.random.default_rng(8)
    found = []
    while len(found) < 6:
        i = {"arrival": [0] * 7, "prompt": rng.integers(1, 4, 7).tolist(), "output": rng.integers(4, 7, 7).tolist()}
        best, nodes, ended = one_wave_search(i, 12, 1 << 20)
        if ended and nodes > 1 << 13 and sum(i["output"]) + 7 + 1 + max(i["output"]) < 64:
            found.append((i, best, 1 << 12))
    found += [(i, t, 1 << 17) for i, t, _ in late_instances(4, 500, 9, 1 << 17, 1 << 20, n=8, o=(2, 6))]
    found = [found[k] for k in rng.permutation(len(found))]
    b = W.from_lists(12, [i for i, _, _ in found], name="opt_mixed")
    r = gpu_opt(B, b)
    assert (r["status"] == 0).all()
    assert r["tel"].tolist() == [t for _, t, _ in found]
    assert (r["nodes"] > [c for _, _, c in found]).all()
    assert (r["tel"] <= O.simulate_batch(b, O.HSF)["tel"]).all()
