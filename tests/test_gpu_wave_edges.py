"""GPU parity of the one-wave engine with the CPU oracle where its step loop
branches: four admissions in one test or one by one (all four, three or fewer
left, a later one that does not fit), a planned end that is the latest, ties with
it and falls below it, more cancellations in a step and more cancelled requests
waiting than a register row holds, the cancelled set in LDS and in global memory,
arrivals between the steps of a jump, and step caps inside a jump or after the last
admission.  All outputs are whole numbers and have to be the same."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_14544_amd import workloads as W
from test_gpu_parity import assert_parity, gpu_run, oracle_run

pytestmark = pytest.mark.gpu

POLICIES = [O.AMAX, O.AMIN, O.HSF, O.AELL, O.ADAPTIVE, O.ARANDOM]


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_14544_amd import binding
    binding.load_library()
    return binding


def make(M, n, count, seed, *, s=(0, 4), o=(1, 12), lower="one", upper="slack", arrive=0):
    """`count` instances of n requests; lower bounds 1, a half or all of the output,
    upper bounds equal to it or above, arrivals over `arrive` steps."""
    r = np.random.default_rng(seed)
    insts = []
    for _ in range(count):
        out = r.integers(o[0], o[1] + 1, n)
        pr = r.integers(s[0], s[1] + 1, n)
        lo = {"one": np.ones(n, int), "half": (out + 1) // 2, "all": out}[lower]
        hi = out if upper == "tight" else out + r.integers(0, 5, n)
        insts.append({"arrival": np.sort(r.integers(0, arrive + 1, n)).tolist(), "prompt": pr.tolist(),
                      "output": out.tolist(), "lower": lo.tolist(), "upper": np.minimum(hi, M - pr).tolist()})
    return W.with_random_order(W.from_lists(M, insts, name=f"edge M={M} n={n} seed={seed}"), seed)


FAMILIES = {
    # one to five requests fit at a time
    "few_at_a_time": lambda: make(26, 40, 24, 1),
    "few_lower_half": lambda: make(30, 40, 24, 2, lower="half"),
    # planned lengths of two values, and of one: ends tie with the latest
    "ties": lambda: make(120, 70, 12, 3, o=(6, 7), lower="all", upper="tight"),
    "one_length": lambda: make(90, 70, 12, 4, s=(1, 1), o=(5, 5), lower="all", upper="tight"),
    # all start at once, and most are cancelled at the next step
    "mass_cancellation": lambda: make(330, 310, 6, 5, s=(0, 0), o=(3, 20)),
    "mass_cancellation_prompts": lambda: make(700, 400, 4, 6, s=(0, 2), o=(2, 40)),
    # full rows, more than one of them, and their free slots
    "rows": lambda: make(2000, 300, 6, 7, o=(1, 30), lower="half"),
    # arrivals in the middle of jumps over long runs, shorter and longer than the head
    "arrivals": lambda: make(160, 90, 10, 8, o=(1, 60), lower="half", arrive=150),
    "arrivals_tight": lambda: make(64, 60, 12, 9, o=(20, 40), lower="all", upper="tight", arrive=300),
}


@pytest.mark.parametrize("algo", POLICIES)
@pytest.mark.parametrize("family", sorted(FAMILIES))
def test_edges(B, family, algo):
    b = FAMILIES[family]()
    g = gpu_run(B, b, algo)
    assert_parity(b, g, oracle_run(b, algo))
    if family.startswith("mass") and algo == O.AMIN:
        assert (g["total_evictions"] > 300).all()
    # a cancelled set of 8 entries in LDS, the rest (then all of it) in global memory
    assert_parity(b, gpu_run(B, b, algo, evicted_lds_limit=8), oracle_run(b, algo))
    last = int(g["makespan"].max())
    for cap in sorted({1, 2, last // 3, last - 1}):
        if cap > 0:
            assert_parity(b, gpu_run(B, b, algo, step_cap=cap), oracle_run(b, algo, step_cap=cap))
