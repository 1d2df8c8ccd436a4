"""GPU parity of the preparation (checks, ranks, tie ranks) with the CPU oracle at
the sizes where it changes: one, four and sixteen waves an instance, sort buffers in
LDS and in the workspace (with tie keys they are larger), key and tie-key ranges of one
and several radix passes, requests that all arrive at step 0 or later, and an invalid
request in any wave's share."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_2508_14544_amd import workloads as W
from test_gpu_parity import assert_parity, gpu_run, oracle_run
from test_gpu_wave_edges import make

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


@pytest.mark.parametrize("algo", POLICIES)
@pytest.mark.parametrize("n,count", [(64, 3), (65, 3), (256, 2), (300, 600), (4096, 2), (4097, 2), (6100, 1),
                                     (12200, 1), (12300, 1), (18500, 1)])
def test_sizes(B, n, count, algo):
    few = n > 4000  # lengths that keep the simulation of a large instance short
    b = make(400 if few else 900, n, count, n, o=(1, 6) if few else (1, 400), lower="all" if few else "half",
             arrive=0 if n % 2 else 50)
    ks = range(min(count, 40))
    assert_parity(b, gpu_run(B, b, algo), oracle_run(b, algo, instances=ks), instances=ks)
    r = np.random.default_rng(n)
    for ties in (r.permutation(b.total_requests), r.integers(-2, 3, b.total_requests),
                 r.integers(-2**31, 2**31, b.total_requests)):
        t = dataclasses.replace(b, tie_key=ties.astype(np.int32))
        assert_parity(t, gpu_run(B, t, algo), oracle_run(t, algo, instances=ks), instances=ks)


@pytest.mark.parametrize("algo", POLICIES)
@pytest.mark.parametrize("n", [200, 1000, 5000])
def test_invalid_request_anywhere(B, n, algo):
    at = [0, 63, 64, n // 2, n - 1]
    good = make(400, n, len(at) + 1, n, o=(1, 6), lower="all")
    for field, value, status in (("output", 0, O.E_INTERVAL), ("prompt", 400, O.E_TOO_BIG), ("arrival", -1, O.E_ARRIVAL)):
        v = np.array(getattr(good, field) if getattr(good, field) is not None else np.zeros(good.total_requests), np.int32)
        for k, i in enumerate(at):
            v[k * n + i] = value
        b = dataclasses.replace(good, **{field: v})
        g = gpu_run(B, b, algo)
        assert g["status"].tolist() == [status] * len(at) + [0]
        assert_parity(b, g, oracle_run(b, algo))
