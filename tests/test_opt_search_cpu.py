"""The plain model of the one-wave search against the oracle's independent one."""
import pytest

from opt_search import one_wave_search
from oracle import oracle as O
from paper_2508_14544_amd import workloads as W


@pytest.mark.parametrize("seed,arrivals", [(1, False), (2, True)])
def test_one_wave_search(seed, arrivals):
    b = W.random_small(seed, 12, 5, s_max=3, o_max=5, M=12, arrivals=arrivals)
    for k in range(b.num_instances):
        best, nodes, ended = one_wave_search(b.instance(k), b.M, 1 << 20)
        assert ended and best == O.opt_tel(b.instance(k), b.M)
        cut, tested, done = one_wave_search(b.instance(k), b.M, nodes - 1)
        assert cut >= best and not done and tested >= nodes - 1
    late = {"arrival": [0, 0, 0, 70], "prompt": [2, 1, 3, 0], "output": [4, 5, 3, 4]}
    assert one_wave_search(late, 9, 1 << 20)[0] == O.opt_tel(late, 9)
