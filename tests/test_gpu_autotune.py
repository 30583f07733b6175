"""The autotuner times the library's own default shape too, so that tuning cannot settle for less."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
G53 = 5.0 / 3.0


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n,physics", [((64, 64), "euler"), ((512, 512), "euler"),
                                       ((32, 32, 32), "mhd")])
def test_default_is_a_candidate(torch_cuda, n, physics):
    from paper_1305_5536_amd.autotune import DEFAULT_CANDIDATES, autotune
    from paper_1305_5536_amd.solver import Solver, cartesian
    lo, hi = (0.0,) * len(n), (1.0,) * len(n)
    s = Solver(cartesian(n, lo, hi), physics=physics, gamma=G53)
    U = s.to_device(W.random_p1_state(n, lo, hi, G53, seed=15, amp=0.2, mhd=physics == "mhd"))
    own = s.tiling
    s.tiling = 3
    e = autotune(s, U, n, reps=3, use_cache=False)
    assert str(own) in e["times"] and s.tiling == e["rows"]
    assert e["times"][str(e["rows"])] == min(e["times"].values())
    e = autotune(s, U, n, candidates=(2, 4), reps=1, use_cache=False)
    assert set(e["times"]) == {"2", "4"} and 1 in DEFAULT_CANDIDATES


@pytest.mark.parametrize("sizes", [[(64, 64), (96, 128), (130, 40)],
                                   [(64 + 19 * i, 64 + 19 * i) for i in range(24)]])
def test_batch_default_is_a_candidate(torch_cuda, sizes):
    from paper_1305_5536_amd.autotune import autotune_batch
    from paper_1305_5536_amd.solver import Solver, batch
    s = Solver(batch(sizes), precision="fp32", gamma=G53)
    U = s.pack([W.random_p1_state(n, (0.0, 0.0), (1.0, 1.0), G53, seed=31 + i, amp=0.2)
                for i, n in enumerate(sizes)])
    own = s.tiling
    e = autotune_batch(s, U, sizes, reps=2, use_cache=False)
    assert f"{own},4,0" in e["times"]
    assert e["times"]["%d,%d,%d" % (e["rows"], e["wpb"], e["grid"])] <= e["times"][f"{own},4,0"]
    assert s.tiling == e["rows"] and s.launch == (e["wpb"], e["grid"])
