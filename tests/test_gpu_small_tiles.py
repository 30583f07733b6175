"""Meshes small enough for one row (plane) per tile by default: the results must be those of any
other tiling, bit for bit, and the default must be that shortest tile.
"""
import numpy as np
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


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,physics", [((5, 1), "euler"), ((61, 7), "euler"), ((130, 33), "euler"),
                                       ((59, 2), "mhd"), ((61, 9), "mhd"), ((63, 5, 1), "mhd"),
                                       ((7, 6, 5), "mhd")])
def test_shortest_tiles_match_longer_ones(torch_cuda, n, physics, precision):
    torch = torch_cuda
    from paper_1305_5536_amd.solver import Solver, cartesian
    dim = len(n)
    lo, hi = (0.0,) * dim, (1.0,) * dim
    s = Solver(cartesian(n, lo, hi), physics=physics, precision=precision, gamma=G53)
    U = s.to_device(W.random_p1_state(n, lo, hi, G53, seed=31, amp=0.2, mhd=physics == "mhd"))
    dt = s.cfl_dt(U, 0.3)
    assert s.tiling == 1
    nxt = torch.empty_like(dt)
    a = s.step(U, dt, cfl=0.3, dt_next=nxt)
    s.check()
    for rows in (2, 3, 8):
        s.tiling = rows
        other = torch.empty_like(dt)
        assert torch.equal(a, s.step(U, dt, cfl=0.3, dt_next=other))
        assert torch.equal(nxt, other)
    s.tiling = 0
    assert s.tiling == 1


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_batch_tiles_follow_the_instances(torch_cuda, precision):
    """Few small instances get short tiles, and the results of the fixed tile of 16 rows; the
    adjoint of each instance equals that of the instance alone, whose tiles differ."""
    torch = torch_cuda
    from paper_1305_5536_amd.solver import Solver, batch, cartesian
    sizes = [(70, 41), (33, 64), (12, 5)]
    s = Solver(batch(sizes), precision=precision, gamma=G53)
    states = [W.random_p1_state(n, (0.0, 0.0), (1.0, 1.0), G53, seed=41 + i, amp=0.2)
              for i, n in enumerate(sizes)]
    U = s.pack(states)
    assert s.tiling == 1
    dt = s.cfl_dt(U, 0.3)
    V1 = s.stage1(U, dt, s.empty())
    lam = torch.as_tensor(np.random.default_rng(3).standard_normal(s.state_len)).to(U)
    adj = s.adjoint_step(U, dt, lam, V1=V1)
    for rows in (4, 16):
        s.tiling = rows
        assert torch.equal(V1, s.stage1(U, dt, s.empty()))
    A, L = (x.reshape(12, -1) for x in (adj, lam))
    for i, n in enumerate(sizes):
        one = Solver(cartesian(n, (0.0, 0.0), (1.0, 1.0)), precision=precision, gamma=G53)
        cut = slice(int(s.offsets[i]), int(s.offsets[i + 1]))
        got = one.adjoint_step(one.to_device(states[i]), dt[i:i + 1].clone(),
                               L[:, cut].contiguous().reshape(-1))
        assert torch.equal(got.reshape(12, -1), A[:, cut])


@pytest.mark.parametrize("shape,tol", [((1030, 517), 1e-14), ((2051, 300), 1e-14)])
def test_fused_step_of_a_large_mesh_matches_the_stage_pair(torch_cuda, shape, tol):
    """Ragged meshes of several rows per wave: the fused step equals the stage kernels to rounding
    (the compiler contracts some products of the row update differently)."""
    from paper_1305_5536_amd.solver import Solver, cartesian
    s = Solver(cartesian(shape, (0.0, 0.0), (1.0, 1.0)), precision="fp64", gamma=G53)
    U = s.to_device(W.random_p1_state(shape, (0.0, 0.0), (1.0, 1.0), G53, seed=9, amp=0.2))
    dt = s.cfl_dt(U, 0.3)
    a = s.step(U, dt).reshape(12, -1)
    V1 = s.stage1(U, dt, s.empty())
    b = s.stage2(U, V1, dt, s.empty()).reshape(12, -1)
    for k in range(12):
        assert (a[k] - b[k]).abs().max() <= tol * b[k].abs().max() * (1 if k % 3 == 0 else shape[0])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("limiter", [True, False])
@pytest.mark.parametrize("shape", [(5, 1), (55, 2), (57, 3), (3, 11), (56, 4), (130, 33),
                                   (113, 340), (113, 341), (113, 680), (113, 681)])
def test_fused_step_of_a_small_mesh_matches_the_stage_pair(torch_cuda, shape, limiter, precision):
    """A few rows (fewer than a workgroup's four, not a multiple of them), ragged strips, and both
    sides of the lines between row-waves and marching waves (256 workgroups, FP32 512): the fused step equals
    the stage kernels to rounding, and the step size it returns is the CFL step of its output.
    Bounds: 45 units of rounding of the largest value (slopes: per cell width)."""
    torch = torch_cuda
    from paper_1305_5536_amd.solver import Solver, cartesian
    tol = 45 * (2.0 ** -52 if precision == "fp64" else 2.0 ** -23)
    s = Solver(cartesian(shape, (0.0, 0.0), (1.0, 1.0)), precision=precision, gamma=G53,
               limiter=limiter)
    U = s.to_device(W.random_p1_state(shape, (0.0, 0.0), (1.0, 1.0), G53, seed=17, amp=0.1))
    dt = s.cfl_dt(U, 0.2)
    nxt = torch.empty_like(dt)
    out = torch.full_like(U, float("nan"))
    a = s.step(U, dt, cfl=0.2, dt_next=nxt, out=out).reshape(12, -1)
    s.check()
    b = s.stage2(U, s.stage1(U, dt, s.empty()), dt, s.empty()).reshape(12, -1)
    scale = b[0::3].abs().max()
    for k in range(12):
        assert (a[k] - b[k]).abs().max() <= tol * scale * (1 if k % 3 == 0 else max(shape))
    want = s.cfl_dt(out, 0.2)
    assert abs(float(nxt) - float(want)) <= tol * float(want)


@pytest.mark.parametrize("n,physics,precision,rows", [
    ((700, 500), "euler", "fp64", 6), ((400, 900), "euler", "fp64", 7),
    ((8, 4096), "euler", "fp64", 4), ((300, 300), "euler", "fp64", 2),
    ((2048, 2048), "euler", "fp64", 36), ((3182, 750), "euler", "fp32", 10),
    ((1000, 750), "euler", "fp32", 7), ((950, 281), "mhd", "fp32", 2),
    ((512, 512), "mhd", "fp64", 5)])
def test_default_rows(torch_cuda, n, physics, precision, rows):
    """Default rows on 256 CUs: the fastest of all rows, measured, on meshes that just fill the
    chip, where a round of waves more or less decides, and on small and large ones."""
    from paper_1305_5536_amd.solver import Solver, cartesian
    if torch_cuda.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("rows of another chip")
    s = Solver(cartesian(n, (0.0, 0.0), (1.0, 1.0)), physics=physics, precision=precision, gamma=G53)
    assert s.tiling == rows
    s.close()
