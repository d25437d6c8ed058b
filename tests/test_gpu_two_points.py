"""Forward pass with two points a thread (batches of two rounds of workgroups and more), where a store holds four or eight levels'
outputs: against the same points in batches that the kernel with one point a thread takes, and against the oracle; the counting
kernel's counts against those of the count pass."""
import pytest
import torch

from oracle import hashgrid_oracle as orc
from paper_2201_05989_amd import HashGrid
from test_gpu_parity import check_fwd, same_forward

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "f32": torch.float32}


def inputs(grid, B, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.rand(B, grid.d, device="cuda", generator=gen).clamp_(max=1 - 2.0 ** -24)
    theta = (torch.rand(grid.n_entries, grid.F, device="cuda", generator=gen) * 2 - 1).to(grid.param_dtype)
    return x, theta, gen


@pytest.mark.parametrize("count", [False, "always"])
@pytest.mark.parametrize("d,L,F,param,io", [
    (2, 8, 1, "f16", "f16"), (3, 16, 1, "f16", "f16"), (3, 16, 1, "f32", "f32"), (3, 4, 2, "f16", "f16"), (3, 16, 2, "f32", "f16"),
    (2, 12, 2, "f16", "f16")])
@pytest.mark.parametrize("B", [1 << 19, (1 << 19) + 2049])
def test_two_points_a_thread(d, L, F, param, io, B, count):
    grid = HashGrid(d, L, F, 1 << 14, 16, 512, param, io)
    x, theta, gen = inputs(grid, B, B + d)
    y = grid.encode_fwd(x, theta, count_for_bwd=count)
    counted = grid._counted is not None
    assert counted == bool(count)
    if counted:
        dy = torch.randn(B, L * F, device="cuda", generator=gen).to(DT[io])
        got = grid.encode_bwd(x, dy)
        want = grid.encode_bwd(x, dy, use_workspace=True)  # counts for itself
        mass = grid.encode_bwd(x, dy.abs(), use_workspace=True)
        # exact sums, each rounded where it is added; chunks with several workgroups add their parts in any order
        assert ((got - want).abs() <= 1e-5 * mass + 1e-30).all()
    step = 100_001
    same_forward(y, torch.cat([grid.encode_fwd(x[b:b + step].contiguous(), theta) for b in range(0, B, step)]), io)


@pytest.mark.parametrize("param,io", [("f16", "f16"), ("f32", "f32")])
def test_one_feature_two_points_against_the_oracle(param, io):
    grid = HashGrid(3, 16, 1, 1 << 16, 16, 1024, param, io)
    x, theta, _ = inputs(grid, 1 << 19, 1)
    for count in (False, "always"):
        y = grid.encode_fwd(x, theta, count_for_bwd=count).cpu().numpy()
        ref = orc.encode_fwd(orc.OracleConfig(3, 16, 1, 1 << 16, 16, 1024), x.cpu().numpy(), theta.cpu().numpy())
        check_fwd(y, ref, 1.0, io)


@pytest.mark.parametrize("d,param", [(2, "f16"), (2, "f32"), (3, "f16"), (3, "f32")])
def test_two_features_are_rounded_alike(d, param):
    """F = 2 in half precision: the sum is rounded to 32 bits and then to 16, plain and counting, at every level of a row."""
    grid = HashGrid(d, 16, 2, 1 << 16, 16, 1024, param, "f16")
    x, theta, _ = inputs(grid, 1 << 19, d)
    assert torch.equal(grid.encode_fwd(x, theta), grid.encode_fwd(x, theta, count_for_bwd="always"))
