"""Forward pass that counts for the sorted backward pass, on points whose pairs of corners straddle two chunks at the finest levels
(lanes without a record): the outputs are those of the plain forward, and a backward pass over its counts gives the gradient of one
that counts for itself."""
import pytest
import torch

from paper_2201_05989_amd import HashGrid

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "f32": torch.float32}


@pytest.mark.parametrize("B", [1 << 18, 1 << 19])  # one point a thread and two
@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("d,L,F,T,param,io", [
    (3, 8, 8, 1 << 17, "f32", "f32"), (3, 8, 8, 1 << 17, "f32", "f16"), (3, 4, 4, 1 << 17, "f32", "f16"), (3, 8, 2, 1 << 16, "f32", "f16"),
    (3, 8, 2, 1 << 16, "f16", "f16"), (3, 8, 1, 1 << 16, "f16", "f32"), (2, 8, 8, 1 << 15, "f16", "f32"),
    (3, 8, 8, 1 << 19, "f16", "f16")])  # the last: 64 KiB of histograms at two points a thread
def test_points_without_records(d, L, F, T, param, io, interp, B):
    N = 1 << 13
    grid = HashGrid(d, L, F, T, 16 if T < 1 << 19 else 128, N, param, io, interp)
    gen = torch.Generator(device="cuda").manual_seed(B + F)
    x = torch.rand(B, d, device="cuda", generator=gen)
    k = torch.randint(1, 5, (B // 2,), device="cuda", generator=gen) * (N // 4) - 1  # the last voxel of a chunk at F = 8
    x[::2, 0] = (k + torch.rand(B // 2, device="cuda", generator=gen) * 0.9 - (0.5 if interp else 0.0)) / N
    x = x.clamp_(max=1 - 2.0 ** -24)
    theta = (torch.rand(grid.n_entries, F, device="cuda", generator=gen) * 2 - 1).to(DT[param])
    plain = grid.encode_fwd(x, theta)
    counting = grid.encode_fwd(x, theta, count_for_bwd="always")
    assert grid._counted is not None
    if io == "f32":
        assert torch.equal(counting, plain)  # the same sums in the same order
    else:  # rounded once or twice where an output is a tie: one unit in the last place, one output in 10^4
        off = (counting.float() - plain.float()).abs()
        assert (off <= 2.0 ** -10 * plain.float().abs() + 2.0 ** -24).all() and (off > 0).sum() <= off.numel() // 10000
    dy = torch.randn(B, L * F, device="cuda", generator=gen).to(DT[io])
    got = grid.encode_bwd(x, dy)
    want = grid.encode_bwd(x, dy, use_workspace=True)
    mass = grid.encode_bwd(x, dy.abs(), use_workspace=True)
    # exact sums; each is rounded where it is added, and chunks with several workgroups and straddling pairs add their parts in any order
    assert ((got - want).abs() <= 1e-5 * mass + 1e-30).all()
