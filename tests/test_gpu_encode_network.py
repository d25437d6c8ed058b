"""The encoding with the network behind it, at the sizes where its kernels change: batches below and above what the split
kernel takes (32768 to 100000 points, by d, the number of levels and the size of the tables), paced and free-running
workgroups (d = 3 or 2, narrow or wide entries, tables within or beyond an L2), points in raster and in random order, one to
four levels a wave, level counts below and beside what the unconditional loop over levels takes, ragged last blocks.

The fused output must equal the network alone on the features the call keeps, bit for bit (the same instructions on the
same halves), and the kept features are the encoding's (one rounding to half; ties may fall either way: 2^-10 of the
value).  The gradient with respect to the position is held to the three calls it stands for, each of which is held to the
oracle in a module of its own: bit for bit, with random tables and weights too (the same products, summed and rounded in the same
order)."""
import pytest
import torch

from paper_2201_05989_amd import HashGrid, mlp_bwd, mlp_fwd

pytestmark = pytest.mark.gpu


def network(n_in, n_out, gen, integers):
    shapes = ((64, n_in), (64, 64), (n_out, 64))
    if not integers:
        return [torch.randn(s, device="cuda", generator=gen).mul_(0.2).half() for s in shapes]
    return [(torch.randint(-1, 2, s, device="cuda", generator=gen) * (torch.rand(s, device="cuda", generator=gen) < 0.2)).half()
            for s in shapes]


@pytest.mark.parametrize("d,L,F,T,N_max,n_out,B,order,interp", [
    (3, 16, 2, 1 << 19, 2048, 3, 1, "random", 0),
    (3, 16, 2, 1 << 19, 2048, 3, 32768, "random", 0),      # split at the last batch it takes, here and in the next pairs
    (3, 16, 2, 1 << 19, 2048, 3, 32769, "random", 0),      # paced, workgroups of two waves
    (3, 16, 4, 1 << 12, 256, 3, 50000, "rays", 0),
    (3, 16, 4, 1 << 12, 256, 3, 50001, "random", 0),       # free-running, 64 features
    (2, 16, 2, 1 << 18, 4096, 3, 70000, "random", 0),
    (2, 16, 2, 1 << 18, 4096, 3, 70001, "random", 0),      # paced by the order of the points, and free-running below
    (3, 8, 4, 1 << 19, 2048, 3, 40000, "random", 0),
    (3, 8, 4, 1 << 19, 2048, 3, 40001, "random", 0),
    (2, 16, 1, 1 << 12, 1024, 3, 100000, "raster", 0),
    (2, 16, 1, 1 << 12, 1024, 3, 100001, "raster", 0),     # free-running, two workgroups a compute unit
    (2, 8, 8, 1 << 12, 1024, 3, 100001, "random", 0),      # one workgroup of half the size, paced
    (2, 4, 2, 1 << 12, 64, 1, 120000, "raster", 0),        # fewer levels than the loop that looks three ahead takes
    (2, 20, 2, 1 << 12, 300, 1, 150001, "raster", 0),
    (3, 4, 2, 1 << 12, 64, 1, 60000, "random", 0),
    (3, 12, 2, 1 << 12, 64, 1, 60000, "random", 1),
    (3, 16, 2, 1 << 19, 2048, 3, 39999, "random", 0),
    (3, 16, 2, 1 << 19, 2048, 4, 40001, "random", 0),      # paced, workgroups of a few waves
    (3, 16, 2, 1 << 14, 512, 1, 300007, "random", 1),      # paced, full workgroups, several blocks each
    (3, 16, 4, 1 << 14, 512, 17, 100001, "random", 0),     # free-running, 64 features
    (3, 8, 8, 1 << 18, 512, 32, 70001, "random", 0),       # paced, eight features an entry, 64 features
    (3, 32, 1, 1 << 12, 256, 2, 70003, "random", 0),       # split, four levels a wave
    (3, 32, 2, 1 << 12, 256, 2, 5, "random", 0),
    (2, 16, 2, 1 << 18, 4096, 3, 100000, "raster", 0),
    (2, 16, 2, 1 << 18, 4096, 3, 262145, "raster", 0),     # free-running
    (2, 16, 2, 1 << 18, 4096, 16, 262145, "random", 1),    # paced by the order of the points
    (2, 12, 2, 1 << 14, 300, 4, 150001, "raster", 1),      # 24 features: a ragged operand
    (2, 8, 8, 1 << 14, 300, 9, 130001, "raster", 0),
    (2, 8, 1, 1 << 10, 64, 1, 110001, "random", 0),        # eight features in all
])
def test_fused_output_is_the_network_on_the_kept_features(d, L, F, T, N_max, n_out, B, order, interp):
    gen = torch.Generator(device="cuda").manual_seed(B)
    grid = HashGrid(d, L, F, T, 16, N_max, "f16", "f16", interp)
    theta = torch.randn((grid.n_entries, F), device="cuda", generator=gen).half()
    x = torch.rand((B, d), device="cuda", generator=gen)
    if order == "raster":
        i = torch.arange(B, device="cuda")
        x = torch.stack([(i % 640) / 640.0, (i // 640) / (B // 640 + 1.0)], dim=1).contiguous()
    elif order == "rays":
        x = (x[:1] + torch.arange(B, device="cuda")[:, None] / B * (x[1:2] - x[:1])).contiguous()
    W = network(L * F, n_out, gen, False)
    y = torch.full((B, L * F), float("nan"), dtype=torch.float16, device="cuda")
    out = grid.encode_mlp_fwd(x, theta, *W, torch.full((B, n_out), float("nan"), device="cuda"), y=y)
    assert torch.equal(out, mlp_fwd(y, *W))
    assert torch.equal(out, grid.encode_mlp_fwd(x, theta, *W))
    ref = grid.encode_fwd(x, theta).float()
    assert ((y.float() - ref).abs() <= 2.0 ** -10 * ref.abs() + 1e-7).all()


@pytest.mark.parametrize("d,L,F,T,n_out,B,interp", [(3, 8, 2, 1 << 14, 1, 1, 0), (3, 8, 4, 1 << 14, 1, 65, 0), (2, 8, 8, 1 << 12, 3, 1000, 0),
                                                    (3, 7, 8, 1 << 14, 32, 777, 0), (2, 12, 2, 1 << 20, 17, 40001, 0),
                                                    (3, 16, 1, 1 << 12, 9, 3001, 1), (2, 24, 1, 1 << 12, 2, 130, 0)])
def test_position_gradient_equals_the_three_calls_where_nothing_rounds(d, L, F, T, n_out, B, interp):
    gen = torch.Generator(device="cuda").manual_seed(100 + B)
    grid = HashGrid(d, L, F, T, 4, 4 << (min(L, 12) - 1), "f16", "f16", interp)
    exact = all(l.N & (l.N - 1) == 0 for l in grid.levels())  # else fractional positions round: compared with a tolerance
    theta = torch.randint(-1, 2, (grid.n_entries, F), device="cuda", generator=gen).half()
    x = ((2 * torch.randint(0, 4, (B, d), device="cuda", generator=gen) + 1).float() / 8).contiguous()
    W = network(L * F, n_out, gen, True)
    for dout in (None, torch.randint(-4, 5, (B, n_out), device="cuda", generator=gen) / 4.0):
        y = torch.empty((B, L * F), dtype=torch.float16, device="cuda")
        dy = torch.empty_like(y)
        grid.encode_mlp_fwd(x, theta, *W, y=y)
        dW = [torch.zeros(w.shape, device="cuda") for w in W]
        mlp_bwd(y, *W, torch.ones((B, n_out), device="cuda") if dout is None else dout, dy, *dW)
        want = grid.encode_bwd_input(x, theta, dy)
        got = grid.encode_mlp_bwd_input(x, theta, *W, dout, torch.full((B, d), float("nan"), device="cuda"))
        assert B == 1 or want.abs().max() > 1
        if exact:
            assert torch.equal(got, want)
        else:  # fp32 sums over the levels in two orders; a half that rounds the other way moves the sum by 2^-11 of a level
            assert ((got - want).abs() <= 2.0 ** -9 * want.abs().max()).all()


@pytest.mark.parametrize("d,L,F,T,n_out,B,interp", [(3, 8, 4, 1 << 15, 1, 30001, 1), (3, 16, 2, 1 << 19, 4, 20000, 0), (2, 8, 1, 1 << 12, 8, 777, 0),
                                                    (3, 12, 2, 1 << 14, 17, 5001, 0), (3, 32, 2, 1 << 12, 32, 3001, 0), (2, 8, 8, 1 << 14, 9, 5000, 1),
                                                    (3, 16, 4, 1 << 14, 16, 2049, 0), (2, 24, 1, 1 << 12, 2, 130, 0),
                                                    (3, 8, 8, 1 << 17, 1, 40001, 0), (2, 16, 4, 1 << 14, 1, 30001, 0), (2, 16, 2, 1 << 17, 3, 30001, 1),
                                                    (2, 32, 2, 1 << 12, 1, 30001, 0), (3, 16, 1, 1 << 14, 1, 30001, 0), (2, 8, 4, 1 << 14, 4, 30001, 1)])
def test_position_gradient_has_the_bits_of_the_three_calls(d, L, F, T, n_out, B, interp):
    gen = torch.Generator(device="cuda").manual_seed(200 + B)
    grid = HashGrid(d, L, F, T, 16, 512, "f16", "f16", interp)
    theta = torch.randn((grid.n_entries, F), device="cuda", generator=gen).mul_(0.5).half()
    x = torch.rand((B, d), device="cuda", generator=gen).clamp_(max=1 - 2.0 ** -24)
    W = network(L * F, n_out, gen, False)
    y = torch.empty((B, L * F), dtype=torch.float16, device="cuda")
    grid.encode_mlp_fwd(x, theta, *W, y=y)
    for dout in (None, torch.randn((B, n_out), device="cuda", generator=gen)):
        dy = torch.empty_like(y)
        mlp_bwd(y, *W, torch.ones((B, n_out), device="cuda") if dout is None else dout, dy, *[torch.zeros(w.shape, device="cuda") for w in W])
        want = grid.encode_bwd_input(x, theta, dy)
        got = grid.encode_mlp_bwd_input(x, theta, *W, dout, torch.full((B, d), float("nan"), device="cuda"))
        assert want.abs().max() > 1
        assert torch.equal(got, want), float((got - want).abs().max() / want.abs().max())


@pytest.mark.parametrize("d,T,B", [(3, 1 << 19, 1000), (3, 1 << 19, 50000), (2, 1 << 14, 120000)])  # split, paced, free-running
def test_not_a_number_in_a_hidden_layer_is_zero_behind_the_relu(d, T, B):
    gen = torch.Generator(device="cuda").manual_seed(B)
    grid = HashGrid(d, 16, 2, T, 16, 512, "f16", "f16")
    theta = torch.full((grid.n_entries, 2), 1e4, device="cuda").half()
    theta[:, 1] = float("nan")
    x = torch.rand((B, d), device="cuda", generator=gen)
    W = network(32, 3, gen, True)
    W[0][:, 1::2] = 0  # NaN * 0: every neuron of the first layer
    assert torch.equal(grid.encode_mlp_fwd(x, theta, *W), torch.zeros((B, 3), device="cuda"))
    theta[:, 1] = 0
    W[0][:, ::2] = 1  # 16 x 1e4, beyond a half: infinity in every neuron of the first layer
    assert (W[1] == 0).any(dim=1).all()  # and infinity * 0 in every one of the second
    y = torch.empty((B, 32), dtype=torch.float16, device="cuda")
    out = grid.encode_mlp_fwd(x, theta, *W, y=y)
    assert torch.isfinite(y).all()
    assert torch.equal(out, torch.zeros_like(out)) and torch.equal(mlp_fwd(y, *W), out)
