"""Forward pass with two points a thread (batches of two rounds of workgroups and more) against the same points in batches that the
kernel with one point a thread takes, where a store holds four or eight levels' outputs, counting and plain."""
import pytest
import torch

from paper_2201_05989_amd import HashGrid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [False, "always"])
@pytest.mark.parametrize("d,L,F,param", [(2, 8, 1, "f16"), (3, 16, 1, "f16"), (3, 4, 2, "f16"), (3, 16, 2, "f32"), (2, 12, 2, "f16")])
@pytest.mark.parametrize("B", [1 << 19, (1 << 19) + 2049])
def test_two_points_a_thread(d, L, F, param, B, count):
    grid = HashGrid(d, L, F, 1 << 14, 16, 512, param, "f16")
    gen = torch.Generator(device="cuda").manual_seed(B + d)
    x = torch.rand(B, d, device="cuda", generator=gen).clamp_(max=1 - 2.0 ** -24)
    theta = (torch.rand(grid.n_entries, F, device="cuda", generator=gen) * 2 - 1).to(torch.float16 if param == "f16" else torch.float32)
    y = grid.encode_fwd(x, theta, count_for_bwd=count).float().reshape(B, -1)
    step = 100_001
    for b in range(0, B, step):
        want = grid.encode_fwd(x[b:b + step].contiguous(), theta).float().reshape(-1, L * F)
        # the same sum in 32 bits, rounded to half precision once or (folded or not) twice: one unit in the last place at most
        assert ((y[b:b + step] - want).abs() <= 2.0 ** -10 * want.abs() + 2.0 ** -24).all()


@pytest.mark.parametrize("d,param", [(2, "f16"), (2, "f32"), (3, "f16"), (3, "f32")])
def test_two_features_are_rounded_alike(d, param):
    """F = 2 in half precision: the sum is rounded to 32 bits and then to 16, plain and counting, at every level of a row."""
    grid = HashGrid(d, 16, 2, 1 << 16, 16, 1024, param, "f16")
    gen = torch.Generator(device="cuda").manual_seed(d)
    x = torch.rand(1 << 19, d, device="cuda", generator=gen).clamp_(max=1 - 2.0 ** -24)
    theta = (torch.rand(grid.n_entries, 2, device="cuda", generator=gen) * 2 - 1).to(torch.float16 if param == "f16" else torch.float32)
    assert torch.equal(grid.encode_fwd(x, theta), grid.encode_fwd(x, theta, count_for_bwd="always"))
