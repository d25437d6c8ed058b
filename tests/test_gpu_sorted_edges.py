"""Sorted backward pass where its kernels change shape: work items around a row of records and around the rows on their way, tables
of counts around the rows that a thread of the scan keeps, and the plain forward's parts of the levels; against the oracle."""
import numpy as np
import pytest
import torch

from oracle import hashgrid_oracle as orc
from paper_2201_05989_amd import HashGrid, synth
from test_gpu_parity import check_fwd, dev, run_case, same_forward, ws_floor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,iot", [(1, "f16"), (2, "f16"), (2, "f32"), (4, "f32"), (8, "f16"), (8, "f32")])
@pytest.mark.parametrize("B", [1, 511, 512, 513, 1023, 1025, 2048, 2049, 4097, 8193])
def test_items_around_a_row_of_records(F, iot, B):
    """d = 2, one chunk: 2 B records in an item of rows of 1024, up to 16384 of them, and beyond that in shares."""
    T = 2048 if F == 8 else 4096
    rng = np.random.default_rng(B * 10 + F)
    x = synth.points_uniform(rng, B, 2)
    run_case(2, 1, F, T, 100, 100, "f32", iot, 0, x, synth.make_tables(rng, T, F, "f32", 1.0), synth.make_dy(rng, B, F, iot),
             do_indices=False, do_dx=False)


@pytest.mark.parametrize("tiles", [64, 256, 512, 1024, 2048])
@pytest.mark.parametrize("more", [0, 1])
def test_scan_of_tables_around_its_row_counts(tiles, more):
    B = 512 * tiles + more
    cfg = orc.OracleConfig(2, 2, 1, 1 << 15, 60, 300)
    rng = np.random.default_rng(tiles + more)
    x, dy = synth.points_uniform(rng, B, 2), synth.make_dy(rng, B, 2, "f16")
    grid = HashGrid(2, 2, 1, 1 << 15, 60, 300, "f16", "f16")
    got = torch.full((grid.n_entries, 1), 7.0, device="cuda")
    grid.encode_bwd(dev(x), dev(dy), got, use_workspace=True, overwrite=True)
    want, mass = orc.encode_bwd(cfg, x, dy), orc.encode_bwd(cfg, x, np.abs(dy.astype(np.float64)))
    # the floor of the fixed-point sums, at most 2^(H - 54) of the largest |dL/dy|; the shares of a chunk are added in single precision
    H = max(3 + int(np.ceil(np.log2(B))), 11)
    assert (np.abs(got.cpu().numpy().reshape(want.shape) - want) <= 1e-5 * mass + float(np.abs(dy).max()) * 2.0 ** (H - 54)).all()


@pytest.mark.parametrize("d,L,F,T,param,io", [
    (2, 4, 2, 1 << 10, "f32", "f32"), (3, 16, 2, 1 << 12, "f16", "f16"), (3, 12, 2, 5003, "f16", "f16"), (2, 8, 1, 1 << 12, "f16", "f16"),
    (3, 3, 8, 1 << 11, "f16", "f16"), (1, 10, 2, 1 << 8, "f32", "f32"), (3, 5, 8, 1 << 11, "f32", "f32")])
@pytest.mark.parametrize("B", [1, 65, 1 << 14, (1 << 14) + 1, 49153, (1 << 16) + 1])
def test_forward_in_parts_of_the_levels(d, L, F, T, param, io, B):
    """1, 2 and 4 parts of whole 16-byte pieces, even and odd numbers of them."""
    rng = np.random.default_rng(B + L)
    grid = HashGrid(d, L, F, T, 8, 128, param, io)
    x, theta = synth.points_uniform(rng, B, d), synth.make_tables(rng, grid.n_entries, F, param, 1.0)
    y = grid.encode_fwd(dev(x), dev(theta))
    at = np.unique(np.concatenate([np.arange(min(B, 700)), np.arange(max(0, B - 700), B)]))
    check_fwd(y.cpu().numpy()[at], orc.encode_fwd(orc.OracleConfig(d, L, F, T, 8, 128), x[at], theta), 1.0, io)
    if B > 65:  # every row, against calls with another number of parts
        same_forward(y, torch.cat([grid.encode_fwd(dev(x[b:b + 4096]), dev(theta)) for b in range(0, B, 4096)]), io)


@pytest.mark.parametrize("L,F,T,param,io,grad,interp", [
    (4, 2, 1 << 22, "f16", "f16", "f32", 0), (4, 2, 1 << 22, "f32", "f32", "f32", 1), (8, 1, 1 << 22, "f32", "f32", "f32", 1),
    (2, 4, 1 << 22, "f16", "f16", "f32", 0), (2, 4, 1 << 22, "f16", "f16", "f16", 1), (2, 8, 1 << 21, "f16", "f16", "f16", 0)])
@pytest.mark.parametrize("B", [1 << 16, (1 << 16) + 513, (1 << 18) + 1025])
def test_tiles_of_twice_the_points(L, F, T, param, io, grad, interp, B):
    """d = 2, levels of 1024 chunks, 2^16 points and more: two points a thread of the scatter pass (one for the records of eight
    features), counted by itself and by the forward, replacing a gradient and adding to one.  One point in eight lies where its pair straddles two chunks of the finest level: those
    pairs are added by the scatter pass, or after the owners have stored."""
    cfg = orc.OracleConfig(2, L, F, T, 1500, 9000, interp)
    grid, lv = HashGrid(2, L, F, T, 1500, 9000, param, io, interp, grad), orc.levels(cfg)
    rng = np.random.default_rng(B + 10 * F + L)
    x, dy = synth.points_uniform(rng, B, 2), synth.make_dy(rng, B, L * F, io)
    chunk = 2048 if F == 8 else 4096
    x[:B // 8, 0] = ((chunk - 0.9 + 0.3 * rng.random(B // 8)) / 9000).astype(np.float32)
    n = np.zeros((lv.total, 1))  # an entry's additions by such pairs: an atomic each
    for l in range(L):
        lo, size, N = int(lv.offset[l]), int(lv.size[l]), int(lv.N[l])
        if lv.dense[l] or N + 1 < chunk:
            continue
        c0 = np.floor(x[:, 0] * np.float32(N) + np.float32(0.5 * interp)).astype(np.int64)
        idx, _ = orc.indices(cfg, x[c0 % chunk == chunk - 1], l)
        n[lo:lo + size, 0] = np.bincount(idx.astype(np.int64).ravel(), minlength=size)
    assert n.sum() >= B // 2
    n, want, mass = dev(n), dev(orc.encode_bwd(cfg, x, dy)), dev(orc.encode_bwd(cfg, x, np.abs(dy.astype(np.float64))))
    xd, gd = dev(x), dev(dy)
    gen = torch.Generator(device="cuda").manual_seed(B)
    theta = torch.randn(grid.n_entries, F, device="cuda", generator=gen).to(grid.param_dtype)
    # A rounding where the owner stores, one of the running sum for every atomic (what was there and the summands' mass bound it); an
    # atomic's half-precision summand is itself rounded, at most u times the mass over all of them and the smallest half for each.
    u, sub = (1.001 * 2.0 ** -11, 2.0 ** -25) if grad == "f16" else (1.001 * 2.0 ** -24, 0.0)
    summands = (n > 0) * u * mass if grad == "f16" else 0.0
    some = torch.randint(-2, 3, (grid.n_entries, F), device="cuda", generator=gen).to(grid.grad_dtype)
    for count in (False, "always"):
        for overwrite, before in ((True, torch.full_like(some, 7.0)), (False, torch.zeros_like(some)), (False, some)):
            base = torch.zeros_like(want) if overwrite else before.double()
            bar = 1e-5 * mass + ws_floor(dy, B) + u * (base + want).abs() + sub + summands + n * (u * (base.abs() + mass) + sub)
            grid.encode_fwd(xd, theta, count_for_bwd=count)
            got = before.clone()
            grid.encode_bwd(xd, gd, got, use_workspace=True, overwrite=overwrite)
            err = (got.double() - base - want).abs()
            assert (err <= bar).all(), (count, overwrite, int((err > bar).sum()))
