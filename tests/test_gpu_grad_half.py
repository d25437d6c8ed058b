"""Half-precision table gradients (grad_dtype = fp16; the paper accumulates its gradients in half
precision with packed two-half atomics, Section 4 "Performance considerations" and Fig. 5), through
the C ABI, against the fp64 oracle.

Bars.  An fp16 result cannot be closer than half a unit in the last place, 2^-11 relative (2^-25
absolute among subnormals).  The sorted pass sums exactly and rounds once where one workgroup owns a
chunk: |g - g*| <= 2^-11 |g*| + 2^-25 on top of its fp32 bar (1e-5 A + fixed-point floor, A the
sum of the absolute values of the entry's summands).  Where several workgroups share a chunk (coarse
1:1 levels of large batches) each adds its partial sum with a rounded atomic: (s + 1) 2^-11 A for
s sharers.  The atomic pass rounds every summand and every running sum: (n + 1) 2^-11 A + n 2^-25
for an entry with n summands - the loss of precision the paper's choice accepts.
"""
import numpy as np
import pytest
import torch

from oracle import hashgrid_oracle as orc
from paper_2201_05989_amd import HashGrid, synth

pytestmark = pytest.mark.gpu

U, SUB = 2.0 ** -11, 2.0 ** -25


def fixed_floor(dy, B):
    H = max(3 + int(np.ceil(np.log2(max(B, 2)))), 11)
    return float(np.abs(dy.astype(np.float64)).max()) * 2.0 ** (H - 54)


def corner_counts(cfg, lv, x):
    n = np.zeros((lv.total, 1))
    for l in range(cfg.L):
        idx, _ = orc.indices(cfg, x, l)
        lo, size = int(lv.offset[l]), int(lv.size[l])
        n[lo:lo + size, 0] = np.bincount(idx.astype(np.int64).ravel(), minlength=size)
    return n


def case(d, L, F, T, N_min, N_max, iot, interp, B, seed, points="uniform"):
    cfg = orc.OracleConfig(d, L, F, T, N_min, N_max, interp)
    lv = orc.levels(cfg)
    rng = np.random.default_rng(seed)
    x = synth.make_points(points, rng, B, d)
    dy = synth.make_dy(rng, B, L * F, iot)
    g_ref = orc.encode_bwd(cfg, x, dy)
    g_abs = orc.encode_bwd(cfg, x, np.abs(dy.astype(np.float64)))
    grid = HashGrid(d, L, F, T, N_min, N_max, "f16", iot, interp, grad_dtype="f16")
    return cfg, lv, x, dy, g_ref, g_abs, grid


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("F", [1, 2, 4, 8])
@pytest.mark.parametrize("iot", ["f16", "f32"])
def test_sorted_pass_rounds_once_where_a_chunk_has_one_owner(F, iot):
    B = 3000  # few enough records per chunk for one workgroup each, on every level
    cfg, lv, x, dy, g_ref, g_abs, grid = case(3, 16, F, 1 << 19, 16, 2048, iot, 0, B, 40 + F)
    assert grid.bwd_workspace_bytes(B) > 0
    xd, gd = dev(x), dev(dy)
    g = grid.encode_bwd(xd, gd, use_workspace=True)
    assert g.dtype == torch.float16
    bound = 1e-5 * g_abs + fixed_floor(dy, B) + U * np.abs(g_ref) + SUB
    err = np.abs(g.cpu().numpy().astype(np.float64) - g_ref)
    assert (err <= bound).all(), f"{int((err > bound).sum())} entries off, worst {np.max(err / bound):.3f} of the bound"
    assert (g.cpu().numpy()[g_abs == 0] == 0).all()
    # replacing whatever the buffer held gives the same gradient; adding into it again doubles it (one more rounding)
    go = grid.encode_bwd(xd, gd, torch.full_like(g, float("nan")), use_workspace=True, overwrite=True)
    assert torch.equal(go, g)
    g2 = grid.encode_bwd(xd, gd, g.clone(), use_workspace=True)
    err2 = np.abs(g2.cpu().numpy().astype(np.float64) - 2 * g_ref)
    assert (err2 <= 2 * bound + 2 * U * np.abs(g_ref) + SUB).all()


@pytest.mark.parametrize("d,L,F,T,N_min,N_max,iot,interp,B,points", [
    (3, 16, 2, 1 << 19, 16, 2048, "f16", 0, 40001, "sdf"),       # coarse chunks shared by several workgroups
    (2, 8, 2, 1 << 16, 8192, 32768, "f16", 0, 20000, "uniform"),  # pairs that straddle two chunks: atomics on the side
    (3, 8, 1, 1000003, 16, 512, "f32", 1, 9000, "uniform"),       # pairs that carry both indices, single features, smoothstep
    (1, 10, 4, 1 << 14, 16, 1 << 16, "f16", 0, 30000, "uniform"),
])
def test_sorted_pass_with_shared_chunks_and_atomic_side_paths(d, L, F, T, N_min, N_max, iot, interp, B, points):
    cfg, lv, x, dy, g_ref, g_abs, grid = case(d, L, F, T, N_min, N_max, iot, interp, B, 60 + B, points)
    if points == "uniform" and d == 2:
        x[: B // 4, 0] = ((4095.75 + 4096.0 * np.random.default_rng(1).integers(0, 2, B // 4)) / 8192.0).astype(np.float32)
        g_ref = orc.encode_bwd(cfg, x, dy)
        g_abs = orc.encode_bwd(cfg, x, np.abs(dy.astype(np.float64)))
    assert grid.bwd_workspace_bytes(B) > 0
    g = grid.encode_bwd(dev(x), dev(dy), use_workspace=True).cpu().numpy().astype(np.float64)
    sharers = int(np.ceil(B * (1 << d) / 16384)) + 2  # no chunk has more workgroups than this; +2 for straddling pairs
    bound = 1e-5 * g_abs + fixed_floor(dy, B) + U * np.abs(g_ref) + SUB + sharers * U * g_abs
    err = np.abs(g - g_ref)
    assert (err <= bound).all(), f"{int((err > bound).sum())} entries off"
    # most entries have a single owner and no side path: they meet the one-rounding bar
    tight = err <= 1e-5 * g_abs + fixed_floor(dy, B) + U * np.abs(g_ref) + SUB
    assert tight.mean() > 0.9


@pytest.mark.parametrize("F", [1, 2, 4, 8])
def test_atomic_pass_accumulates_in_half_precision_as_the_paper_does(F):
    B = 2000
    cfg, lv, x, dy, g_ref, g_abs, grid = case(3, 8, F, 1 << 14, 16, 512, "f16", 0, B, 80 + F)
    n = corner_counts(cfg, lv, x)
    g = grid.encode_bwd(dev(x), dev(dy), use_workspace=False)
    assert g.dtype == torch.float16
    err = np.abs(g.cpu().numpy().astype(np.float64) - g_ref)
    bound = (n + 1) * U * g_abs + n * SUB
    assert (err <= bound).all(), f"{int((err > bound).sum())} entries off"
    assert (g.cpu().numpy()[g_abs == 0] == 0).all()
    # entries with a single summand: the summand rounded once
    one = (n[:, 0] == 1)
    assert one.sum() > 100
    assert (err[one] <= U * g_abs[one] + SUB).all()


def test_half_gradients_need_a_four_byte_boundary():
    grid = HashGrid(3, 4, 1, 1 << 10, 4, 32, "f16", "f16", grad_dtype="f16")
    B = 1000
    x = torch.rand((B, 3), device="cuda") * 0.99
    dy = torch.ones((B, 4), dtype=torch.float16, device="cuda")
    buf = torch.zeros(grid.n_entries + 2, dtype=torch.float16, device="cuda")
    ws = torch.empty(grid.bwd_workspace_bytes(B), dtype=torch.uint8, device="cuda")
    odd = buf[1:1 + grid.n_entries]
    assert odd.data_ptr() % 4 == 2
    lib = grid._lib
    assert lib.hashgrid_encode_bwd(grid._h, B, x.data_ptr(), dy.data_ptr(), odd.data_ptr(), None) == 1
    assert lib.hashgrid_encode_bwd_ws(grid._h, B, x.data_ptr(), dy.data_ptr(), odd.data_ptr(), ws.data_ptr(),
                                      ws.numel(), 0, None) == 1
    assert lib.hashgrid_encode_bwd(grid._h, B, x.data_ptr(), dy.data_ptr(), buf.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert float(buf[grid.n_entries:].abs().sum()) == 0.0
