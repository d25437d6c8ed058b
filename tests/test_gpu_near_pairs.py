"""Sorted backward pass where a pair's record carries both indices (table sizes that are no power of two, one dimension), at the
edges of that form: batches whose corners all need a record of their own (twice the records that the scatter pass has room to
sort in LDS), far steps, and non-finite gradients, which must not reach entries beside a corner's own record."""
import numpy as np
import pytest
import torch

from oracle import hashgrid_oracle as orc
from paper_2201_05989_amd import HashGrid, synth
from test_gpu_parity import dev, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["vertices", "first voxel", "far steps"])
@pytest.mark.parametrize("d,L,F,T,N,iot,interp,B", [
    (3, 4, 2, 100003, 256, "f32", 0, 5001), (3, 3, 8, 9973, 128, "f32", 0, 1500), (2, 5, 4, 65535, 4096, "f16", 1, 4097),
    (1, 3, 2, 1 << 12, 1 << 14, "f16", 0, 3000)])
def test_pairs_at_the_edges_of_the_record(d, L, F, T, N, iot, interp, B, kind):
    cfg = orc.OracleConfig(d, L, F, T, N, N, interp)
    rng = np.random.default_rng(B)
    x = synth.points_uniform(rng, B, d)
    if kind == "vertices":
        x = (rng.integers(0, N, (B, d)) / N).astype(np.float32)
    elif kind == "first voxel":
        x[:, 0] = rng.random(B) / N
    else:
        k = 1 << rng.integers(3, 7, B)
        x[:, 0] = (rng.integers(0, N // 128, B) * k + k - 0.5 - rng.random(B) / 3) / N
    x = np.clip(x.astype(np.float32), 0, np.float32(1 - 2.0 ** -24))
    lv = orc.levels(cfg)
    run_case(d, L, F, T, N, N, "f32", iot, interp, x, synth.make_tables(rng, lv.total, F, "f32", 1.0),
             synth.make_dy(rng, B, L * F, iot), do_indices=False, do_dx=False)


def test_non_finite_gradients_reach_the_entries_they_belong_to():
    cfg = orc.OracleConfig(3, 4, 2, 5003, 16, 64)
    rng = np.random.default_rng(3)
    x = synth.points_uniform(rng, 3000, 3)
    x[17] = [0.25 / 16, 0.4, 0.6]  # first voxel: a record for each corner
    dy = synth.make_dy(rng, 3000, 8, "f32")
    dy[17, 3], dy[1000, 0] = np.inf, np.nan
    grid = HashGrid(3, 4, 2, 5003, 16, 64, "f32", "f32")
    got = grid.encode_bwd(dev(x), dev(dy), use_workspace=True).cpu().numpy()
    want = grid.encode_bwd(dev(x), dev(dy), use_workspace=False).cpu().numpy()  # the pass of atomic additions
    np.testing.assert_array_equal(np.isfinite(got), np.isfinite(want))
    ok = np.isfinite(want)
    a = orc.encode_bwd(cfg, x, np.abs(np.where(np.isfinite(dy), dy, 0).astype(np.float64)))
    assert (~ok).sum() > 8 and (np.abs(got[ok] - want[ok]) <= 2e-5 * a[ok] + 1e-30).all()


def test_non_finite_gradient_at_a_vertex_reaches_both_corners_of_a_pair():
    """The upper corner's weight is 0 there, and 0 times infinity is not a number: as in the pass of atomic additions."""
    rng = np.random.default_rng(5)
    x = (rng.integers(0, 64, (2000, 3)) / 64).astype(np.float32)
    dy = synth.make_dy(rng, 2000, 2, "f32")
    dy[100, 0] = np.inf
    grid = HashGrid(3, 1, 2, 50021, 64, 64, "f32", "f32")
    got = grid.encode_bwd(dev(x), dev(dy), use_workspace=True).cpu().numpy()
    want = grid.encode_bwd(dev(x), dev(dy), use_workspace=False).cpu().numpy()
    np.testing.assert_array_equal(np.isfinite(got), np.isfinite(want))
    assert (~np.isfinite(want)).sum() == 8


@pytest.mark.parametrize("d,F,iot,interp,T,N_min,N_max,B", [
    (3, 2, "f16", 0, (1 << 24) - 3, 8192, 65536, 4096 + 513), (2, 1, "f32", 1, (1 << 24) - 3, 8192, 65536, 9000),
    (1, 2, "f32", 0, 1 << 24, 1 << 23, 1 << 25, 5000)])
def test_very_many_chunks(d, F, iot, interp, T, N_min, N_max, B):
    """More than 16384 chunks in all: the scatter pass writes its records unsorted, one or two a pair."""
    cfg = orc.OracleConfig(d, 5, F, T, N_min, N_max, interp)
    lv = orc.levels(cfg)
    assert sum(-(-int(n) // 4096) for n in lv.size) > 16384
    rng = np.random.default_rng(B)
    x = synth.points_uniform(rng, B, d)
    x[: B // 4] = rng.integers(0, N_min, (B // 4, d)) / N_min  # vertices
    x[B // 4: B // 2, 0] = rng.random(B // 2 - B // 4) / N_min  # first voxel
    x[B // 2: 3 * B // 4, 0] = (4095.75 + 4096 * rng.integers(0, N_min // 4096, 3 * B // 4 - B // 2)) / N_min  # far steps
    x = np.clip(x.astype(np.float32), 0, np.float32(1 - 2.0 ** -24))
    theta = synth.make_tables(rng, lv.total, F, "f16", 1.0)
    grid = run_case(d, 5, F, T, N_min, N_max, "f16", iot, interp, x, theta, synth.make_dy(rng, B, 5 * F, iot), do_indices=False,
                    do_dx=False)
    assert grid.bwd_workspace_bytes(B) > 0
