"""The plan of the sorted backward pass, checked on the host, point by point (no GPU): tests/plan_check.hip
is compiled for the host and runs the same rows_of the count and scatter kernels run.  For every pair
of corners it must give the bin, the chunk-local index and the step to the upper corner that lead,
under the record's rules, to the two entries Section 3 and Eq. 4 define, within the bounds the
kernels index with (bin inside its level, index inside its chunk, chunk inside 4096 entries)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2201_05989_amd import binding, synth
from paper_2201_05989_amd.build import CSRC, INCLUDE, LIB_PATH, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan_check(tmp_path_factory):
    binding.load_library()  # raises if libhashgrid.so is not built
    out = str(tmp_path_factory.mktemp("plan") / "libplan_check.so")
    lib_dir = os.path.dirname(LIB_PATH)
    cmd = [hipcc(), "--cuda-host-only", "-O2", "-ffp-contract=off", "-fPIC", "-shared", f"-I{INCLUDE}", f"-I{CSRC}",
           os.path.join(HERE, "plan_check.hip"), "-o", out, f"-L{lib_dir}", "-lhashgrid", f"-Wl,-rpath,{lib_dir}"]
    subprocess.run(cmd, check=True, capture_output=True)
    lib = ctypes.CDLL(out)
    lib.plan_check.restype = ctypes.c_uint64
    lib.plan_check.argtypes = [ctypes.POINTER(binding.hashgrid_config), ctypes.c_uint32, ctypes.c_void_p,
                               ctypes.POINTER(ctypes.c_uint64)]

    def run(d, L, F, T, N_min, N_max, interp, x):
        cfg = binding.hashgrid_config(d, L, F, T, N_min, N_max, binding.HG_F16, binding.HG_F16, interp, binding.HG_F32)
        x = np.ascontiguousarray(x, dtype=np.float32)
        crossing = ctypes.c_uint64(0)
        bad = lib.plan_check(ctypes.byref(cfg), len(x), x.ctypes.data, ctypes.byref(crossing))
        return bad, crossing.value

    run.lib = lib
    return run


@pytest.mark.parametrize("name", ["tiny2d", "image2d", "sdf3d", "nerf3d", "large3d"])
def test_plan_of_every_workload(plan_check, name):
    w = synth.WORKLOADS[name]
    x = synth.make_points(w.points, np.random.default_rng(11), 20000, w.d)
    for interp in (0, 1):
        bad, crossing = plan_check(w.d, w.L, w.F, w.T, w.N_min, w.N_max, interp, x)
        assert bad == 0
        assert (crossing > 0) == (w.N_max >= 4096)  # pairs straddle chunks only at such resolutions


@pytest.mark.parametrize("seed", range(40))
def test_plan_of_random_configurations(plan_check, seed):
    rng = np.random.default_rng(300 + seed)
    d = int(rng.integers(2, 4))
    F = int(rng.choice([1, 2, 4, 8]))
    L = int(rng.integers(1, 17))
    T = 1 << int(rng.integers(0, 24 if F == 8 else 25))
    N_min = int(rng.integers(1, 40))
    N_max = int(N_min * rng.choice([1, 2, 7, 100, 3000]) + rng.integers(0, 5))
    interp = int(rng.integers(0, 2))
    x = synth.points_uniform(rng, 3000, d)
    # grid vertices, the last voxel and the voxels whose pair straddles two chunks, on top of random points
    x[:50] = 0.0
    x[50:100] = 1 - 2.0 ** -24
    x[100:400, 0] = ((4095.75 + 4096.0 * rng.integers(0, 2, 300)) / 8192.0).astype(np.float32)
    bad, _ = plan_check(d, L, F, T, N_min, N_max, interp, x)
    served = binding.HashGrid(d, L, F, T, N_min, N_max, "f16", "f16", interp).bwd_workspace_bytes(3000) > 0
    assert bad == (0 if served else 2 ** 64 - 1)


@pytest.mark.parametrize("seed", range(24))
def test_plan_with_a_record_per_corner(plan_check, seed):
    # table sizes that are not powers of two (Eq. 4's mod T) and one-dimensional inputs: no pairing
    rng = np.random.default_rng(700 + seed)
    d = int(rng.integers(1, 4))
    F = int(rng.choice([1, 2, 4, 8]))
    L = int(rng.integers(1, 12))
    T = int(rng.choice([1, 2, 3, 1000, 4097, 12345, 1000003, 5 * 2 ** 20 + 1])) if d > 1 or seed % 2 else 1 << int(rng.integers(0, 22))
    N_min = int(rng.integers(1, 40))
    N_max = int(N_min * rng.choice([1, 2, 7, 100, 3000]) + rng.integers(0, 5))
    interp = int(rng.integers(0, 2))
    x = synth.points_uniform(rng, 3000, d)
    x[:50] = 0.0
    x[50:100] = 1 - 2.0 ** -24
    bad, _ = plan_check(d, L, F, T, N_min, N_max, interp, x)
    served = binding.HashGrid(d, L, F, T, N_min, N_max, "f16", "f16", interp).bwd_workspace_bytes(3000) > 0
    assert served and bad == 0


def test_plan_where_half_of_the_pairs_straddle_two_chunks(plan_check):
    rng = np.random.default_rng(5)
    for d in (2, 3):
        x = synth.points_uniform(rng, 6000, d)
        x[:3000, 0] = ((4095.75 + 4096.0 * rng.integers(0, 2, 3000)) / 8192.0).astype(np.float32)
        bad, crossing = plan_check(d, 3, 2, 1 << 16, 8192, 32768, 0, x)
        assert bad == 0 and crossing >= 3 * 3000


def test_order_of_records_inside_a_run_is_a_permutation(plan_check):
    """The scatter pass spreads the records a tile puts into one bin (records of neighbouring points apart,
    for the accumulate pass's LDS atomics): whatever the run length, every slot of the run is used exactly once."""
    plan_check.lib.spread_check.restype = ctypes.c_uint32
    plan_check.lib.spread_check.argtypes = [ctypes.c_uint32]
    assert plan_check.lib.spread_check(4096) == 0


@pytest.mark.parametrize("n", [1, 4096, 8388608, 2 ** 32 - 1])
def test_records_of_an_item_never_run_backwards(plan_check, n):
    """Whatever two words a work item holds (counts of another batch, sums that passed 2^32), the accumulate pass walks forwards over
    records there is room for."""
    check = plan_check.lib.item_records_check
    check.restype, check.argtypes = ctypes.c_uint32, [ctypes.c_uint32]
    assert check(n) == 0


@pytest.mark.parametrize("L,F,T,N_max,io,wide", [
    (16, 2, 1 << 22, 32768, "f16", (1 << 16, 1 << 17, 1 << 20)), (16, 1, 1 << 22, 32768, "f32", (1 << 16, 1 << 17, 1 << 20)),
    (8, 4, 1 << 22, 4096, "f16", (1 << 16, 1 << 17, 1 << 20)), (16, 2, 1 << 22, 32768, "f32", (1 << 16,)),
    (16, 4, 1 << 22, 32768, "f16", (1 << 16,)), (8, 4, 1 << 22, 4096, "f32", ()), (8, 8, 1 << 22, 8192, "f16", ()), (8, 8, 1 << 21, 4096, "f32", ()),
    (16, 2, 1 << 21, 32768, "f16", ()), (16, 2, 1 << 24, 1 << 17, "f16", None), (16, 2, 4000003, 32768, "f16", ())])
def test_wide_tiles_where_two_scatter_workgroups_fit_a_compute_unit(plan_check, L, F, T, N_max, io, wide):
    """1024 points a tile of the sort for records of up to 16 bytes where that leaves two workgroups: 2048 records of 8 + F * size bytes
    and 2 more, three words for each of up to 4096 chunks of a part (2048 where a batch of 2^16 points doubles the parts)."""
    io = {"f16": binding.HG_F16, "f32": binding.HG_F32}[io]
    cfg = binding.hashgrid_config(2, L, F, T, 16, N_max, io, io, 0, binding.HG_F32)
    mult_of = plan_check.lib.tile_mult_of
    mult_of.restype, mult_of.argtypes = ctypes.c_uint32, [ctypes.POINTER(binding.hashgrid_config), ctypes.c_uint32]
    for B in ((1 << 16) - 1, 1 << 16, 1 << 17, 1 << 20):
        assert mult_of(ctypes.byref(cfg), B) == (8 if wide is None else 2 if B in wide else 1), B


@pytest.mark.parametrize("d,T,entry_bytes,parts", [
    (3, 1 << 19, 4, {1: 4, 1 << 14: 4, (1 << 14) + 1: 2, 1 << 17: 2, (1 << 17) + 1: 1}),
    (3, 1 << 20, 4, {1 << 14: 4, 1 << 16: 2, (1 << 16) + 1: 1}), (3, 1 << 22, 2, {1 << 16: 2, 100003: 1}), (3, 1 << 24, 2, {100003: 2}),
    (2, 1 << 22, 2, {100003: 2}), (3, 1 << 19, 8, {1 << 16: 2, (1 << 16) + 1: 1}),
    (3, 1 << 20, 16, {1 << 14: 4, 20011: 1, 24577: 2, 1 << 15: 2, 34000: 1}), (2, 1 << 20, 16, {20011: 2, 49152: 2, 49153: 1}),
    (3, 1 << 19, 32, {8192: 4, 8193: 2, 1 << 14: 2, 20011: 1}), (2, 1 << 19, 32, {1 << 14: 4, 1 << 15: 2, 34000: 1}),
    (1, 1 << 19, 32, {34000: 2, 49153: 1})])
def test_parts_of_the_levels_in_the_plain_forward(plan_check, d, T, entry_bytes, parts):
    """Two or four parts only up to the batch at which they stop to pay, by what an entry weighs, d and the table's size."""
    of = plan_check.lib.level_parts_of
    of.restype, of.argtypes = ctypes.c_uint32, [ctypes.c_uint32] * 4
    assert {B: of(d, T, entry_bytes, B) for B in parts} == parts
