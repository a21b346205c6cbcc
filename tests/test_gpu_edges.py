"""Edge cases of the field path: the largest lateral sizes (4096-point
transforms), the largest layer count, and rejected batch sizes."""
import ctypes

import numpy as np
import pytest

import oracle
from hfd_testlib import plan_for, rel_err, run_field
from paper_1910_07054_amd import hfd
from paper_1910_07054_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hfd.load()


# (nx, ny, nz): nx = 2048 -> Lx = 4096 (x passes at their largest length),
# ny = 2048 -> Ly = 4096 (five-pass y transforms at their largest length),
# nz = 64 (largest layer count; 16 target groups in the five-pass mixing)
EDGE = [(2048, 3, 1), (3, 2048, 2), (7, 5, 64)]


@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("case", EDGE, ids=lambda c: "x".join(map(str, c)))
def test_largest_sizes_match_bruteforce(case, fp64):
    nx, ny, nz = case
    wl = W.small_case(nx, ny, nz, seed=1200 + nz, batch=1)
    plan = plan_for(wl, flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    h, mused = run_field(plan, wl.m)
    ref = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mused[0])
    assert rel_err(h[0], ref) < (1e-10 if fp64 else 1e-5)
    plan.destroy()


def test_equidistant_largest_layer_count():
    nx, ny, nz, t = 6, 5, 64, 0.5
    rng = np.random.default_rng(1264)
    m = W.random_unit(rng, (nz, ny, nx))[None]
    zb = np.arange(nz) * t
    plan = hfd.Plan(nx, ny, 2.0, 1.5, np.full(nz, t), zb, batch_max=1, flags=hfd.HFD_EQUIDISTANT)
    assert plan.info().Lz == 128
    h, mused = run_field(plan, m)
    ref = oracle.field(nx, ny, 2.0, 1.5, zb, np.full(nz, t), mused[0])
    assert rel_err(h[0], ref) < 1e-5
    plan.destroy()


def test_rejected_batch_sizes():
    import torch
    wl = W.small_case(8, 6, 2, seed=1300, batch=2)
    plan = plan_for(wl)
    m = torch.zeros((2, 3, 2, 6, 8), device="cuda")
    h = torch.empty_like(m)
    lib = hfd.load()
    assert lib.hfd_demag_field(plan.handle, m.data_ptr(), h.data_ptr(), 0, None) == hfd.HFD_EINVAL
    assert lib.hfd_demag_field(plan.handle, m.data_ptr(), h.data_ptr(), -1, None) == hfd.HFD_EINVAL
    assert lib.hfd_demag_field(plan.handle, m.data_ptr(), h.data_ptr(), 3, None) == hfd.HFD_EBATCH
    # aliasing input and output is rejected
    assert lib.hfd_demag_field(plan.handle, m.data_ptr(), m.data_ptr(), 1, None) == hfd.HFD_EINVAL
    assert lib.hfd_demag_field(plan.handle, m.data_ptr(), h.data_ptr(), 2, None) == hfd.HFD_OK
    torch.cuda.synchronize()
    plan.destroy()


# five-pass y transforms whose groups walk over several columns, a few blocks of
# which have one round more than the others, and a call with few columns (the
# five-pass path is forced where the fused one would be taken); Ly = 8, 64, 2048, 64
@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B", [(128, 3, 7, 100), (40, 20, 6, 29), (5, 520, 2, 86), (130, 17, 1, 1)])
def test_y_transforms_of_many_columns_match_bruteforce(nx, ny, nz, B, fp64):
    wl = W.small_case(nx, ny, nz, seed=1500 + nz, batch=1)
    one = wl.m[0]
    m = np.stack([np.roll(one, 5 * b, axis=-1) for b in range(B)])
    plan = hfd.Plan(nx, ny, wl.dx, wl.dy, wl.thickness[0], wl.z_bottom[0], batch_max=B,
                    flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    plan.set_path(B, 1, 0)
    h, mused = run_field(plan, m)
    for b in (0, B // 2, B - 1):
        ref = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mused[b])
        assert rel_err(h[b], ref) < (1e-10 if fp64 else 1e-5), b
    plan.destroy()


# transforms with radix-16 passes at 1024 and 2048 points: x passes (2000 cells: 2048
# after the split), fused and five-pass y passes, the crop inside and at the end of
# the half that the last pass stores
@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz", [(513, 2, 2), (1024, 1, 1), (1100, 2, 1), (2, 257, 1), (3, 512, 4),
                                      (2, 300, 5), (2, 513, 3), (1, 1024, 1)])
def test_radix_16_transforms_match_bruteforce(nx, ny, nz, fp64):
    wl = W.small_case(nx, ny, nz, seed=1600 + nx + ny, batch=2)
    plan = plan_for(wl, flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    h, mused = run_field(plan, wl.m)
    for b in range(2):
        ref = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mused[b])
        assert rel_err(h[b], ref) < (1e-10 if fp64 else 1e-5), b
    plan.destroy()


# threads per block of the generic fused kernel: launches on both sides of the line
# between one round of transforms and one thread per frequency, where the two differ
@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B", [(33, 30, 3, 15), (33, 30, 3, 17), (33, 10, 8, 40), (33, 6, 12, 40),
                                        (9, 60, 11, 33), (70, 100, 2, 3), (33, 3, 4, 3)])
def test_fused_threads_per_block_match_bruteforce(nx, ny, nz, B, fp64):
    wl = W.small_case(nx, ny, nz, seed=1700 + ny, batch=1)
    m = np.stack([np.roll(wl.m[0], b, axis=-1) for b in range(B)])
    plan = hfd.Plan(nx, ny, wl.dx, wl.dy, wl.thickness[0], wl.z_bottom[0], batch_max=B,
                    flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    h, mused = run_field(plan, m)
    for b in (0, B // 2, B - 1):
        ref = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mused[b])
        assert rel_err(h[b], ref) < (1e-10 if fp64 else 1e-5), b
    plan.destroy()


# x passes of 256-point transforms (16 values per lane), every tile height
@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz", [(129, 3, 2), (256, 5, 1), (200, 7, 3), (255, 1, 1)])
def test_x_passes_of_256_points_match_bruteforce(nx, ny, nz, fp64):
    wl = W.small_case(nx, ny, nz, seed=1800 + nx, batch=2)
    plan = plan_for(wl, flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    refs = None
    for ty in (0, 4, 8, 12, 16, 24, 32):
        plan.set_path(2, 1, ty)
        h, mused = run_field(plan, wl.m)
        if refs is None:
            refs = [oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mu) for mu in mused]
        for b in range(2):
            assert rel_err(h[b], refs[b]) < (1e-10 if fp64 else 1e-5), (ty, b)
    plan.destroy()


# 128-point x transforms on both sides of the row count from which a lane takes 16 values
@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B", [(128, 2, 2, 700), (65, 3, 1, 911), (100, 1, 3, 910)])
def test_x_passes_of_128_points_many_rows(nx, ny, nz, B, fp64):
    wl = W.small_case(nx, ny, nz, seed=1900 + nx, batch=1)
    m = np.stack([np.roll(wl.m[0], b, axis=-1) for b in range(B)])
    plan = hfd.Plan(nx, ny, wl.dx, wl.dy, wl.thickness[0], wl.z_bottom[0], batch_max=B,
                    flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    refs = {}
    for ty in (0, 4, 8, 16, 24, 32):
        plan.set_path(B, 1, ty)
        h, mused = run_field(plan, m)
        for b in (0, B // 2, B - 1):
            if b not in refs:
                refs[b] = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mused[b])
            assert rel_err(h[b], refs[b]) < (1e-10 if fp64 else 1e-5), (ty, b)
    plan.destroy()


# 4096-point column transforms, more columns than blocks: one column per group in the
# FP64 forward pass, walking groups in the others
@pytest.mark.parametrize("fp64", [False, True], ids=["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,nz,B", [(5, 1025, 2, 43), (3, 2048, 1, 86), (1, 1300, 1, 1)])
def test_y_transforms_of_4096_points(nx, ny, nz, B, fp64):
    wl = W.small_case(nx, ny, nz, seed=2200 + ny, batch=1)
    m = np.stack([np.roll(wl.m[0], 7 * b, axis=-2) for b in range(B)])
    plan = hfd.Plan(nx, ny, wl.dx, wl.dy, wl.thickness[0], wl.z_bottom[0], batch_max=B,
                    flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    h, mused = run_field(plan, m)
    plan.destroy()
    rng = np.random.default_rng(ny)
    smp = np.stack([rng.integers(0, nz, 30), rng.integers(0, ny, 30), rng.integers(0, nx, 30)], axis=1)
    smp[0], smp[1] = (0, 0, 0), (nz - 1, ny - 1, nx - 1)
    for b in (0, B // 2, B - 1):
        ref = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], mused[b], samples=smp)
        got = h[b][:, smp[:, 0], smp[:, 1], smp[:, 2]].T
        err = np.abs(got - ref).max() / np.linalg.norm(ref, axis=1).max()
        assert err < (1e-10 if fp64 else 1e-5), (b, err)
