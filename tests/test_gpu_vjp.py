"""GPU parity of the vector-Jacobian products (adjoint in m, thickness
gradient) against the oracle and against finite differences."""
import numpy as np
import pytest

import oracle
from paper_1910_07054_amd import hfd
from paper_1910_07054_amd import workloads as W
from hfd_testlib import plan_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hfd.load()


def _vjp(plan, m_np, g_np, want_m=True, want_t=True):
    import torch
    dt = np.float64 if plan.fp64 else np.float32
    m = torch.from_numpy(np.ascontiguousarray(m_np.astype(dt))).cuda()
    g = torch.from_numpy(np.ascontiguousarray(g_np.astype(dt))).cuda()
    gm, gt = plan.vjp(m, g, want_m=want_m, want_t=want_t)
    torch.cuda.synchronize()
    return (None if gm is None else gm.cpu().numpy().astype(np.float64),
            None if gt is None else gt.cpu().numpy())


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("store", [False, True])
def test_thickness_gradient_matches_oracle(fp64, store):
    wl = W.small_case(13, 11, 4, seed=401, batch=2)
    flags = (hfd.HFD_FP64 if fp64 else hfd.HFD_FP32) | (hfd.HFD_STORE_DTENSOR if store else 0)
    plan = plan_for(wl, flags=flags)
    g = np.random.default_rng(9).standard_normal(wl.m.shape)
    dt = np.float64 if fp64 else np.float32
    mr, gr = wl.m.astype(dt).astype(np.float64), g.astype(dt).astype(np.float64)
    _, gt = _vjp(plan, wl.m, g, want_m=False)
    for b in range(2):
        ref = oracle.thickness_grad(wl.nx, wl.ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0],
                                    mr[b], gr[b])
        err = np.abs(gt[b] - ref).max() / np.abs(ref).max()
        assert err < (1e-10 if fp64 else 2e-5), (b, err, gt[b], ref)
    plan.destroy()


def test_thickness_gradient_several_stacks_and_split_path():
    """n_geom stacks in one batch (each state uses its own stack) on the
    five-pass path; also both gradients requested in one call."""
    rng = np.random.default_rng(12)
    nx, ny, nz, G = 9, 14, 3, 3
    t = rng.uniform(0.5, 2.5, (G, nz))
    zb = np.stack([W.stack_bottoms(t[g], [0.3, 0.0]) for g in range(G)])
    m = np.stack([W.random_unit(rng, (nz, ny, nx)) for _ in range(G * 2)])
    g = rng.standard_normal(m.shape)
    plan = hfd.Plan(nx, ny, 2.0, 1.0, t, zb, batch_max=G * 2,
                    flags=hfd.HFD_FP64 | hfd.HFD_SPLIT_PASSES)
    gm, gt = _vjp(plan, m, g)
    for b in range(G * 2):
        k = b // 2
        ref_t = oracle.thickness_grad(nx, ny, 2.0, 1.0, zb[k], t[k], m[b], g[b])
        assert np.abs(gt[b] - ref_t).max() < 1e-10 * np.abs(ref_t).max()
        ref_m = oracle.field(nx, ny, 2.0, 1.0, zb[k], t[k], g[b], transpose=True)
        assert np.abs(gm[b] - ref_m).max() < 1e-11 * np.abs(ref_m).max()
    plan.destroy()


@pytest.mark.parametrize("chunk", [0, 1, 2, 4])
def test_both_gradients_on_the_fused_path_in_state_runs(chunk):
    """Both gradients in one call on the fused path (one x pass of grad_h per
    run of states feeds the gradient's spectra and the adjoint pass), with the
    states of two stacks in one run (chunk 0: the whole batch of 4) or in
    runs of 1, 2 or 4 states (hfd_set_fused); against the oracle per state."""
    rng = np.random.default_rng(13)
    nx, ny, nz, G, bpg = 12, 10, 3, 2, 2
    t = rng.uniform(0.5, 2.5, (G, nz))
    zb = np.stack([W.stack_bottoms(t[g], [0.3, 0.0]) for g in range(G)])
    m = np.stack([W.random_unit(rng, (nz, ny, nx)) for _ in range(G * bpg)])
    g = rng.standard_normal(m.shape)
    plan = hfd.Plan(nx, ny, 2.0, 1.5, t, zb, batch_max=G * bpg)
    assert plan.info().fused
    plan.set_fused(G * bpg, chunk)
    gm, gt = _vjp(plan, m, g)
    for b in range(G * bpg):
        k = b // bpg
        ref_t = oracle.thickness_grad(nx, ny, 2.0, 1.5, zb[k], t[k], m[b], g[b])
        assert np.abs(gt[b] - ref_t).max() < 2e-5 * np.abs(ref_t).max(), (chunk, b)
        ref_m = oracle.field(nx, ny, 2.0, 1.5, zb[k], t[k], g[b], transpose=True)
        assert np.abs(gm[b] - ref_m).max() < 1e-5 * np.abs(ref_m).max(), (chunk, b)
    plan.destroy()


def test_dot_product_identity_on_gpu():
    """<g, A m> = <A^T g, m> with both operators from the GPU (FP64)."""
    import torch
    wl = W.small_case(31, 17, 5, seed=402)
    plan = plan_for(wl, flags=hfd.HFD_FP64)
    g = np.random.default_rng(3).standard_normal(wl.m.shape)
    m = torch.from_numpy(wl.m).cuda()
    Am = plan.field(m).cpu().numpy()
    ATg, _ = _vjp(plan, wl.m, g, want_t=False)
    assert np.vdot(g, Am) == pytest.approx(np.vdot(ATg, wl.m), rel=1e-12)
    plan.destroy()


def test_thickness_gradient_matches_fp64_finite_differences():
    """Central differences of L = <g, h> computed by the GPU FP64 path with the
    stack re-set (layers above the thickened one move up)."""
    import torch
    wl = W.small_case(20, 16, 3, seed=403)
    t0, z0 = wl.thickness[0].copy(), wl.z_bottom[0].copy()
    plan = plan_for(wl, flags=hfd.HFD_FP64)
    g = np.random.default_rng(8).standard_normal(wl.m.shape)
    _, gt = _vjp(plan, wl.m, g, want_m=False)
    m = torch.from_numpy(wl.m).cuda()
    eps = 1e-5
    for k in range(3):
        vals = []
        for sgn in (1, -1):
            t, z = t0.copy(), z0.copy()
            t[k] += sgn * eps
            z[k + 1:] += sgn * eps
            plan.set_thickness(t, z)
            vals.append(np.vdot(g, plan.field(m).cpu().numpy()))
        fd = (vals[0] - vals[1]) / (2 * eps)
        assert gt[0, k] == pytest.approx(fd, rel=1e-6, abs=1e-9)
    plan.destroy()


@pytest.mark.parametrize("nz, gaps", [(1, None), (20, "mixed")], ids=["one_layer", "twenty_layers_gaps"])
def test_thickness_gradient_interface_counts(nz, gaps):
    """One layer (two interface positions) and 20 layers where some layers
    touch and others have gaps (32 positions: several source chunks and the
    widest per-position accumulator), FP64 against the oracle."""
    rng = np.random.default_rng(40 + nz)
    nx, ny = 7, 6
    t = rng.uniform(0.4, 2.0, nz)
    if gaps is None:
        zb = W.stack_bottoms(t, np.zeros(nz - 1))
    else:
        gv = np.where(np.arange(nz - 1) % 5 == 2, 0.0, rng.uniform(0.05, 0.6, nz - 1))
        gv[::4] = 0.0
        zb = W.stack_bottoms(t, gv)
    m = W.random_unit(rng, (nz, ny, nx))[None]
    g = rng.standard_normal(m.shape)
    plan = hfd.Plan(nx, ny, 1.5, 2.0, t, zb, batch_max=1, flags=hfd.HFD_FP64)
    _, gt = _vjp(plan, m, g, want_m=False)
    ref = oracle.thickness_grad(nx, ny, 1.5, 2.0, zb, t, m[0], g[0])
    assert np.abs(gt[0] - ref).max() < 1e-10 * np.abs(ref).max(), (gt[0], ref)
    plan.destroy()


@pytest.mark.parametrize("store", [False, True], ids=["recompute", "stored"])
def test_thickness_gradient_after_reset_to_fewer_offsets(store):
    """Two stacks; after set_thickness to stacks with fewer distinct interface
    offsets (equal layers) the offset tables keep their allocated stride, and
    every stack's gradient still matches the oracle (FP64)."""
    rng = np.random.default_rng(77)
    nx, ny, nz, G = 6, 5, 3, 2
    flags = hfd.HFD_FP64 | (hfd.HFD_STORE_DTENSOR if store else 0)
    t1 = rng.uniform(0.5, 2.5, (G, nz))
    z1 = np.stack([W.stack_bottoms(t1[g], [0.2, 0.45]) for g in range(G)])
    plan = hfd.Plan(nx, ny, 1.0, 1.5, t1, z1, batch_max=G, flags=flags)
    t2 = np.array([[1.0, 1.0, 1.0], [0.7, 0.7, 0.7]])
    z2 = np.stack([W.stack_bottoms(t2[g], [0.0, 0.0]) for g in range(G)])
    m = np.stack([W.random_unit(rng, (nz, ny, nx)) for _ in range(G)])
    g = rng.standard_normal(m.shape)
    for t, z in ((t1, z1), (t2, z2)):
        if t is t2:
            plan.set_thickness(t, z)
        _, gt = _vjp(plan, m, g, want_m=False)
        for b in range(G):
            ref = oracle.thickness_grad(nx, ny, 1.0, 1.5, z[b], t[b], m[b], g[b])
            assert np.abs(gt[b] - ref).max() < 1e-10 * np.abs(ref).max(), (store, b, gt[b], ref)
    plan.destroy()


@pytest.mark.parametrize("nx, ny", [(1, 1), (1, 9), (40, 1)], ids=["1x1", "1x9", "40x1"])
def test_thickness_gradient_degenerate_lateral_shapes(nx, ny):
    """One cell, one column, one row (8-point padded axes, waves with lanes past
    the ky range, a single kx column besides the packed one), FP64 against the
    oracle, touching and gapped layers."""
    rng = np.random.default_rng(90 + nx + ny)
    nz = 3
    t = rng.uniform(0.5, 2.0, nz)
    zb = W.stack_bottoms(t, [0.0, 0.4])
    m = W.random_unit(rng, (nz, ny, nx))[None]
    g = rng.standard_normal(m.shape)
    plan = hfd.Plan(nx, ny, 1.0, 2.0, t, zb, batch_max=1, flags=hfd.HFD_FP64)
    _, gt = _vjp(plan, m, g, want_m=False)
    ref = oracle.thickness_grad(nx, ny, 1.0, 2.0, zb, t, m[0], g[0])
    assert np.abs(gt[0] - ref).max() < 1e-10 * np.abs(ref).max(), (gt[0], ref)
    plan.destroy()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("nz", [2, 3, 4, 16, 17, 22, 23])
def test_thickness_gradient_group_and_staging_edges(nz, fp64):
    """Layer counts around the groups of three positions and layers and around
    the largest stacks whose spectra are staged in LDS (22 layers in FP32, 16 in
    FP64); columns of more than one ky tile, touching layers and gaps mixed."""
    wl = W.small_case(3, 34, nz, seed=430 + nz)
    plan = plan_for(wl, flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    g = np.random.default_rng(nz).standard_normal(wl.m.shape)
    dt = np.float64 if fp64 else np.float32
    _, gt = _vjp(plan, wl.m, g, want_m=False)
    ref = oracle.thickness_grad(wl.nx, wl.ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0],
                                wl.m[0].astype(dt).astype(np.float64), g[0].astype(dt).astype(np.float64))
    err = np.abs(gt[0] - ref).max() / np.abs(ref).max()
    assert err < (1e-10 if fp64 else 2e-5), err
    plan.destroy()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("nz,B", [(1, 60), (2, 60), (3, 60), (8, 60), (9, 60), (4, 8), (5, 8)])
def test_thickness_gradient_waves_per_tile(nz, B, fp64):
    """Both sides of each line of the waves-per-tile rule: 72 blocks per state,
    so 4320 of them, or 576."""
    wl = W.small_case(33, 3, nz, seed=460 + nz)
    plan = hfd.Plan(wl.nx, wl.ny, wl.dx, wl.dy, wl.thickness[0], wl.z_bottom[0], batch_max=B,
                    flags=hfd.HFD_FP64 if fp64 else hfd.HFD_FP32)
    m = np.stack([np.roll(wl.m[0], b, axis=-1) for b in range(B)])
    g = np.random.default_rng(nz).standard_normal(m.shape)
    dt = np.float64 if fp64 else np.float32
    _, gt = _vjp(plan, m, g, want_m=False)
    for b in (0, B // 2, B - 1):
        ref = oracle.thickness_grad(wl.nx, wl.ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0],
                                    m[b].astype(dt).astype(np.float64), g[b].astype(dt).astype(np.float64))
        err = np.abs(gt[b] - ref).max() / np.abs(ref).max()
        assert err < (1e-10 if fp64 else 2e-5), (b, err)
    plan.destroy()


def test_thickness_gradient_after_reset_to_more_offset_tables():
    """12 stacks that share one offset table (4 different ones, each three times),
    set to 12 unrelated ones: as many offsets per table, but three tables (one
    holds 42 offsets at this size and 4 layers have 11).  The gradients are those
    of a plan created with the second geometry, bit for bit."""
    import torch
    nx = ny = 260
    nz, G = 4, 12
    rng = np.random.default_rng(47)
    t2 = rng.uniform(0.5, 3.0, size=(G, nz))
    t1 = np.repeat(rng.uniform(0.5, 3.0, size=(G // 3, nz)), 3, axis=0)
    m = torch.from_numpy(rng.standard_normal((G, 3, nz, ny, nx)).astype(np.float32)).cuda()
    g = torch.from_numpy(rng.standard_normal((G, 3, nz, ny, nx)).astype(np.float32)).cuda()
    plan = hfd.Plan(nx, ny, 2.0, 2.0, t1, batch_max=G)
    plan.vjp(m, g, want_m=False)
    plan.set_thickness(t2)
    got = plan.vjp(m, g, want_m=False)[1].cpu()
    plan.destroy()
    fresh = hfd.Plan(nx, ny, 2.0, 2.0, t2, batch_max=G)
    ref = fresh.vjp(m, g, want_m=False)[1].cpu()
    fresh.destroy()
    assert torch.isfinite(ref).all()
    assert torch.equal(got, ref)


def test_thickness_gradient_with_long_derivative_rows():
    """42 stacks of 32 layers, whose stored table has 22177 offsets: two rows of it
    (the packed column's) are over 2 GiB and one is not, so that the kernel with a
    descriptor per row takes the call.  Against a plan without the stored table,
    which goes through short tables and the staged kernel; the two differ in the
    order of FP64 sums."""
    import torch
    nx, ny, nz, G = 3, 2048, 32, 42
    rng = np.random.default_rng(48)
    t = rng.uniform(0.5, 3.0, size=(G, nz))
    m = torch.from_numpy(rng.standard_normal((G, 3, nz, ny, nx)).astype(np.float32)).cuda()
    g = torch.from_numpy(rng.standard_normal((G, 3, nz, ny, nx)).astype(np.float32)).cuda()
    gt = []
    for flags in (hfd.HFD_STORE_DTENSOR, hfd.HFD_FP32):
        plan = hfd.Plan(nx, ny, 2.0, 2.0, t, batch_max=G, flags=flags)
        gt.append(plan.vjp(m, g, want_m=False)[1].cpu().numpy())
        plan.destroy()
    assert np.abs(gt[0] - gt[1]).max() < 1e-9 * np.abs(gt[1]).max()
