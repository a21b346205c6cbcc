"""Five-pass mixing of many layers in whole blocks, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1910_07054_amd import hfd
from paper_1910_07054_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hfd.load()


# FP32 mixing above 32 layers (four target layers per wave) with 512 tiles or more,
# so that a block owns its tile: 9 to 16 waves paced by barriers, results in place,
# the packed column's second sweep; full and partly filled last groups (33, 50), one
# and two ky tiles per column
@pytest.mark.parametrize("nz,ny,B", [(33, 20, 64), (36, 40, 32), (48, 20, 65), (50, 40, 33), (64, 20, 64), (64, 34, 32)])
def test_wide_mixing_in_whole_blocks(nz, ny, B):
    import torch
    nx = 5
    Ly = 8
    while Ly < 2 * ny:
        Ly *= 2
    assert (Ly // 2 + 31) // 32 * 8 * B >= 512
    wl = W.small_case(nx, ny, nz, seed=2000 + nz)
    m = np.stack([np.roll(wl.m[0], b, axis=-2) for b in range(B)]).astype(np.float32)
    plan = hfd.Plan(nx, ny, wl.dx, wl.dy, wl.thickness[0], wl.z_bottom[0], batch_max=B, flags=hfd.HFD_SPLIT_PASSES)
    md = torch.from_numpy(m).cuda()
    h = plan.field(md).cpu().numpy()
    gm = plan.vjp(None, md, want_t=False)[0].cpu().numpy()
    plan.destroy()
    rng = np.random.default_rng(nz)
    smp = np.stack([rng.integers(0, nz, 40), rng.integers(0, ny, 40), rng.integers(0, nx, 40)], axis=1)
    smp[0], smp[1] = (0, 0, 0), (nz - 1, ny - 1, nx - 1)
    for b in (0, B - 1):
        for got, transpose in ((h, False), (gm, True)):
            ref = oracle.field(nx, ny, wl.dx, wl.dy, wl.z_bottom[0], wl.thickness[0], m[b].astype(np.float64),
                               samples=smp, transpose=transpose)
            val = got[b][:, smp[:, 0], smp[:, 1], smp[:, 2]].T
            err = np.abs(val - ref).max() / np.linalg.norm(ref, axis=1).max()
            assert err < 1e-5, (b, transpose, err)
