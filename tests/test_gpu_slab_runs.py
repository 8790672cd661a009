"""GPU tests of how a slab's runs of slices are dealt out to workgroups: lower
runs and mirrored ones together in one workgroup (a slab about the mid-plane),
an odd number of runs, and one run to a workgroup where there are few."""

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, require_gpu, scan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# 576 tiles (two runs to a workgroup) and 64 (one); nz odd and even
@pytest.mark.parametrize("n,nz,s", [(264, 90, 3), (264, 91, 3), (97, 81, 2)])
def test_runs_match_the_volume(n, nz, s):
    p, r = 24, 4.0 * n
    proj = scan(n, p, r, 6, 700 + n).to(DEV)
    with pkg.Plan(n, p, r, s=s, skip=s - 1, nz=nz) as plan:
        filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
        plan.filter(proj, filt)
        plan.backproject(filt, vol, ws)
        zr = plan.get_tuning()["z_run"]
        mid = nz // 2
        # one run of each side, two and one, many, a single slice on either side
        for z0, nzs in ((mid - 8, 16), (mid - 16, 32), (mid - 24, 33), (mid - 3, 20), (mid - 1, 2), (mid, 1), (zr, 40), (0, nz)):
            v0, nr = plan.band_rows(z0, nzs)
            _, fb, wb = plan.empty_band(nr)
            fb.copy_(filt[:, v0:v0 + nr])
            plan.decompose_band(fb, v0, wb)
            slab = torch.full((nzs, n, n), float("nan"), dtype=torch.float32, device=DEV)
            plan.reconstruct_slab(fb, wb, v0, nr, z0, slab)
            torch.cuda.synchronize()
            want = vol[z0:z0 + nzs]
            if z0 % zr == 0:
                assert torch.equal(slab, want), (z0, nzs)
            # row positions below 512 rounded to 2^-16: a sample moves by that
            # part of its neighbour's difference, at most twice the largest
            assert float((slab - want).abs().max()) <= 2e-5 * float(vol.abs().max()), (z0, nzs)


def test_thin_slabs_take_short_runs():
    """A volume in runs of 16 pairs: thin slabs that start their own runs may
    take the kernel of 8, slabs at the z run take the volume's bits."""
    n, nz, p, r, s = 144, 50, 24, 1.6 * 144, 3
    assert pkg.backproject_shape(dict(n=n, nz=nz, p=p, r=r, s=s, skip=2))["pairs"] == 16
    proj = scan(n, p, r, 6, 41).to(DEV)
    with pkg.Plan(n, p, r, s=s, skip=2, nz=nz) as plan:
        filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
        plan.filter(proj, filt)
        plan.backproject(filt, vol, ws)
        zr = plan.get_tuning()["z_run"]
        for z0, nzs in ((19, 11), (23, 2), (1, 7), (1, 49), (26, 9), (2, 16), (0, 7), (zr, 5)):
            v0, nr = plan.band_rows(z0, nzs)
            _, fb, wb = plan.empty_band(nr)
            fb.copy_(filt[:, v0:v0 + nr])
            plan.decompose_band(fb, v0, wb)
            slab = torch.full((nzs, n, n), float("nan"), dtype=torch.float32, device=DEV)
            plan.reconstruct_slab(fb, wb, v0, nr, z0, slab)
            torch.cuda.synchronize()
            want = vol[z0:z0 + nzs]
            if z0 % zr == 0:
                assert torch.equal(slab, want), (z0, nzs)
            assert float((slab - want).abs().max()) <= 2e-5 * float(vol.abs().max()), (z0, nzs)
