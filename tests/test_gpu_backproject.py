"""GPU tests of the backprojection's shapes: slice pairs about the mid-plane,
16 x 16 and 8 x 8 tiles, angle groups, runs that end past the middle, and
slabs that start anywhere, against the FP64 oracle or the whole volume."""

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, gpu_reconstruct, oracle_reconstruct, report, require_gpu, scan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# n, nz, p, r, s, skip: a single slice, one pair, an odd middle, runs of 4 and
# 8 pairs with a remainder, squares of 8, 9, 12 and 24 voxels, fewer angles
# than angle groups and a close source (all small volumes, which take angle
# groups: every shape by name is in test_gpu_backproject_shapes.py)
CASES = [(32, 1, 48, 256.0, 1, 0), (32, 2, 45, 128.0, 2, 0), (33, 7, 3, 132.0, 0, 0), (48, 48, 67, 192.0, 2, 0),
         (72, 33, 64, 288.0, 3, 1), (64, 17, 48, 100.0, 2, 0), (96, 95, 24, 384.0, 2, 1), (64, 64, 16, 256.0, 3, 0),
         (120, 40, 24, 480.0, 0, 0), (192, 61, 20, 768.0, 3, 1)]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_shapes_match_oracle(case):
    n, nz, p, r, s, skip = case
    proj = scan(n, p, r, 6, 300 + n)
    got, _ = gpu_reconstruct(proj, n, p, r, s=s, skip=skip, nz=nz)
    # the FP32 path's bar (rel-RMSE against FP64)
    slices = None if n < 100 else [0, nz // 2, nz - 1]
    ref = oracle_reconstruct(proj, r, s, skip, nz=nz, slices=slices)
    err, _ = report(f"backprojection {case}", got if slices is None else got[slices], ref, bar=1e-4)
    assert err <= 1e-4


@pytest.mark.parametrize("case", [(64, 61, 90, 256.0, 2, "f32"), (192, 45, 20, 768.0, 3, "bf16"), (64, 64, 48, 100.0, 1, "f16")],
                         ids=["small", "tiles8", "close"])
def test_slabs_at_any_slice_match_the_volume(case):
    n, nz, p, r, s, store = case
    proj = scan(n, p, r, 6, 320 + n).to(DEV)
    with pkg.Plan(n, p, r, s=s, nz=nz, store=store) as plan:
        filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
        plan.filter(proj, filt)
        plan.backproject(filt, vol, ws)
        zr = plan.get_tuning()["z_run"]
        for z0, nzs in ((0, 1), (3, 5), (nz // 2 - 2, 5), (nz // 2, 1), (nz - 7, 7), (1, nz - 2), (zr, nz - zr), (0, nz)):
            v0, nr = plan.band_rows(z0, nzs)
            pb, fb, wb = plan.empty_band(nr)
            pb.copy_(proj[:, v0:v0 + nr, :])
            plan.filter_band(pb, v0, fb)
            plan.decompose_band(fb, v0, wb)
            slab = torch.full((nzs, n, n), float("nan"), dtype=torch.float32, device=DEV)
            plan.reconstruct_slab(fb, wb, v0, nr, z0, slab)
            torch.cuda.synchronize()
            want = vol[z0:z0 + nzs]
            if z0 % zr == 0:
                assert torch.equal(slab, want), (z0, nzs)
            # row positions below 64 rounded to 2^-19 move a sample by that
            # part of its neighbour's difference, itself at most twice the
            # largest sample: 4e-6 of max |vol| with random signs over the angles
            assert float((slab - want).abs().max()) <= 1e-5 * float(vol.abs().max()), (z0, nzs)
