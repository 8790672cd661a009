"""The filter of short rows (several row pairs per wave, one buffer range over a
workgroup's rows, the transform's lower half only) at the edges of its
transform lengths, against the FP64 oracle; bands with an odd number of rows,
whose last pair is one row, against the whole detector bit for bit, with the
memory behind the band untouched."""

import numpy as np
import pytest
import torch

import paper_1708_07515_amd as pkg
from oracle import fdk as ofdk
from gpu_common import DEV, report, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _proj(p, rows, n, seed):
    return torch.from_numpy(np.random.default_rng(seed).uniform(0.0, 1.0, (p, rows, n)).astype(np.float32))


# M / 2 and M / 2 + 1 for every short transform length, and odd counts of pairs
@pytest.mark.parametrize("n", [2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 257])
def test_short_rows_match_oracle(n):
    p, r = 3, 4.0 * n
    proj = _proj(p, n, n, n)
    with pkg.Plan(n, p, r, s=0) as plan:
        filt = plan.empty_filtered()
        plan.filter(proj.to(DEV), filt)
        torch.cuda.synchronize()
        got = filt.cpu().double().numpy()
    ref = ofdk.filter_rows(proj.numpy(), r, np.arange(n)).data
    err, mxr = report(f"filter n={n}", got, ref)
    # the pre-weighted row is rounded (2 u relative) before a filter of gain
    # below 1, and the transform adds 4 log2(M) u of the result
    u = 2.0 ** -24
    pw = proj.numpy().astype(np.float64) * ofdk.cosine_weight(n, r)[None]
    m = max(8, 1 << int(np.ceil(np.log2(2 * n - 1))))
    bound = u * (2.0 * np.linalg.norm(pw) / np.linalg.norm(ref) + 4 * np.log2(m))
    assert err <= bound and mxr <= 4 * bound


@pytest.mark.parametrize("n,v0,rows", [(16, 2, 1), (33, 4, 7), (64, 0, 63), (100, 10, 21), (200, 8, 5), (300, 6, 3)])
@pytest.mark.parametrize("store", ["f32", "bf16"])
def test_band_of_odd_rows(n, v0, rows, store):
    p = 5
    proj = _proj(p, n, n, n + rows).to(DEV)
    with pkg.Plan(n, p, 4.0 * n, s=0, store=store) as plan:
        full = plan.empty_filtered()
        plan.filter(proj, full)
        band = proj[:, v0:v0 + rows].contiguous()
        buf = torch.full((p * rows * n + 4096,), 7.0, dtype=full.dtype, device=DEV)
        plan.filter_band(band, v0, buf[:p * rows * n].view(p, rows, n))
        torch.cuda.synchronize()
        want = full[:, v0:v0 + rows]
        if rows % 2:    # the band's last row is alone in its transform: not the same rounding as beside a row
            want, got = want[:, :rows - 1], buf[:p * rows * n].view(p, rows, n)[:, :rows - 1]
        assert torch.equal(got, want)
        last = buf[:p * rows * n].view(p, rows, n)[:, -1].double()
        ref = full[:, v0 + rows - 1].double()
        eps = 2.0 ** -8 if store == "bf16" else 2.0 ** -18
        assert (last - ref).norm() <= eps * full.double().norm() / np.sqrt(n)
        assert bool((buf[p * rows * n:] == 7.0).all())
