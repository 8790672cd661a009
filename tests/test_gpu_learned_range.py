"""GPU test of the learned gradient over the range of its FP32 input: the
kernel splits dR into BF16 parts, and a gradient is linear in dR, so scaling dR
by a power of two scales every bit of it, up to the largest floats."""

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# the row-reusing form (D = 4 divides P) and the general one
@pytest.mark.parametrize("p", [48, 50])
@pytest.mark.parametrize("interp", ["linear", "cubic"])
def test_gradient_scales_with_its_input(p, interp):
    with pkg.Plan(32, p, 128.0, s=2, interp=interp) as plan:
        g = torch.Generator().manual_seed(p)
        filt = (0.1 * torch.randn(plan.p, 32, 32, generator=g)).to(DEV)
        weights = (0.05 * torch.randn(pkg.LEARNED_PARAMS, generator=g)).to(torch.bfloat16).to(DEV)
        at = plan.workspace_elems // 3 + torch.arange(4) * 97
        # the largest float (BF16's rounding would carry it to infinity), 24 bits set, few bits, a negative
        value = torch.tensor([3.4028234663852886e38, 2.0 ** 127 * 1.9999998807907104, 2.0 ** 126, -3.4e38])

        def grad(i, scale):
            dws = torch.zeros(plan.workspace_elems)
            dws[at[i]] = value[i] * scale
            out = torch.empty(pkg.LEARNED_PARAMS, device=DEV)
            plan.learned_backward(filt, dws.to(DEV), weights, out)
            torch.cuda.synchronize()
            return out

        for i in range(4):
            want = grad(i, 2.0 ** -60)
            assert torch.isfinite(want).all() and want.abs().sum() > 0
            for e in (-20, 0):
                got = grad(i, 2.0 ** e)
                assert torch.equal(got, want * 2.0 ** (60 + e)), (i, e)
