"""Segments of the decimated angles add the same projections in the same order
as a walk over all of them: a band of a few rows, whose decimation is cut into
segments, gives the bits of a whole volume's, which fills the chip uncut -- for
every window and shift (with more windows open a segment starts further back).
Cone-corrected rows have no bands: their chunk counts change the tasks, and so
the segments."""

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, require_gpu, scan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _rows(plan, ws, nrows, v0, nr):
    """Rows [v0, v0 + nr) of every square, of a workspace of nrows rows."""
    out, at = [], 0
    for w in plan.get_bounds()["width"].tolist():
        size = plan.p_dec * nrows * w
        out.append(ws[at:at + size].view(plan.p_dec, nrows, w)[:, v0:v0 + nr].contiguous())
        at += size
    return out


# 64 squares x 256 rows fill the chip with every window; 45 decimated angles
@pytest.mark.parametrize("knobs", [{}, dict(store="bf16"), dict(decim="sinc", taps=2), dict(decim="sinc", taps=4),
                                   dict(decim="sinc", taps=6), dict(interp="cubic"),
                                   dict(decim="sinc", taps=6, interp="cubic", store="f16")],
                         ids=lambda k: "-".join(str(v) for v in k.values()) or "plain")
def test_band_equals_uncut_volume(knobs):
    n, p, s = 256, 360, 3
    filt = torch.randn((p, n, n), generator=torch.Generator().manual_seed(3)).to(DEV)
    with pkg.Plan(n, p, 4.0 * n, s=s, **knobs) as plan:
        filt = filt.to(plan.store_torch_dtype())
        ws = plan.empty_workspace()
        plan.decompose(filt, ws)
        typed = ws[:plan.workspace_bytes].view(plan.store_torch_dtype())
        for v0, nr in ((0, 2), (6, 5), (100, 16), (222, 34)):
            fb = filt[:, v0:v0 + nr].contiguous()
            wb = torch.full((plan.band_workspace_elems(nr),), 7.0, dtype=fb.dtype, device=DEV)
            plan.decompose_band(fb, v0, wb)
            torch.cuda.synchronize()
            for a, b in zip(_rows(plan, typed, n, v0, nr), _rows(plan, wb, nr, 0, nr)):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (v0, nr)


# one chunk's 2048 and more tasks uncut, four chunks' in two segments
@pytest.mark.parametrize("knobs", [dict(rows="cone"), dict(rows="cone", decim="sinc", taps=6),
                                   dict(rows="cone", decim="sinc", taps=4, interp="cubic")],
                         ids=lambda k: "-".join(str(v) for v in k.values()))
@pytest.mark.parametrize("n,s", [(300, 1), (96, 2)])
def test_chunks_of_cone_rows(n, s, knobs):
    p = 128
    filt = torch.randn((p, n, n), generator=torch.Generator().manual_seed(4)).to(DEV)
    with pkg.Plan(n, p, 4.0 * n, s=s, **knobs) as plan:
        outs = []
        for c in (1, 2, 4):
            plan.set_tuning(decim_chunks=c)
            ws = plan.empty_workspace()
            ws.fill_(7)
            plan.decompose(filt, ws)
            torch.cuda.synchronize()
            outs.append(ws[:plan.workspace_bytes])
        assert all(torch.equal(outs[0], o) for o in outs[1:])


# widths on both sides of the pieces' limits, every count of rows per wave
@pytest.mark.parametrize("n,p,s,store", [(37, 48, 3, "f32"), (41, 48, 3, "f32"), (100, 140, 3, "f32"), (100, 140, 2, "bf16"),
                                         (154, 64, 2, "f32"), (298, 48, 3, "f16"), (512, 80, 5, "f32")])
def test_one_chunk_equals_more(n, p, s, store):
    filt = torch.randn((p, n, n), generator=torch.Generator().manual_seed(5)).to(DEV)
    with pkg.Plan(n, p, 4.0 * n, s=s, store=store) as plan:
        filt = filt.to(plan.store_torch_dtype())
        outs = []
        for c in (1, 2):
            plan.set_tuning(decim_chunks=c)
            ws = plan.empty_workspace()
            ws.fill_(7)
            plan.decompose(filt, ws)
            torch.cuda.synchronize()
            outs.append(ws[:plan.workspace_bytes])
        assert torch.equal(*outs)
