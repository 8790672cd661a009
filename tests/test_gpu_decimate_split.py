"""The ways the decimation kernel splits a plan's work -- rows packed side by
side into a wave, pieces of wide squares' columns, one to eight column chunks,
segments of the decimated angles, row groups that end inside a task, a band of
rows, a batch's tasks -- add the same samples with the same weights in the same
order, so the decimated sub-sinograms must be bitwise equal whatever the split.
Covers widths on both sides of the splits' limits, odd sizes, the three storage
types, cone-corrected rows, the windowed sinc and the cubic shift."""

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, log, require_gpu, scan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# n, p, r, s, k, store, knobs
CASES = [
    (8, 11, 32.0, 1, 0, "f32", {}),                                        # a few lanes, few windows
    (17, 23, 40.0, 2, 2, "bf16", {}),                                      # eight rows side by side, ragged
    (33, 40, 70.0, 1, 0, "f32", {}),
    (64, 90, 256.0, 3, 0, "f16", {}),
    (96, 128, 384.0, 2, 0, "f32", {}),                                     # three pieces of 15
    (120, 160, 480.0, 2, 1, "f32", {}),                                    # near the 63-column limit
    (131, 150, 524.0, 2, 0, "bf16", {}),
    (101, 136, 202.0, 3, 0, "f16", dict(rows="cone")),
    (90, 120, 360.0, 2, 0, "f32", dict(decim="sinc", taps=6, rows="cone", interp="cubic")),
    (75, 100, 300.0, 1, 0, "f32", dict(interp="cubic")),                   # 58 columns: near the cubic limit
    (193, 220, 772.0, 2, 0, "f32", dict(decim="sinc", taps=4, interp="cubic")),
]


def _close_bits(a, b):
    return torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("case", CASES)
def test_splits_equal(case):
    n, p, r, s, k, store, knobs = case
    proj = scan(n, p, r, 6, n).to(DEV)
    with pkg.Plan(n, p, r, s=s, skip=k, store=store, **knobs) as plan:
        filt = plan.empty_filtered()
        plan.filter(proj, filt)
        default = plan.get_tuning()["decim_chunks"]
        e = plan.workspace_bytes

        def run(c):
            plan.set_tuning(decim_chunks=c)
            ws = plan.empty_workspace()
            ws.fill_(7)
            plan.decompose(filt, ws)
            torch.cuda.synchronize()
            return ws[:e]

        base = run(default)
        log(f"decimation split {case}: max width {plan.info.max_width}, default {default}")
        for c in (1, 2, 4, 8):
            if c == 8 and knobs.get("taps", 2) > 2:
                continue
            assert _close_bits(base, run(c)), c


@pytest.mark.parametrize("n,p,s,z0,nzs", [(64, 90, 3, 20, 9), (96, 120, 2, 0, 5), (40, 57, 2, 33, 7)])
def test_band_equals_full(n, p, s, z0, nzs):
    r = 4.0 * n
    proj = scan(n, p, r, 6, n + 1).to(DEV)
    with pkg.Plan(n, p, r, s=s) as plan:
        filt = plan.empty_filtered()
        plan.filter(proj, filt)
        ws = plan.empty_workspace()
        plan.decompose(filt, ws)
        v0, nrows = plan.band_rows(z0, nzs)
        _, fb, wb = plan.empty_band(nrows)
        fb.copy_(filt[:, v0:v0 + nrows])
        wb.fill_(7)
        plan.decompose_band(fb, v0, wb)
        torch.cuda.synchronize()
        full, band = ws.view(torch.float32), wb.view(torch.float32)
        pd = plan.p_dec
        at_f = at_b = 0
        for w in plan.get_bounds()["width"].tolist():
            f = full[at_f:at_f + pd * n * w].view(pd, n, w)[:, v0:v0 + nrows]
            b = band[at_b:at_b + pd * nrows * w].view(pd, nrows, w)
            assert torch.equal(f, b)
            at_f += pd * n * w
            at_b += pd * nrows * w


def test_batch_equals_single():
    vols = [dict(n=32, p=45, r=128.0, s=2), dict(n=49, p=67, r=196.0, s=2), dict(n=64, p=90, r=256.0, s=3),
            dict(n=150, p=96, r=600.0, s=1)]
    with pkg.Batch(vols, store="bf16") as b:
        proj = [scan(v["n"], v["p"], v["r"], 6, i).to(DEV) for i, v in enumerate(vols)]
        filt = [pl.empty_filtered() for pl in b.plans]
        ws = [pl.empty_workspace() for pl in b.plans]
        b.bind(proj, filt, ws, [pl.empty_volume() for pl in b.plans])
        b.run()
        torch.cuda.synchronize()
        for v, f, w in zip(vols, filt, ws):
            with pkg.Plan(**v, store="bf16") as plan:
                one = plan.empty_workspace()
                plan.decompose(f, one)
                torch.cuda.synchronize()
                e = plan.workspace_bytes
                assert _close_bits(w[:e], one[:e]), v


@pytest.mark.parametrize("store,wide", [("f32", ()), ("bf16", ()), ("f16", (150, 52, 600.0, 1)),
                                        ("f32", (298, 20, 1192.0, 1)), ("bf16", (340, 20, 1360.0, 1))])
def test_large_batch_equals_single(store, wide):
    """Batches of at least 4096 tasks, whose lanes take four rows of a narrow
    volume each, alone and beside a volume of two, four or eight column chunks."""
    vols = [dict(n=n, p=72, r=4.0 * n, s=4) for n in (65, 96, 99, 131)]
    if wide:
        n, p, r, s = wide
        vols.insert(2, dict(n=n, p=p, r=r, s=s))
    with pkg.Batch(vols, store=store) as b:
        filt, ws = [], []
        for i, pl in enumerate(b.plans):
            g = torch.Generator().manual_seed(40 + i)
            f = torch.randn(pl.empty_filtered().shape, generator=g).to(pl.store_torch_dtype())
            filt.append(f.to(DEV))
            ws.append(pl.empty_workspace())
        proj = [torch.zeros((pl.p, pl.n, pl.n), device=DEV) for pl in b.plans]
        b.bind(proj, filt, ws, [pl.empty_volume() for pl in b.plans])
        b.run()
        torch.cuda.synchronize()
        for v, f, w in zip(vols, filt, ws):
            with pkg.Plan(**v, store=store) as plan:
                one = plan.empty_workspace()
                plan.decompose(f, one)
                torch.cuda.synchronize()
                e = plan.workspace_bytes
                assert torch.equal(w[:e], one[:e]), v
