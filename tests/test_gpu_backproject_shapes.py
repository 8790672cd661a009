"""GPU parity of every backprojection kernel shape, each case with the shape it
runs asserted: the whole volume against the FP64 oracle, slabs against the
volume, a batch against the plans of its volumes, and the checked build's
footprint counters."""

import json
import os
import subprocess
import sys

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, log, oracle_reconstruct, report, require_gpu, scan
from shapes import BATCHES, SHAPES, key, volume

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _open(spec, store="f32"):
    plan = pkg.Plan(**volume(spec), store=store)
    if spec[5]:
        plan.set_tuning(z_run=spec[5], tile_w=64, tile_h=64)
    return plan


@pytest.mark.parametrize("shape", sorted(SHAPES), ids=lambda k: "-".join(map(str, k)))
def test_shape(shape):
    spec = SHAPES[shape]
    n, nz, ratio, s, skip, zr = spec
    assert key(pkg.backproject_shape(volume(spec), z_run=zr)) == shape
    p = volume(spec)["p"]
    proj = scan(n, p, ratio * n, 6, 500 + n)
    with _open(spec) as plan:
        filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
        plan.filter(proj.to(DEV), filt)
        plan.backproject(filt, vol, ws)
        zrun = plan.get_tuning()["z_run"]
        # slabs: at the z run (the volume's bits), about the mid-plane, at the end
        cuts = [(z0, c) for z0, c in ((0, min(nz, 2 * zrun)), (nz // 2 - 3, 7), (max(0, nz - 5), min(nz, 5)),
                                      (nz // 2 - nz % 2, 1), (zrun, nz - zrun)) if z0 >= 0 and c > 0]
        for z0, c in cuts:
            v0, nr = plan.band_rows(z0, c)
            if not nr:          # a tall volume's end: no detector row reaches it
                assert not vol[z0:z0 + c].any()
                continue
            _, fb, wb = plan.empty_band(nr)
            fb.copy_(filt[:, v0:v0 + nr])
            plan.decompose_band(fb, v0, wb)
            slab = torch.full((c, n, n), float("nan"), dtype=torch.float32, device=DEV)
            plan.reconstruct_slab(fb, wb, v0, nr, z0, slab)
            torch.cuda.synchronize()
            if z0 % zrun == 0:
                assert torch.equal(slab, vol[z0:z0 + c]), (z0, c)
            # row positions below 512 rounded to 2^-16 move a sample by that part
            # of its neighbour's difference, itself at most twice the largest
            # sample, with random signs over the angles
            assert float((slab - vol[z0:z0 + c]).abs().max()) <= 2e-5 * float(vol.abs().max()), (z0, c)
        got = vol.cpu().double().numpy()
    slices = sorted({0, nz // 3, (nz - 1) // 2, nz // 2, nz - 1})
    ref = oracle_reconstruct(proj, ratio * n, s, skip, nz=nz, slices=slices)
    # the FP32 path's bar (rel-RMSE against FP64)
    err, _ = report(f"backprojection shape {shape}", got[slices], ref, bar=1e-4)
    assert err <= 1e-4


@pytest.mark.parametrize("shape", sorted(BATCHES), ids=lambda k: "-".join(map(str, k)))
def test_batch_shape(shape):
    spec = BATCHES[shape]
    vols = [volume(spec), volume(spec, p=56)]
    assert key(pkg.backproject_shape(vols, batch=True)) == shape
    with pkg.Batch(vols, store="f16") as b:
        proj = [scan(v["n"], v["p"], v["r"], 6, 600 + i).to(DEV) for i, v in enumerate(vols)]
        filt = [pl.empty_filtered() for pl in b.plans]
        ws = [pl.empty_workspace() if pl.s else None for pl in b.plans]
        vol = [pl.empty_volume() for pl in b.plans]
        b.bind(proj, filt, ws, vol)
        b.run()
        torch.cuda.synchronize()
        for v, f, w, got in zip(vols, filt, ws, vol):
            with pkg.Plan(**v, store="f16") as plan:
                want = plan.empty_volume()
                plan.reconstruct(f, w, want)
                torch.cuda.synchronize()
                # the same data; coordinates round as in test_shape, the
                # angles' sums as FP32 sums of at most 40 terms do
                assert float((got - want).abs().max()) <= 2e-5 * float(want.abs().max())


def test_checked_build_counts_no_events():
    checked = os.path.join(os.path.dirname(HERE), "paper_1708_07515_amd", "libfdkod_checked.so")
    assert os.path.exists(checked), "libfdkod_checked.so is missing: build with __graft_entry__.build()"
    out = subprocess.run([sys.executable, "-u", os.path.join(HERE, "checked_shapes.py")],
                         env=dict(os.environ, FDKOD_LIB=checked), stdout=subprocess.PIPE, stderr=subprocess.PIPE,
                         timeout=110, text=True)
    log(out.stdout)
    assert out.returncode == 0, out.stderr[-2000:]
    lines = [json.loads(x) for x in out.stdout.splitlines() if x.startswith("{")]
    assert len(lines) == len(SHAPES)
    for rec in lines:
        assert rec["counts"] == [0, 0, 0, 0], rec
