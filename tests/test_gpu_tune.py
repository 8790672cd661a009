"""GPU tests of the tuner's choice where several keys run one kernel: the
plan's own key stays, whatever the timings' noise, and so does what follows
from it (the slabs of a streamed reconstruction, the cache file's line)."""

import pytest
import torch

import paper_1708_07515_amd as pkg
from gpu_common import DEV, oracle_reconstruct, report, require_gpu, scan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# every z run takes one shape (small volumes, in angle groups); squares too
# narrow for the row-staged decimation, whose chunk count 0 means 1
@pytest.mark.parametrize("n,r,s", [(64, 512.0, 2), (48, 192.0, 1)])
def test_one_kernel_keeps_the_key(n, r, s, tmp_path, monkeypatch):
    assert len({tuple(v for k, v in pkg.backproject_shape(dict(n=n, p=90, r=r, s=s), z_run=z).items() if k != "z_run")
                for z in (16, 32)}) == 1
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("FDKOD_TUNE_CACHE", str(cache))
    proj = scan(n, 90, r, 6, 900 + n).to(DEV)
    with pkg.Plan(n, 90, r, s=s) as plan:
        want = plan.get_tuning()
        nbytes = plan.streamed_bytes(20)
        filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
        plan.filter(proj, filt)
        for _ in range(6):
            got = plan.tune(filt, ws, vol)
            for k in ("z_run", "tile_w", "tile_h", "angles_per_stage"):
                assert got[k] == want[k]
            assert plan.streamed_bytes(20) == nbytes
    assert len({line.rsplit(" ", 1)[0] for line in cache.read_text().splitlines()}) == 1


def test_distinct_kernels_are_all_tried_and_right():
    """Enough waves for kernels without angle groups: runs of 16 and of 32
    slices differ, each against the oracle, and the tuner returns one of them."""
    n, p, r, s = 200, 24, 800.0, 3
    shapes = {z: tuple(pkg.backproject_shape(dict(n=n, p=p, r=r, s=s, skip=2), z_run=z)[k] for k in ("tile", "pairs"))
              for z in (16, 32, 64)}
    assert shapes[16] != shapes[32] == shapes[64]
    proj = scan(n, p, r, 6, 77)
    slices = [0, 70, 99, 100, 199]
    ref = oracle_reconstruct(proj, r, s, 2, slices=slices)
    with pkg.Plan(n, p, r, s=s, skip=2) as plan:
        filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
        plan.filter(proj.to(DEV), filt)
        for z, th in ((16, 48), (32, 64), (64, 96)):
            plan.set_tuning(z_run=z, tile_w=32, tile_h=th, angles_per_stage=1)
            plan.backproject(filt, vol, ws)
            torch.cuda.synchronize()
            err, _ = report(f"z run {z}", vol[slices].double().cpu().numpy(), ref, bar=1e-4)
            assert err <= 1e-4
        assert plan.tune(filt, ws, vol)["z_run"] in (16, 64)      # 32 runs the current key's kernel


def test_batch_keeps_its_key():
    vols = [dict(n=64, p=90, r=256.0, s=2), dict(n=48, p=67, r=192.0, s=1)]
    with pkg.Batch(vols) as b:
        proj = [scan(v["n"], v["p"], v["r"], 6, i).to(DEV) for i, v in enumerate(vols)]
        b.bind(proj, [q.empty_filtered() for q in b.plans], [q.empty_workspace() for q in b.plans],
               [q.empty_volume() for q in b.plans])
        one = len({tuple(v for k, v in pkg.backproject_shape(vols, batch=True, z_run=z).items() if k != "z_run")
                   for z in (16, 32)}) == 1
        got = [b.tune()["z_run"] for _ in range(4)]
        assert not one or set(got) == {32}
