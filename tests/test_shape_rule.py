"""Host tests of the backprojection's shape rule: what it returns holds the
geometry, leaves the compute unit enough waves wherever the source is, and is
one of the shapes that the GPU parity tests run."""

import math
import random

import pytest

import paper_1708_07515_amd as pkg
from shapes import BATCHES, SHAPES, key, volume


def footprint(n, nz, r, tile, pairs, side=0):
    """Detector columns and rows of a tile times a run of `pairs` slices at the
    worst angle and slice, with the margins of the kernel (two samples)."""
    near = r - (n - 1) / math.sqrt(2.0)
    mag, lat, diag = r / near, (n - 1) / math.sqrt(2.0) / near, (tile - 1) * math.sqrt(2.0)
    per_z, top = (mag, r) if not side else ((near + side * math.sqrt(0.5)) / near, near + side * math.sqrt(0.5))
    rows = (pairs - 1) * per_z + max((nz - 1) / 2.0, 2.0 * pairs) * top * diag / near ** 2
    return math.ceil(diag * mag * math.hypot(1.0, lat) + 0.05) + 2, math.ceil(rows + 0.05) + 2


# Keys (z run, columns, rows) of the footprint of a 16 x 16 block that decide
# whether a plan has a backprojection at all.
KEYS = [(z, w, h) for z in (32, 16) for w in (32, 64) for h in (48, 64)] + [(64, 32, 96)]


def accepted(n, nz, r, side):
    for z in (32, 16, 64):
        near = r - (n - 1) / math.sqrt(2.0)
        mag, lat, diag = r / near, (n - 1) / math.sqrt(2.0) / near, 15 * math.sqrt(2.0)
        per_z, top = (mag, r) if not side else ((near + side * math.sqrt(0.5)) / near, near + side * math.sqrt(0.5))
        cols = diag * mag * math.hypot(1.0, lat)
        rows = (z - 1) * per_z + ((nz - 1) / 2.0 + z) * top * diag / near ** 2
        if max(cols, rows) < 1e6 and any(k[0] == z and math.ceil(cols + 1e-6) + 4 <= k[1]
                                         and math.ceil(rows + 1e-6) + 4 <= k[2] for k in KEYS):
            return z
    return 0


def draws(count, seed):
    rng = random.Random(seed)
    while count:
        n = rng.choice([rng.randint(2, 40), rng.randint(2, 300), rng.randint(300, 2000)])
        r = n * math.exp(rng.uniform(math.log(0.75), math.log(12)))
        s = rng.randint(0, 3)
        if r <= (n - 1) / math.sqrt(2.0) or (1 << s) > n:
            continue
        count -= 1
        yield dict(n=n, p=64, r=r, s=s, nz=max(1, min(65536, int(n * math.exp(rng.uniform(-4, 3))))),
                   rows="cone" if s and rng.random() < 0.3 else "detector")


def test_shapes_hold_what_the_keys_accept():
    for v in draws(6000, 11):
        side = (v["n"] + (1 << v["s"]) - 1) >> v["s"] if v["rows"] == "cone" else 0
        z = accepted(v["n"], v["nz"], v["r"], side)
        try:
            sh = pkg.backproject_shape(v)
        except pkg.FdkodError as e:
            assert e.code == "E_UNSUPPORTED" and not z, v
            continue
        assert sh["z_run"] == z, v
        cols, rows = footprint(v["n"], v["nz"], v["r"], sh["tile"], sh["pairs"], side)
        assert cols <= sh["columns"] and rows <= sh["rows"], (v, sh)
        assert key(sh) in SHAPES, (v, sh)


@pytest.mark.parametrize("ratio", [1.6, 1.75, 2.0, 2.25, 2.5, 2.75])
@pytest.mark.parametrize("n,s", [(64, 2), (100, 0), (128, 3), (160, 3), (200, 0), (200, 3), (500, 1), (500, 3),
                                 (1000, 4)])
def test_close_sources_keep_their_waves(n, s, ratio):
    """A footprint between 32 and 56 columns takes a shape staged little wider,
    so that two workgroups of 16 x 16 tiles (six waves of 8 x 8 ones) fit a
    compute unit: in 64 columns one does, at half the rate or less."""
    v = dict(n=n, p=120, r=ratio * n, s=s)
    for sh in (pkg.backproject_shape(v), pkg.backproject_shape([v, v], batch=True)):
        cols, _ = footprint(n, n, ratio * n, sh["tile"], sh["pairs"])
        assert sh["columns"] < cols + (12 if sh["tile"] == 16 else 8), sh
        assert sh["waves"] >= (2 if sh["tile"] == 16 else 1), sh


def test_every_shape_has_its_geometry():
    for k, spec in SHAPES.items():
        assert key(pkg.backproject_shape(volume(spec), z_run=spec[5])) == k
    for k, spec in BATCHES.items():
        vols = [volume(spec), volume(spec, p=56)]
        assert key(pkg.backproject_shape(vols, batch=True)) == k


def test_arguments():
    with pytest.raises(pkg.FdkodError):
        pkg.backproject_shape(dict(n=64, p=90, r=10.0))
    with pytest.raises(pkg.FdkodError):
        pkg.backproject_shape(dict(n=64, p=90, r=256.0), z_run=8)
    with pytest.raises(pkg.FdkodError):
        pkg.backproject_shape(dict(n=64, p=90, r=60.0))      # a footprint beyond every shape
    lib = pkg.load_library()
    assert lib.fdkod_backproject_shape(None, 1, 0, 0, None) == 1
