"""Reconstructions of every backprojection shape's geometry under the checked
build of the library (loaded through FDKOD_LIB, in a process of its own): the
kernels' event counters after each whole volume and slab.  Prints one JSON
line per shape."""

import json
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(HERE))
sys.path.insert(0, HERE)

import torch  # noqa: E402

import paper_1708_07515_amd as pkg  # noqa: E402
from shapes import SHAPES, volume  # noqa: E402


def main():
    dev = "cuda:0"
    pkg.check_counts(reset=True)
    for shape, spec in sorted(SHAPES.items()):
        v = volume(spec)
        proj = torch.randn((v["p"], v["n"], v["n"]), generator=torch.Generator().manual_seed(1))
        with pkg.Plan(**v) as plan:
            if spec[5]:
                plan.set_tuning(z_run=spec[5], tile_w=64, tile_h=64)
            filt, ws, vol = plan.empty_filtered(), plan.empty_workspace(), plan.empty_volume()
            plan.filter(proj.to(dev), filt)
            plan.backproject(filt, vol, ws)
            z0, c = v["nz"] // 2 - 3, 7
            v0, nr = plan.band_rows(z0, c)
            _, fb, wb = plan.empty_band(nr)
            fb.copy_(filt[:, v0:v0 + nr])
            plan.decompose_band(fb, v0, wb)
            plan.reconstruct_slab(fb, wb, v0, nr, z0, torch.empty((c, v["n"], v["n"]), device=dev))
            torch.cuda.synchronize()
        print(json.dumps({"shape": list(shape), "counts": pkg.check_counts(reset=True)}), flush=True)


if __name__ == "__main__":
    main()
