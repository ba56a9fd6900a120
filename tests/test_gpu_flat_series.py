"""The flat-sky map where a tile's far segments act through power series: tile
edges and remainders, one series, two and none, against the oracle on sampled
pixels.  A far segment's terms come from FP64 sums of FP32 weights (2^-24
each) and leave out 5e-10; a near one's come from some ten FP32 operations of
2^-24 each: 1e-6 of the map's rms bounds the rms error."""
import math

import numpy as np
import pytest

import oracle
import synth
from helpers import err_metrics

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def render(fp):
    from paper_1204_5041_amd import binding as B
    sky = B.Sky(64, fp.eta0, B.CSMAP_FORM_FP32C)
    for bx in fp.boxes:
        t = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
             for a in (bx.x_rel, bx.xdot, bx.xprime, bx.dsigma)]
        sky.add_box(*t, origin=tuple(bx.origin), eta_lo=bx.eta_lo, eta_hi=bx.eta_hi)
    got = sky.render_flat(fp.center, fp.e1, fp.e2, fp.nx, fp.ny, fp.pix,
                          fp.accept_cos).cpu().numpy()
    sky.close()
    return got


@pytest.mark.parametrize("nx,ny,nseg", [
    (32, 32, 3000),        # one tile, every segment near
    (33, 31, 70_000),      # a remainder of one pixel
    (300, 1, 4001),        # one row, below and above the pairs that pay for a series
    (300, 1, 300),
    (129, 65, 20_000),     # one series
    (640, 600, 90_000),    # two series, ragged at both tile sizes
    (1500, 45, 300_001),   # two series, one row of coarse tiles
])
def test_series_match_oracle(nx, ny, nseg):
    fp = synth.flat_pencil(nseg, 64, seed=nx + ny)
    fp.nx, fp.ny, fp.pix = nx, ny, math.radians(7.2) / max(nx, ny)
    got = render(fp)
    rng = np.random.default_rng(nx)
    edge = np.array([0, 15, 16, 31, 32, 63, 127, 128, 255, 256, nx - 1])
    ii = np.concatenate([np.minimum(edge, nx - 1), rng.integers(0, nx, 300)])
    jj = np.concatenate([np.minimum(edge[::-1], ny - 1), rng.integers(0, ny, 300)])
    t = np.stack([(ii + 0.5 - nx / 2) * fp.pix, (jj + 0.5 - ny / 2) * fp.pix], 1)
    ref = oracle.flat_points(t, fp.frame, fp.accept_cos, fp.eta0, fp.boxes)
    e = err_metrics(got[jj, ii], ref)
    print(nx, ny, nseg, e, flush=True)
    assert e["rel_rms"] <= 1e-6 and e["rel_max"] <= 1e-4, e


def test_weights_that_are_not_finite_reach_every_pixel():
    fp = synth.flat_pencil(40_000, 64, seed=5)
    fp.nx, fp.ny, fp.pix = 200, 200, math.radians(7.2) / 200
    base = render(fp)
    assert np.isfinite(base).all()
    fp.boxes[0].dsigma[:50] = np.inf
    assert not np.isfinite(render(fp)).any()
