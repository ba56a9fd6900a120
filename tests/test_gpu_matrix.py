"""The matrix-core forward kernel (FP32C, default shape,
Nside >= 64, Nside x segments >= 65536) against
the FP64 oracle on sampled pixels, at the sizes where its blocks and tiles end
and for segments that leave its fast path.  Bars of the FP32C form: rel-rms
1e-5, rel-max 1e-4, pair counts exact."""
import numpy as np
import pytest

import oracle
import synth
from helpers import err_metrics, sky_from_workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    from paper_1204_5041_amd import binding
    assert torch.cuda.is_available()
    return binding


def check(B, w, options=None, count=4000, replays=1):
    pix = np.unique(np.concatenate([synth.sample_pixels(w.npix, count, 5), np.arange(64),
                                    np.arange(w.npix - 64, w.npix)]))
    ref = oracle.theta_pixels(w.nside, pix, w.eta0, w.boxes)
    pairs = 0
    every = np.arange(w.npix)
    for b in w.boxes:
        if b.n:
            pairs += int(oracle.visible(w.nside, every, w.eta0, b).sum()) * \
                int(oracle.kept(w.eta0, b).sum())
    sky = sky_from_workload(w, B.CSMAP_FORM_FP32C, options)
    for _ in range(replays):
        got = sky.render().cpu().numpy()
        st = sky.stats()
        e = err_metrics(got[pix], ref)
        print(e, st["steps"], st["near_steps"], flush=True)
        assert st["pairs"] == pairs
        assert e["rel_rms"] <= 1e-5 and e["rel_max"] <= 1e-4, e
    sky.close()
    return st


def boxes_of(sizes, seed=940):
    dirs = synth.uniform_directions(len(sizes), seed)
    return [synth.make_box(n, seed + 1 + b, origin=1.5 * dirs[b] - 0.5, eta_lo=0.0, eta_hi=16.0,
                           dtype=np.float32) for b, n in enumerate(sizes)]


@pytest.mark.parametrize("sizes", [[1], [16, 0, 17], [63, 64, 65], [127, 129, 15], [1000]])
def test_ragged_blocks(B, sizes):
    # a box of 600 segments beside them, so that the launch takes this kernel
    check(B, synth.Workload("m", 128, 16.0, boxes_of(sizes + [600])))


@pytest.mark.parametrize("schedule", [0, 1, 2])
@pytest.mark.parametrize("tiling,rings", [(1, 0), (2, 0), (2, 1), (2, 2), (2, 64)])
def test_tilings(B, schedule, tiling, rings):
    w = synth.Workload("m", 85, 16.0, boxes_of([700, 90]))
    check(B, w, {B.CSMAP_OPT_SCHEDULE: schedule, B.CSMAP_OPT_TILING: tiling,
                 B.CSMAP_OPT_BLOCK_RINGS: rings}, replays=2)


def test_visibility_rules(B):
    """Nside 512: caps, a box rule and a box around the observer."""
    w = synth.Workload("m", 512, 3.0, [
        synth.make_box(300, 31, origin=(-0.5, -0.5, -0.5), eta_lo=2.2, eta_hi=3.0,
                       dtype=np.float32),
        synth.make_box(257, 33, origin=(0.8, -0.4, 0.2), eta_lo=0.9, eta_hi=1.6,
                       dtype=np.float32, vis=synth.VIS_BOX),
        synth.make_box(120, 34, origin=(-1.9, 0.4, -0.6), eta_lo=0.0, eta_hi=3.0,
                       dtype=np.float32, vis=synth.VIS_CAP,
                       cap_dir=np.array([-0.8, 0.6, 0.0]), cap_cos=0.7)])
    st = check(B, w, {B.CSMAP_OPT_GRAPH: 1}, count=8000, replays=3)
    assert st["near_steps"] > 0


@pytest.mark.parametrize("what", ["zero", "negative", "tiny", "huge", "cusp"])
def test_unusual_segments(B, what):
    """dsigma of 0, of either sign, of 1e-34 (below the split's range) beside
    ordinary ones, of 1e34, and segments moving at 0.999 c."""
    w = synth.Workload("m", 150, 16.0, boxes_of([400, 65]))
    for b in w.boxes:
        ds = b.dsigma
        if what == "zero":
            ds[::3] = 0.0
        elif what == "negative":
            ds[::2] *= -1.0
        elif what == "tiny":
            ds[::3] = 1e-34
        elif what == "huge":
            ds *= np.float32(1e34)
        else:
            x, v, t, _ = synth.near_luminal_segments(len(ds), 71, [0.5, 0.96, 0.999])
            b.xdot[:], b.xprime[:] = v, t
    check(B, w)
