"""Record slices of the forward launch: tiles whose records are cut over
several wavefronts, against the FP64 oracle.  Bars as for every forward
shape: pair counts exact, FP64 within 1e-12, FP32C within rel-rms 1e-5 and
rel-max 1e-4."""
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


def many_boxes(vis, sizes, nside):
    """More boxes than a wavefront has lanes, with record counts around the
    run of 32 records that slices are made of, empty boxes among them."""
    dirs = synth.uniform_directions(len(sizes), 901)
    boxes = []
    for b, n in enumerate(sizes):
        kw = dict(vis=synth.VIS_CAP, cap_dir=dirs[b], cap_cos=0.3) if vis else {}
        boxes.append(synth.make_box(n, 910 + b, origin=2.0 * dirs[b] - 0.5, eta_lo=0.0,
                                    eta_hi=16.0, dtype=np.float32, **kw))
    return synth.Workload("slices", nside, 16.0, boxes)


SIZES = {"ragged": [0, 1, 31, 32, 33, 64, 97] * 21, "one": [5000], "tail": [0] * 70 + [200, 0]}


@pytest.mark.parametrize("form", ["fp64", "fp32c"])
@pytest.mark.parametrize("sizes", sorted(SIZES))
@pytest.mark.parametrize("vis", [False, True])
@pytest.mark.parametrize("nside,K", [(1, 1), (5, 8), (16, 2)])
def test_sliced_maps(B, form, sizes, vis, nside, K):
    w = many_boxes(vis, SIZES[sizes], nside)
    pix = np.arange(w.npix)
    ref = oracle.theta_pixels(nside, pix, w.eta0, w.boxes)
    pairs = sum(int(oracle.visible(nside, pix, w.eta0, b).sum()) * b.n for b in w.boxes if b.n)
    f = B.CSMAP_FORM_FP64 if form == "fp64" else B.CSMAP_FORM_FP32C
    sky = sky_from_workload(w, f, {B.CSMAP_OPT_PIX_PER_LANE: K, B.CSMAP_OPT_GRAPH: 1})
    out = torch.empty(w.npix, dtype=torch.float64, device="cuda")
    rms, mx = (1e-12, 1e-12) if form == "fp64" else (1e-5, 1e-4)
    for _ in range(3):   # the first call captures, the others replay
        out.fill_(float("nan"))
        got = sky.render(out).cpu().numpy()
        e = err_metrics(got, ref)
        assert sky.stats()["pairs"] == pairs
        assert e["rel_rms"] <= rms and e["rel_max"] <= mx, e
    sky.close()


@pytest.mark.parametrize("form", ["fp64", "fp32c"])
@pytest.mark.parametrize("n", [1, 63, 65, 128, 257, 513])
def test_sliced_directions(B, form, n):
    """Every number of pixels per lane that render_dirs picks by n."""
    w = many_boxes(False, [700, 0, 33], 4)
    d = synth.uniform_directions(n, 77)
    r = np.sqrt((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2])
    ref = oracle.theta_dirs(d / r[:, None], w.eta0, w.boxes, use_vis=True)
    f = B.CSMAP_FORM_FP64 if form == "fp64" else B.CSMAP_FORM_FP32C
    sky = sky_from_workload(w, f)
    got = sky.render_dirs(torch.from_numpy(d).cuda()).cpu().numpy()
    e = err_metrics(got, ref)
    rms, mx = (1e-12, 1e-12) if form == "fp64" else (1e-5, 1e-4)
    assert sky.stats()["pairs"] == n * 733
    assert e["rel_rms"] <= rms and e["rel_max"] <= mx, e
    sky.close()


@pytest.mark.parametrize("K", [1, 2, 4, 8])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 67])
def test_fp64_windows(B, K, n):
    """Windows of four terms per division and their remainders, with exact
    coincidences (Nside 1 pixel 4 is +x) filling a whole window."""
    box = synth.make_box(n, 991, origin=(0.0, 0.0, 0.0), eta_lo=0.0, eta_hi=16.0)
    box.x_rel[::2] = (0.5, 0.0, 0.0)
    box.x_rel[:4] = (0.5, 0.0, 0.0)
    w = synth.Workload("windows", 1, 16.0, [box])
    ref = oracle.theta_pixels(1, np.arange(12), w.eta0, w.boxes)
    sky = sky_from_workload(w, B.CSMAP_FORM_FP64, {B.CSMAP_OPT_PIX_PER_LANE: K})
    e = err_metrics(sky.render().cpu().numpy(), ref)
    assert e["rel_rms"] <= 1e-12 and e["rel_max"] <= 1e-12, e
    sky.close()
