"""A sky used again without waiting: boxes dropped and added while earlier
work is in flight, the schedules in turn on one plan, tensors of another
stream, and host arrays.  Every map equals that of a fresh sky bit for bit."""
import ctypes

import numpy as np
import pytest

import synth
from helpers import sky_from_workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    from paper_1204_5041_amd import binding
    assert torch.cuda.is_available()
    return binding


def workload(seed, sizes, vis=False, nside=64):
    dirs = synth.uniform_directions(len(sizes), seed)
    boxes = []
    for b, n in enumerate(sizes):
        kw = dict(vis=synth.VIS_CAP, cap_dir=dirs[b], cap_cos=0.5) if vis else {}
        boxes.append(synth.make_box(n, seed + 1 + b, origin=2.0 * dirs[b] - 0.5, eta_lo=0.0,
                                    eta_hi=16.0, dtype=np.float32, **kw))
    return synth.Workload("reuse", nside, 16.0, boxes)


def fill(sky, w):
    for bx in w.boxes:
        t = [torch.from_numpy(a).cuda() for a in (bx.x_rel, bx.xdot, bx.xprime, bx.dsigma)]
        kw = {}
        if bx.cap_dir is not None:
            kw = dict(cap_dir=tuple(bx.cap_dir), cap_cos=bx.cap_cos)
        sky.add_box(*t, origin=tuple(bx.origin), eta_lo=bx.eta_lo, eta_hi=bx.eta_hi, vis=bx.vis,
                    **kw)


def fresh(B, w, form, options=None):
    sky = sky_from_workload(w, form, options)
    m = sky.render()
    torch.cuda.synchronize()
    sky.close()
    return m


@pytest.mark.parametrize("form", ["fp64", "fp32c"])
@pytest.mark.parametrize("graph", [0, 1])
def test_reset_and_render_back_to_back(B, form, graph):
    f = B.CSMAP_FORM_FP64 if form == "fp64" else B.CSMAP_FORM_FP32C
    ws = [workload(10, [900]), workload(20, [300, 0, 40], vis=True), workload(30, [1]),
          workload(40, [5000, 64]), workload(50, [300, 0, 40], vis=True)]
    want = [fresh(B, w, f) for w in ws]
    sky = B.Sky(64, 16.0, f)
    sky.set_option(B.CSMAP_OPT_GRAPH, graph)
    got = []
    for w in ws + ws[::-1]:
        sky.reset()
        fill(sky, w)
        got.append(sky.render())
    torch.cuda.synchronize()
    for k, (g, w) in enumerate(zip(got, want + want[::-1])):
        assert torch.equal(g, w), k
    sky.close()


def test_schedules_in_turn(B):
    w = workload(60, [700, 90, 33], vis=True)
    sky = sky_from_workload(w, B.CSMAP_FORM_FP64)
    for schedule in (1, 2, 0, 2, 1):
        sky.set_option(B.CSMAP_OPT_SCHEDULE, schedule)
        assert torch.equal(sky.render(), fresh(B, w, B.CSMAP_FORM_FP64,
                                               {B.CSMAP_OPT_SCHEDULE: schedule})), schedule
    sky.close()


def test_tensors_of_another_stream(B):
    """The copies run on the sky's stream: memory that the caller's stream
    gets back after a reset must not be handed out before they are done."""
    w = workload(70, [200_000], nside=16)
    want = fresh(B, w, B.CSMAP_FORM_FP64)
    side = torch.cuda.Stream()
    sky = B.Sky(16, 16.0, B.CSMAP_FORM_FP64, stream=side)
    for _ in range(3):
        sky.reset()
        torch.cuda.synchronize()
        fill(sky, w)
        out = torch.empty(w.npix, dtype=torch.float64, device="cuda")
        sky._keep.clear()
        junk = [torch.full((200_000, 3), float("nan"), device="cuda") for _ in range(6)]
        sky.render(out)
        side.synchronize()
        assert torch.equal(out, want)
        del junk
    sky.close()


def test_host_arrays(B):
    w = workload(80, [257])
    want = fresh(B, w, B.CSMAP_FORM_FP64)
    bx = w.boxes[0]
    b = B.csmap_box()
    b.n, b.dtype = bx.n, B.CSMAP_F32
    b.x_rel, b.xdot, b.xprime, b.dsigma = (a.ctypes.data for a in (bx.x_rel, bx.xdot, bx.xprime,
                                                                  bx.dsigma))
    b.origin = (ctypes.c_double * 3)(*[float(v) for v in bx.origin])
    b.ext = (ctypes.c_double * 3)(1.0, 1.0, 1.0)
    b.eta_lo, b.eta_hi, b.vis = bx.eta_lo, bx.eta_hi, B.CSMAP_VIS_ALL
    sky = B.Sky(64, 16.0, B.CSMAP_FORM_FP64)
    B.csmap_add_box(sky.handle, b)
    assert torch.equal(sky.render(), want)
    sky.close()
