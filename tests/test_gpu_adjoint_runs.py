"""The adjoint's runs of pixels (rings cut at 64 pixels and at the chunks'
ends, far and close runs) and its combination of chunks over boxes, against
the oracle's gradient: relative L2 per group within 1e-4, as for every
adjoint shape."""
import numpy as np
import pytest

import oracle
import synth
from helpers import GRAD_GROUPS, grad_group_errors, sky_from_workload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nside,split", [(1, 0), (2, 1), (3, 5), (7, 3), (16, 0), (17, 200),
                                         (33, 1)])
@pytest.mark.parametrize("vis", [False, True])
def test_runs(nside, split, vis):
    from paper_1204_5041_amd import binding as B
    dirs = synth.uniform_directions(5, 51)
    boxes = []
    for b, n in enumerate((65, 0, 1, 130, 64)):
        kw = dict(vis=synth.VIS_CAP, cap_dir=dirs[b], cap_cos=-0.2) if vis and b % 2 else {}
        # the slab cuts some of box 3's segments off
        boxes.append(synth.make_box(n, 60 + b, origin=1.5 * dirs[b] - 0.5, eta_lo=0.0,
                                    eta_hi=14.4 if b == 3 else 16.0, dtype=np.float32, **kw))
    w = synth.Workload("runs", nside, 16.0, boxes)
    rng = np.random.Generator(np.random.PCG64(nside))
    cot = rng.standard_normal(w.npix)
    sky = sky_from_workload(w, B.CSMAP_FORM_FP32C, {B.CSMAP_OPT_ADJ_SPLIT: split})
    grads = sky.backward(torch.from_numpy(cot).cuda())
    got = np.concatenate([np.concatenate([t.cpu().numpy().reshape(len(g[3]), k)
                                          for t, k in zip(g, (3, 3, 3, 1))], 1) for g in grads])
    total = sum(b.n for b in boxes)
    ref = oracle.grad(nside, np.arange(w.npix), cot, w.eta0, boxes, np.arange(total))
    kept = np.concatenate([oracle.kept(w.eta0, b) for b in boxes]).astype(bool)
    assert np.all(got[~kept] == 0.0)
    e = grad_group_errors(got, ref)
    print(nside, split, vis, e, flush=True)
    for name, _ in GRAD_GROUPS:
        assert e[name] <= 1e-4, e
    sky.close()
