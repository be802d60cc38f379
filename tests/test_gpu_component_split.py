"""Groups of very different component counts on an image of few tiles, whose components are dealt
to several workgroups (plain, re-centred and adaptive): dense Jacobian and gradient against the FP64
oracle."""
import numpy as np
import pytest

import oracle
from paper_2308_01957_amd import synth
from tests import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["uniform", "recentre", "adaptive"])
@pytest.mark.parametrize("n_sersic,n_point", [(1, 3), (2, 0), (7, 5)])
def test_components_dealt_to_workgroups(n_sersic, n_point, mode):
    from paper_2308_01957_amd import apx
    H, W = 41, 70
    spec = synth.blend(seed_id=700 + n_sersic, H=H, W=W, n_sersic=n_sersic, n_point=n_point, P=9)
    if n_sersic == 7:                       # groups of 4, 2 and 1 galaxies, and the stars'
        for c, box in zip(spec["comps"][4:7], [(3, 5, 33, 60), (3, 5, 33, 60), (10, 20, 31, 53)]):
            c["box"] = box
    if mode == "recentre":
        spec["recentre"] = dict(method=2, a=3)
    elif mode == "adaptive":
        spec["sampling"] = dict(s=3, rule=synth.RULE_MIDPOINT, mode=synth.MODE_ADAPTIVE, k=1e-3)
    spec = cases.with_data(spec)
    print(f"[case] {spec['name']} {mode}", flush=True)
    P = apx.Problem(spec)
    d, w = P.pixels(spec["data"]), P.pixels(spec["weight"])
    th = spec["theta_init"]
    J = P.jacobian(th).cpu().numpy().T.astype(np.float64)
    g, _ = P.chi2_grad(th, d, w)
    P.check()
    Jo = oracle.jacobian(spec, th)
    scale = np.maximum(np.max(np.abs(Jo), axis=0), 1e-30)
    assert np.all(np.max(np.abs(J - Jo), axis=0) <= 3e-5 * scale), np.max(np.max(np.abs(J - Jo), axis=0) / scale)
    go = oracle.chi2_grad(spec, th, spec["data"], spec["weight"])
    r, wv = oracle.residual(spec, th, spec["data"], spec["weight"], [0])
    assert np.all(np.abs(g.cpu().numpy() - go) <= 1e-4 * np.maximum(np.abs(go), 2.0 * (np.abs(wv * r) @ np.abs(Jo))))
