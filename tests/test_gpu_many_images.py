"""Sums over the images of one sub-problem and over the columns tied to one parameter, on both sides
of the counts where they get launches of their own (8 and 9 exposures of one galaxy) and beyond,
against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2308_01957_amd import synth
from tests import cases

pytestmark = pytest.mark.gpu


def exposures(m, H=37, W=45):
    """m exposures of one galaxy (every parameter of it tied), each with a sky of its own."""
    one = synth.blend(seed_id=5, H=H, W=W, n_sersic=1, n_point=0, P=7)
    n = one["n_par"]
    spec = dict(one, name="exposures%d" % m, images=[], comps=[], noise=[])
    for k in range(m):
        spec["images"].append(dict(one["images"][0], sub=0, sky_par=n - 1 + k))
        spec["comps"] += [dict(c, image=k) for c in one["comps"]]
        spec["noise"].append(np.random.default_rng(k).standard_normal((H, W)))
    spec["n_par"], spec["subs"] = n - 1 + m, [(0, n - 1 + m)]
    for key in ("theta_true", "theta_init"):
        spec[key] = np.concatenate([one[key][:n - 1], one[key][n - 1] + 0.5 * np.arange(m)])
    return cases.with_data(spec)


@pytest.mark.parametrize("m", [8, 9, 21])
def test_sums_over_exposures(m):
    from paper_2308_01957_amd import apx
    spec = exposures(m)
    print(f"[case] {spec['name']}", flush=True)
    P = apx.Problem(spec)
    d, w = P.pixels(spec["data"]), P.pixels(spec["weight"])
    th = spec["theta_init"]
    c2o = oracle.chi2(spec, th, spec["data"], spec["weight"])
    assert np.allclose(P.chi2(th, d, w).cpu().numpy(), c2o, rtol=1e-10)
    A, g, c2 = P.jtwj(th, d, w)
    Ao, go, _ = oracle.jtwj(spec, th, spec["data"], spec["weight"])
    s = np.sqrt(np.diag(Ao))
    # the Jacobian's 3e-5 of a column's largest entry, as in the tests of the block kernels
    assert np.all(np.abs(P.block(A, 0).cpu().numpy() - Ao) <= 1e-4 * np.outer(s, s))
    assert np.all(np.abs(g.cpu().numpy() - go) <= 1e-4 * s * np.sqrt(c2o.sum()))
    gr, c2g = P.chi2_grad(th, d, w)
    assert np.allclose(c2g.cpu().numpy(), c2o, rtol=1e-10)
    assert np.all(np.abs(gr.cpu().numpy() + 2.0 * go) <= 2e-4 * s * np.sqrt(c2o.sum()))
    seed = np.random.default_rng(1).standard_normal(P.n_pix).astype(np.float32)
    v = P.render_vjp(th, P.torch.from_numpy(seed).to(P.device)).cpu().numpy()
    J = oracle.jacobian(spec, th)
    assert np.all(np.abs(v - seed.astype(np.float64) @ J) <= 1e-4 * (np.abs(seed.astype(np.float64)) @ np.abs(J)))
    t, st = P.lm_init(th, d, w)
    P.lm_run(3, d, w, t, st)
    P.check()
    to, _ = oracle.lm_fit(spec, th, spec["data"], spec["weight"], 3)
    assert np.all(np.abs(t.cpu().numpy() - to) <= 1e-5 * (np.abs(to) + 1.0))
