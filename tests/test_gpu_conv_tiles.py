"""The model and adjoint convolutions at the PSF sizes and image sizes where their kernels
change: stamps the same upside down and not, the smallest and largest windows, images of few
tiles (two outputs per lane) and of many (eight), and a sub-pixel grid of few tiles (always
eight), against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2308_01957_amd import synth
from tests import cases

pytestmark = pytest.mark.gpu


def _spec(P, H, W, even, up=1):
    rng = np.random.default_rng(P)
    psf = synth.moffat_psf(P, max(1.5, P / 8.0), 2.5) if even else synth.asymmetric_psf(P, rng)
    spec = synth.blend(seed_id=400 + P, H=H, W=W, n_sersic=2, n_point=2, P=P, psf=psf)
    if up > 1:
        spec = synth.with_psf_upsampling(spec, up, P)
    return cases.with_data(spec)


@pytest.mark.parametrize("even", [True, False], ids=["mirror", "lopsided"])
@pytest.mark.parametrize("P,H,W", [(1, 33, 31), (3, 40, 67), (15, 65, 33), (41, 37, 70), (43, 64, 49), (51, 30, 33),
                                   (53, 48, 64), (63, 41, 45)])
def test_few_tiles(P, H, W, even):
    _check(_spec(P, H, W, even))


@pytest.mark.parametrize("even", [True, False], ids=["mirror", "lopsided"])
@pytest.mark.parametrize("P", [5, 33, 41, 43, 63])
def test_many_tiles(P, even):
    # 32 x 64 tiles of a 1000 x 300 image: 160, more than half the compute units
    _check(_spec(P, 1000, 300, even), gradient=False)


@pytest.mark.parametrize("P", [7, 45])
def test_few_tiles_of_sub_pixels(P):
    _check(_spec(P, 30, 37, True, up=4))


def _check(spec, gradient=True):
    from paper_2308_01957_amd import apx
    print(f"[case] {spec['name']}", flush=True)
    prob = apx.Problem(spec)
    th = spec["theta_init"]
    dd, ww = prob.pixels(spec["data"]), prob.pixels(spec["weight"])
    m = prob.split(prob.render(th))[0].astype(np.float64)
    c2 = float(prob.chi2(th, dd, ww).cpu()[0])
    prob.check()
    mo = oracle.model_image(spec, th, 0)
    assert np.all(np.abs(m - mo) <= cases.tol_pixels(mo))
    # an FP64 sum of P^2 products is within 2 P + 4 ulp of each pixel's value, and chi^2 moves by
    # at most sum 2 w |r| dm
    d, w = (np.asarray(x[0], dtype=np.float64) for x in (spec["data"], spec["weight"]))
    dm = (2 * np.asarray(spec["images"][0]["psf"]).shape[0] + 40) * 2.2e-16 * np.abs(mo).max()
    c2o = float(oracle.chi2(spec, th, spec["data"], spec["weight"])[0])
    assert abs(c2 - c2o) <= np.sum(2 * w * np.abs(d - mo)) * dm + 1e-12 * c2o, (c2, c2o)
    if gradient:
        g, _ = prob.chi2_grad(th, dd, ww)
        go = oracle.chi2_grad(spec, th, spec["data"], spec["weight"])
        J = oracle.jacobian(spec, th)
        scale = np.maximum(np.abs(go), np.sum(np.abs(J * (2 * w * (d - mo)).reshape(-1, 1)), axis=0))
        assert np.all(np.abs(g.cpu().numpy() - go) <= 1e-4 * scale)
