"""The binomial series and the exponential of the FP64 render (k_model.hip, sersic64.h), with the
degrees and radii that the source states: their error over every Sersic index, on the CPU in
extended precision; and, on the GPU, the render by the series against the one node by node."""
import os
import re

import numpy as np
import pytest

from paper_2308_01957_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2308_01957_amd", "csrc")
LD = np.longdouble
EPS = np.finfo(np.float64).eps
needs_extended = pytest.mark.skipif(np.finfo(LD).eps > 2e-19, reason="no 80-bit long double")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def _radii():
    model, internal = _source("k_model.hip"), _source("apx_internal.h")
    near = int(re.search(r"constexpr int BIN_DEG = (\d+);", internal).group(1))
    far = int(re.search(r"constexpr int BIN_DEG_FAR = (\d+);", model).group(1))
    rho = re.search(r"bin_rho\(int deg\) \{ return deg == BIN_DEG \? ([\d.]+) : ([\d.]+); \}", model)
    return [(near, float(rho.group(1))), (far, float(rho.group(2)))]


@needs_extended
@pytest.mark.parametrize("deg,rho", _radii())
def test_binomial_series_within_its_radius(deg, rho):
    """(1 + d)^g from deg terms, g = 1 / (2 n), n in [0.36, 10], |d| <= rho: the part left out is
    below 1.4e-16, and the sum in FP64 as the kernel forms it (d times Horner's value, to which 1 is
    added by the exponent's FMA) is within two roundings of that."""
    d = np.concatenate([np.linspace(-rho, rho, 4001), np.logspace(-12, np.log10(rho), 200)])
    for n in np.concatenate([np.linspace(0.36, 1.0, 65), np.linspace(1.0, 10.0, 181)]):
        g = LD(0.5) / LD(n)
        exact = np.expm1(g * np.log1p(d.astype(LD)))
        coef, c64, g64 = [g], [0.5 / n], 0.5 / n
        for k in range(1, deg):
            coef.append(coef[-1] * (g - k) / LD(k + 1))
            c64.append(c64[-1] * (g64 - k) * (1.0 / (k + 1)))
        q, q64 = np.zeros_like(exact), np.zeros_like(d)
        for k in range(deg - 1, -1, -1):
            q, q64 = q * d + coef[k], q64 * d + c64[k]
        assert np.max(np.abs(d * q - exact)) <= 1.4e-16, n
        # rounding: of each coefficient and step, relative to the series' own size
        size = np.abs(d) * float(g) * 1.2
        assert np.max(np.abs(d * q64 - exact) - 4 * EPS * size) <= 1.4e-16, n


@needs_extended
def test_exponential_of_scaled_arguments():
    """2^(f / 64), |f| <= 1/2, by the series of degree 5: within 4e-17 of the exact value."""
    c = [LD(1.0)]
    for k in range(1, 6):
        c.append(c[-1] * np.log(LD(2)) / 64 / k)
    f = np.linspace(-0.5, 0.5, 20001).astype(LD)
    p = np.zeros_like(f)
    for k in range(5, -1, -1):
        p = p * f + c[k]
    assert np.max(np.abs(p / np.exp2(f / 64) - 1)) <= 4e-17


@pytest.mark.gpu
@pytest.mark.parametrize("s,rule", [(2, 0), (3, 0), (4, 1), (5, 1)])
@pytest.mark.parametrize("k_re", [0.0, 1.5])
def test_series_and_node_by_node_render_agree(s, rule, k_re):
    """chi^2 of apx_chi2 (series and folded stamp rows) and of apx_lm_init (node by node, row by row)
    over Sersic indices, axis ratios and radii from end to end of their ranges, one component an
    image: within the rounding of the two models."""
    from paper_2308_01957_amd import apx
    H, W, P = 61, 75, 9
    rng = np.random.default_rng(s)
    stamp = synth.moffat_psf(P, 2.0, 2.5)
    images, comps, subs, theta = [], [], [], []
    for k, (n, q, re) in enumerate((n, q, re) for n in (0.36, 0.5, 1.0, 2.5, 4.0, 10.0) for q in (0.02, 0.4, 1.0)
                                   for re in (0.05, 3.0, 300.0)):
        phi = rng.uniform(0, 6)
        c, z = np.cos(phi), np.sin(phi)
        aff = np.array([3.0, c, -z, 1.0, z, c])
        x, y = rng.uniform(25, 50), rng.uniform(20, 40)
        p0 = len(theta)
        theta += [aff[0] + c * x - z * y, aff[3] + z * x + c * y, q, rng.uniform(0, 3), n, re, 1.0, 5.0]
        images.append(dict(H=H, W=W, psf=stamp, affine=aff, sub=k, sky_par=p0 + 7, sky_fixed=0.0))
        comps.append(dict(type=synth.SERSIC, image=k, box=(-4, -4, H + 4, W + 4), par=list(range(p0, p0 + 7)),
                          fixed=[0.0] * 7))
        subs.append((p0, 8))
    spec = dict(name="series_s%d" % s, images=images, comps=comps, n_par=len(theta), subs=subs,
                sampling=dict(s=s, rule=rule, mode=synth.MODE_WITHIN_K_RE if k_re else synth.MODE_UNIFORM, k=k_re))
    print(f"[case] {spec['name']} k {k_re}", flush=True)
    prob = apx.Problem(spec)
    theta = np.array(theta)
    m = prob.render(theta).cpu().numpy().astype(np.float64).reshape(len(images), -1)
    prob.check()
    data = np.maximum(m, 0.0) * (1.0 + 0.1 * rng.standard_normal(m.shape))
    d = prob.pixels([v.reshape(H, W) for v in data])
    w = prob.pixels([np.ones((H, W), np.float32)] * len(images))
    c2 = prob.chi2(theta, d, w).cpu().numpy()
    _, st = prob.lm_init(theta, d, w)
    fit = prob.lm_state(st)["chi2"]
    # a node's value is within 40 eps (exponent up to 30, times a few roundings) of the exact one in
    # both, a convolved pixel within 2 P + 4 more of the largest; chi^2 follows by 2 w |r| dm
    r = d.cpu().numpy().astype(np.float64).reshape(m.shape) - m
    dm = 2 * (40 + 2 * P + 4) * EPS * np.abs(m).max(axis=1)
    assert np.all(np.abs(c2 - fit) <= 2 * np.sum(np.abs(r), axis=1) * dm + 1e-12 * c2), np.max(np.abs(c2 - fit) / c2)
