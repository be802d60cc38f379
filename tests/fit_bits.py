"""A batch of cutouts whose stamps, data and start are made with additions, products and quotients
only, so that every machine has them to the bit, and the fit of six of them to three iterations
(tests/golden/fit_bits.txt)."""
import math

import numpy as np

from paper_2308_01957_amd import synth

SKY = 40.0


def _stamp(P, scale):
    v = np.arange(P, dtype=np.float64) - (P - 1) // 2
    u = 1.0 + (v[:, None] * v[:, None] + v[None, :] * v[None, :]) / (scale * scale)
    f = 1.0 / (u * u)
    return (f / math.fsum(f.ravel())).astype(np.float32)


def cutout(number):
    """(size, stamp, start of the galaxies, data, weight) of one cutout."""
    rng = np.random.Generator(np.random.PCG64(number))
    side, P = 48 + int(rng.integers(0, 60)), 15 + 2 * int(rng.integers(0, 9))
    y, x = np.arange(side, dtype=np.float64)[:, None], np.arange(side, dtype=np.float64)[None, :]
    d, start = np.full((side, side), SKY), []
    for _ in range(1 + int(rng.integers(0, 5))):
        u = rng.random(7)
        x0, y0 = side * (0.25 + 0.5 * u[0]), side * (0.25 + 0.5 * u[1])
        t, q, re = u[2], 0.35 + 0.5 * u[3], 2.0 + 5.0 * u[4]
        c, s = (1.0 - t * t) / (1.0 + t * t), 2.0 * t / (1.0 + t * t)
        xp, yp = (x - x0) * c + (y - y0) * s, ((y - y0) * c - (x - x0) * s) / q
        r2 = (xp * xp + yp * yp) / (re * re)
        d = d + (100.0 + 900.0 * u[5]) / ((1.0 + r2) * (1.0 + r2))
        # near the profile: position angle by its half-angle tangent, n, Re, log10 Ie
        start.append([x0 + 0.4, y0 - 0.3, q + 0.05, 2.0 * t - 0.4 * t * t * t, 1.0 + u[6], 1.1 * re, 2.0 + 0.5 * u[5]])
    var = d + 20.0
    noise = rng.random((4, side, side))
    n = (noise[0] + noise[1]) + (noise[2] + noise[3]) - 2.0
    data = (d + np.sqrt(3.0 * var) * n).astype(np.float32)
    return side, _stamp(P, 0.12 * P), start, data, (1.0 / var).astype(np.float32)


def batch(numbers):
    """The spec of these cutouts as one batch (its own sky and galaxies each), data and weights in it."""
    images, comps, subs, theta, data, weight = [], [], [], [], [], []
    for k, number in enumerate(numbers):
        side, stamp, start, d, w = cutout(number)
        p0, c = len(theta), (stamp.shape[0] - 1) // 2
        for g in start:
            comps.append(dict(type=synth.SERSIC, image=k, box=(-c, -c, side + c, side + c),
                              par=list(range(len(theta), len(theta) + 7)), fixed=[0.0] * 7))
            theta += g
        theta.append(SKY + 1.0)
        images.append(dict(H=side, W=side, psf=stamp, affine=synth.IDENTITY_AFFINE.copy(), sub=k, sky_par=len(theta) - 1,
                           sky_fixed=0.0))
        subs.append((p0, len(theta) - p0))
        data.append(d)
        weight.append(w)
    return dict(name="fit_bits%d" % len(images), images=images, comps=comps, n_par=len(theta), subs=subs,
                sampling=dict(s=3, rule=synth.RULE_MIDPOINT, mode=synth.MODE_UNIFORM, k=0.0),
                theta_init=np.array(theta), data=data, weight=weight)
