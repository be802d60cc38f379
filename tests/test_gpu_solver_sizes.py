"""The solvers of one sub-problem at every size where they change kernels (register rows for
8, 16, 24, 40 and 64 columns, the blocked solver above 64), one below and one above each: the
damped Newton step of an LM iteration, the covariance and its factor."""
import numpy as np
import pytest

from paper_2308_01957_amd import synth
from tests import cases

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def _field(n):
    # one Sersic (7 columns), n - 8 point sources, the sky
    spec = cases.with_data(synth.blend(seed_id=500 + n, H=70, W=83, n_sersic=1, n_point=n - 8, P=7))
    assert spec["n_par"] == n
    return spec


@pytest.mark.parametrize("n", [8, 9, 16, 17, 24, 25, 40, 41, 63, 64, 65, 97])
def test_solves_of_every_size(n):
    from paper_2308_01957_amd import apx
    spec = _field(n)
    print(f"[case] {n}", flush=True)
    prob = apx.Problem(spec)
    d, w = prob.pixels(spec["data"]), prob.pixels(spec["weight"])
    th = np.array(spec["theta_init"])
    A, g, _ = prob.jtwj(th, d, w)
    A, g = prob.block(A, 0).cpu().numpy(), g.cpu().numpy()
    C, _ = prob.covariance(th, d, w)
    F, _ = prob.covariance_factor(th, d, w)
    C, F = prob.block(C, 0).cpu().numpy(), prob.block(F, 0).cpu().numpy()
    prob.check()
    # a Cholesky solve is exact for a matrix within 4 n eps |L||L^T| of the given one, and
    # |L||L^T| <= sqrt(a_kk a_ll); 1e-12 more covers the rounding of J^T W J between two runs
    # of the same sums.  Scaled by its diagonal the matrix keeps that bound uniform.
    s = np.sqrt(np.diag(A))
    Ci = np.linalg.inv(A / np.outer(s, s))
    E = (8 * n * EPS + 1e-12) * np.ones((n, n))
    tol = np.abs(Ci) @ E @ np.abs(Ci)
    Co = Ci / np.outer(s, s)
    assert np.all(np.abs(C - Co) * np.outer(s, s) <= tol), float(np.max(np.abs(C - Co) * np.outer(s, s) / tol))
    assert np.all(np.abs(F @ F.T - Co) * np.outer(s, s) <= tol)
    assert np.all(np.tril(F, -1) == 0.0) and np.all(np.diag(F) > 0)
    # the first step from lambda = 1e-2 unless the trial was refused
    tg, st = prob.lm_init(th, d, w)
    lam = float(prob.lm_state(st)["lambda"][0])
    prob.lm_run(1, d, w, tg, st)
    prob.check()
    state = prob.lm_state(st)
    h = tg.cpu().numpy() - th
    if int(state["n_accept"][0]) == 0:
        assert np.all(h == 0.0)
        return
    M = A / np.outer(s, s) + lam * np.eye(n)
    Mi = np.linalg.inv(M)
    ho = Mi @ (g / s)
    tolh = np.abs(Mi) @ (E @ np.abs(ho) + 1e-12 * np.abs(Mi) @ np.abs(g / s)) + 4 * EPS * s * np.abs(th)
    assert np.all(np.abs(h * s - ho) <= tolh), float(np.max(np.abs(h * s - ho) / tolh))
