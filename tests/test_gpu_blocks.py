"""J^T W J and J^T W r of column groups of every width that the 4 x 4-block kernels tell
apart (block shapes of two groups, a group with itself below and above 36 columns, single
columns), on windows whose pixel counts are not multiples of a run, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2308_01957_amd import synth
from tests import cases

pytestmark = pytest.mark.gpu

H, W, P = 45, 37, 7
FULL, PART, THIN = (-3, -3, H + 3, W + 3), (5, 8, 31, 33), (-3, 17, 44, 18)

# Sersics per window, point sources
GROUPS = {
    "7x7": ({FULL: 1, PART: 1}, 0),                 # 2 x 2 tiles
    "7x1": ({FULL: 1}, 2),                          # 2 x 1 and 1 x 1
    "14x1_14x7": ({FULL: 2, PART: 1}, 1),           # 4 x 1 and 4 x 2
    "14x14": ({FULL: 2, PART: 2}, 0),               # 4 x 4
    "28x7_thin": ({FULL: 4, THIN: 1}, 0),           # 8 x 2, a window one pixel wide
    "21x14": ({PART: 3, THIN: 2}, 1),               # 8 x 4 with empty tiles, 8 x 1
    "35": ({FULL: 5}, 0),                           # the widest single-group kernel
    "42": ({FULL: 6}, 0),                           # with itself on 8 x 4 blocks
    "42x42": ({FULL: 6, PART: 6}, 0),
    "63x7": ({FULL: 9, PART: 1}, 1),                # 64-wide tiles and 8 x 2 blocks
}


@pytest.mark.parametrize("name", sorted(GROUPS))
def test_normal_equations_of_every_group_width(name):
    from paper_2308_01957_amd import apx
    groups, n_point = GROUPS[name]
    n = sum(groups.values())
    spec = synth.blend(seed_id=300 + n, H=H, W=W, n_sersic=n, n_point=n_point, P=P)
    boxes = [b for b, k in groups.items() for _ in range(k)]
    for comp, box in zip(spec["comps"], boxes):
        comp["box"] = box
    spec = cases.with_data(spec)
    print(f"[case] {name}", flush=True)
    prob = apx.Problem(spec)
    th = spec["theta_init"]
    A, g, c2 = prob.jtwj(th, prob.pixels(spec["data"]), prob.pixels(spec["weight"]))
    prob.check()
    Ao, go, c2o = oracle.jtwj(spec, th, spec["data"], spec["weight"])
    A = prob.block(A, 0).cpu().numpy()
    d = np.sqrt(np.diag(Ao))
    # 3e-5 of a column's largest entry in each Jacobian entry (the Jacobian's own bound)
    # cannot move an entry by more than 1e-4 of the geometric mean of its diagonal
    assert np.all(np.abs(A - Ao) <= 1e-4 * np.outer(d, d)), float(np.max(np.abs(A - Ao) / np.outer(d, d)))
    assert np.array_equal(A, A.T)
    c2o = float(np.sum(c2o))
    assert np.all(np.abs(g.cpu().numpy() - go) <= 1e-4 * d * np.sqrt(c2o))
