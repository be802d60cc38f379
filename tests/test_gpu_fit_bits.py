"""A fit keeps its result to the bit: theta after four iterations of five cutouts whose later
iterations follow the last bits of the earlier ones (a theta that moves by 1e-14 turns the
rounding of FP32 derivative images, and with it the next step by 1e-8), on FFT-tile Jacobians,
alone and as part of a larger batch."""
import os

import numpy as np
import pytest

from tests import fit_bits

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "fit_bits.txt")


def _golden():
    with open(GOLDEN) as f:
        rows = [line.split() for line in f if not line.startswith("#")]
    return {int(r[0]): np.array([float.fromhex(v) for v in r[1:]]) for r in rows}


@pytest.mark.parametrize("others", [[], list(range(1, 25))], ids=["alone", "among_others"])
@pytest.mark.parametrize("graph", [False, True], ids=["eager", "graph"])
def test_theta_of_a_fit_is_the_same_to_the_bit(others, graph):
    from paper_2308_01957_amd import apx
    golden = _golden()
    spec = fit_bits.batch(others + sorted(golden))
    spec["conv_mode"] = apx.CONV_AUTO
    print(f"[case] {spec['name']} graph={graph}", flush=True)
    P = apx.Problem(spec, tiles=apx.TILES_FIXED)
    d, w = P.pixels(spec["data"]), P.pixels(spec["weight"])
    t, st = P.lm_init(spec["theta_init"], d, w)
    P.lm_run(4, d, w, t, st, use_graph=graph)
    P.check()
    t = t.cpu().numpy()
    for (p0, n), number in zip(spec["subs"][len(others):], sorted(golden)):
        assert np.array_equal(t[p0:p0 + n], golden[number]), (number, np.max(np.abs(t[p0:p0 + n] - golden[number])))
