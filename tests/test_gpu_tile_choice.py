"""The tiles of the launches that add FP64 sums over their tiles follow from the description alone:
whatever the autotuner times, a problem's model shapes, and the Jacobian shapes of a field with
wide groups, are those of a plan made without a GPU."""
import pytest
import torch  # noqa: F401  (its HIP runtime is the one to load, also where a plan comes first)

from paper_2308_01957_amd import synth
from tests import cases

pytestmark = pytest.mark.gpu

SPECS = {
    "cutouts": lambda: synth.cutouts(seed_id=17, n_cutouts=300),
    "cutouts_fp32": lambda: synth.cutouts(seed_id=18, n_cutouts=150),
    "wide_groups": cases.wide_groups,
    "wide_group_near_128_tiles": lambda: synth.blend(seed_id=41, H=500, W=470, n_sersic=6, n_point=2, P=11),
    "live_psf": lambda: synth.live_psf(3, H=150, W=170, n_star=4, n_sersic=6, P=21),
}


@pytest.mark.parametrize("name", sorted(SPECS))
def test_shapes_of_summed_launches_are_the_plans(name):
    from paper_2308_01957_amd import apx
    spec = SPECS[name]()
    objective = 1 if name.endswith("fp32") else 0
    print(f"[case] {spec['name']}", flush=True)
    plan = apx.Plan(spec, objective=objective, tiles=apx.TILES_AUTOTUNE)
    kinds = (0, 1) if name.startswith("wide") else (0,)
    want = [plan.tile_shapes(k) for k in kinds]
    plan.close()
    for _ in range(2):
        P = apx.Problem(spec, objective=objective)
        assert [P.tile_shapes(k) for k in kinds] == want
        P.close()
