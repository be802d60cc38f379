"""Problems whose workspace comes near the library's scratch array of 64 MiB still fit it: where
short runs of pixels for J^T W J would not, the plan takes longer ones."""
import os

import pytest
import torch  # noqa: F401  (its HIP runtime is the one to load, also where a plan comes first)

from paper_2308_01957_amd import synth

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2308_01957_amd", "libapx.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libapx.so not built")

SPECS = {
    "bands": lambda: synth.multiband(232460, H=95, W=104, n_gal=39, n_band=2, n_epoch=1, P=37),
    "live_psf": lambda: synth.live_psf(888598, H=568, W=335, n_star=35, n_sersic=5, P=41),
    "blend": lambda: synth.blend(243674, H=469, W=414, n_sersic=5, n_point=58, P=41),
    "cutouts": lambda: synth.cutouts(984769, n_cutouts=36, max_comp=3),
}


@pytest.mark.parametrize("name", sorted(SPECS))
def test_problems_near_the_limit_fit_the_scratch(name):
    from paper_2308_01957_amd import apx
    plan = apx.Plan(SPECS[name]())
    assert 56 << 20 < plan.workspace_bytes <= 64 << 20, plan.workspace_bytes / 2 ** 20
    plan.close()


@pytest.mark.gpu
def test_longer_runs_on_the_scratch():
    """The normal equations of such a problem (pairs of narrow groups on the longer runs) on the
    scratch are those of the same plan on a workspace."""
    from paper_2308_01957_amd import apx
    spec = SPECS["bands"]()
    print(f"[case] {spec['name']}", flush=True)
    out = []
    for scratch in (False, True):
        P = apx.Problem(spec, tiles=apx.TILES_MODEL, scratch=scratch)
        gen = torch.Generator(device="cpu").manual_seed(4)
        d = (40.0 + 10.0 * torch.rand(P.n_pix, generator=gen)).to(P.device)
        w = torch.rand(P.n_pix, generator=gen).to(P.device)
        out.append([v.clone() for v in P.jtwj(spec["theta_true"], d, w)])
        P.check()
        P.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
