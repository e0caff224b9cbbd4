"""The one-system stencil on both sides of the size up to which it reads the
links through the last-level cache (192 MB of links).  The large lattices repeat
a small one in x, y and z (the temporal boundary stays one), so D-hat_ee on them
is the oracle's result for the small one, repeated.  Tolerances of the other
operator tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
import synth
from gpu_checks import say

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1709_08785_amd as wc  # noqa: E402

TOL = {wc.FP64: 1e-13, wc.FP32: 1e-5, wc.FP16: 2e-3}
KAPPA = 0.13
BASE = (14, 4, 4, 48)


# MB of links: FP64 155 | 310, FP32 103 | 202 (two columns), 152 | 303 (full), 135 (8 reals), FP16 101
@pytest.mark.parametrize("prec,recon,reps", [
    (wc.FP64, 12, (1, 5, 5)), (wc.FP64, 12, (2, 5, 5)),
    (wc.FP32, 12, (2, 5, 5)), (wc.FP32, 12, (2, 7, 7)),
    (wc.FP32, 18, (1, 7, 7)), (wc.FP32, 18, (2, 7, 7)),
    (wc.FP32, 8, (2, 7, 7)), (wc.FP16, 12, (2, 7, 7)),
])
def test_dhat_on_both_sides_of_the_link_cache(prec, recon, reps):
    U = synth.random_links(BASE, 0.3, 1951)
    psi = synth.gaussian_source(BASE, 2951)
    Finv = oracle.site_invert(oracle.clover_field(U, BASE, KAPPA, 1.0))
    want = oracle.dhat_ee(U, Finv, KAPPA, oracle.restrict(psi, 0))

    def tiled(a):
        d = torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
        lead = [1] if d.dim() == 7 else []  # the links' direction
        return d.repeat(*lead, 1, reps[2], reps[1], reps[0], 1, 1)

    dims = tuple(b * r for b, r in zip(BASE, reps + (1,)))
    say(dims, "prec", prec, "links", recon)
    lat = wc.Lattice(dims)
    lat.load_links(tiled(U))
    lat.set_link_recon(recon)
    lat.build_clover(KAPPA, 1.0)
    half = lat.parity_view(lat.pack(tiled(psi), prec), 0, prec)
    out = lat.new_eo(prec, 2)
    out.zero_()
    lat.apply_Dee_oo(lat.parity_view(out, 0, prec), half, prec)
    got = lat.unpack(out, prec)
    ref = tiled(want)
    err = float(torch.linalg.vector_norm(got - ref) / torch.linalg.vector_norm(ref))
    say("error", err)
    assert err < TOL[prec]
    lat.close()
