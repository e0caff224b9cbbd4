"""Reconstruct-8 links are read through the last-level cache up to 120 MB by a
stencil launch by itself and up to 192 MB in a solve.  D-hat_ee with 99 and 135 MB
of links against the oracle (lattices that repeat a small one, as in the test of
the other link forms), and a solve with 135 MB to its true residual."""
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

KAPPA = 0.13
BASE = (14, 4, 4, 48)


@pytest.mark.parametrize("reps,solve", [((2, 6, 6), False), ((2, 7, 7), True)])
def test_recon8_on_both_sides_of_its_line(reps, solve):
    U = synth.random_links(BASE, 0.3, 1953)
    psi = synth.gaussian_source(BASE, 2953)
    Finv = oracle.site_invert(oracle.clover_field(U, BASE, KAPPA, 1.0))
    want = oracle.dhat_ee(U, Finv, KAPPA, oracle.restrict(psi, 0))

    def tiled(a):
        d = torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
        lead = [1] if d.dim() == 7 else []  # the links' direction
        return d.repeat(*lead, 1, reps[2], reps[1], reps[0], 1, 1)

    dims = tuple(b * r for b, r in zip(BASE, reps + (1,)))
    lat = wc.Lattice(dims)
    lat.load_links(tiled(U))
    lat.set_link_recon(8)
    lat.build_clover(KAPPA, 1.0)
    half = lat.parity_view(lat.pack(tiled(psi), wc.FP32), 0, wc.FP32)
    out = lat.new_eo(wc.FP32, 2)
    out.zero_()
    lat.apply_Dee_oo(lat.parity_view(out, 0, wc.FP32), half, wc.FP32)
    ref = tiled(want)
    err = float(torch.linalg.vector_norm(lat.unpack(out, wc.FP32) - ref) / torch.linalg.vector_norm(ref))
    say(dims, "error", err)
    assert err < 1e-5  # as the other FP32 operator tests
    if solve:
        _, info = lat.solve(tiled(psi), KAPPA, 1.0, 1e-10)
        assert info["true_rel_residual"] <= 1e-10
    lat.close()
