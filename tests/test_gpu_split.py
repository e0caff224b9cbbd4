"""The stencil with a tile's four directions on four wavefronts, at the edges of
its range: a lattice of one partly filled tile, a ragged last tile, and both
sides of the tile count up to which FP16 storage and reconstruct-8 links take
it (1024 tiles at 16^3x32).  MULT into each parity, D-hat_ee and D against the
oracle, with the tolerances of the other operator tests."""
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("dims", [(4, 4, 2, 2), (6, 10, 4, 6), (16, 16, 16, 32), (16, 18, 16, 32)])
def test_split_stencil_matches_oracle(dims):
    U = synth.random_links(dims, 0.3, 1950)
    psi = synth.gaussian_source(dims, 2950)
    lat = wc.Lattice(dims)
    lat.load_links(dev(U))
    lat.build_clover(KAPPA, 1.0)
    F = oracle.clover_field(U, dims, KAPPA, 1.0)
    Finv = oracle.site_invert(F)
    mult = [oracle.htilde(U, Finv, oracle.restrict(psi, 1 - p), p) for p in (0, 1)]
    even = oracle.restrict(psi, 0)
    dhat = oracle.dhat_ee(U, Finv, KAPPA, even)
    full = oracle.apply_D(U, F, KAPPA, psi)
    for prec, recon in ((wc.FP64, 12), (wc.FP32, 12), (wc.FP32, 8), (wc.FP32, 18), (wc.FP16, 12)):
        lat.set_link_recon(recon)
        eo = lat.pack(dev(psi), prec)
        half = [lat.parity_view(eo, p, prec) for p in (0, 1)]
        out = lat.new_eo(prec, 2)
        for p in (0, 1):
            lat.apply_mult(lat.parity_view(out, p, prec), half[1 - p], p, prec)
        got = lat.unpack(out, prec).cpu().numpy()
        errs = [rel(oracle.restrict(got, p), mult[p]) for p in (0, 1)]
        out = lat.new_eo(prec, 2)
        lat.apply_Dee_oo(lat.parity_view(out, 0, prec), half[0], prec)
        errs.append(rel(lat.unpack(out, prec).cpu().numpy(), dhat))
        if prec != wc.FP16:
            errs.append(rel(lat.apply_D(dev(psi), prec).cpu().numpy(), full))
        say(dims, "prec", prec, "links", recon, errs)
        assert max(errs) < TOL[prec]
    lat.close()
