"""Which form the multi-system stencil takes depends on the precision, the
number of fields and the tiles of the lattice, and how many of a tile's systems
a workgroup takes on the tiles alone.  Both sides of each line: FP16 fields
below and from 6 on above 1024 tiles, and FP32 fields on lattices of 1 (ragged),
162 (six groups), 1024 and 1152 tiles, with and without the fused reductions (a
short batched solve), against the one-field stencil and the oracle."""
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
# against the one-field stencil: the rounding of the stored output
SAME = {wc.FP32: 1e-6, wc.FP16: 2e-3}
TOL = {wc.FP32: 1e-5, wc.FP16: 2e-3}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.mark.parametrize("dims,prec,ns", [((4, 2, 2, 6), wc.FP32, (2, 5, 16)), ((12, 12, 12, 12), wc.FP32, (2, 7, 16)),
                                          ((16, 16, 16, 32), wc.FP32, (3, 12)), ((16, 18, 16, 32), wc.FP32, (2, 5)),
                                          ((4, 2, 2, 6), wc.FP16, (2, 16)), ((16, 16, 16, 32), wc.FP16, (2, 7)),
                                          ((16, 18, 16, 32), wc.FP16, (2, 5, 6))])
def test_forms_match_the_one_field_stencil(dims, prec, ns):
    U = synth.random_links(dims, 0.3, 1970)
    lat = wc.Lattice(dims)
    lat.load_links(dev(U))
    lat.build_clover(KAPPA, 1.0)
    psis = [oracle.restrict(synth.gaussian_source(dims, 2970 + k), 0) for k in range(max(ns))]
    Finv = oracle.site_invert(oracle.clover_field(U, dims, KAPPA, 1.0))
    ref = oracle.dhat_ee(U, Finv, KAPPA, psis[0])
    ins = [lat.parity_view(lat.pack(dev(p), prec), 0, prec).clone() for p in psis]
    one = lat.new_eo(prec, 2)
    single = []
    for e in ins:
        lat.apply_Dee_oo(lat.parity_view(one, 0, prec), e, prec)
        single.append(lat.unpack(one, prec).cpu().numpy())
    for g in (2, 4):
        lat.set_multi_rhs(g)
        for n in ns:
            outs = [lat.new_eo(prec, 2) for _ in range(n)]
            lat.apply_Dee_oo_batch([lat.parity_view(o, 0, prec) for o in outs], ins[:n], prec)
            got = [lat.unpack(o, prec).cpu().numpy() for o in outs]
            errs = [rel(got[k], single[k]) for k in range(n)]
            say(dims, "prec", prec, "G", g, "fields", n, max(errs), rel(got[0], ref))
            assert max(errs) < SAME[prec] and rel(got[0], ref) < TOL[prec]
    lat.set_multi_rhs(-1)
    n = min(5, max(ns))
    bs = [dev(synth.gaussian_source(dims, 3970 + k) * 10.0 ** (k - 2)) for k in range(n)]
    xs, infos = lat.solve_batch(bs, KAPPA, 1.0, 1e-11, inner_prec=prec)
    for k in (0, n - 1):
        r, bn = oracle.residual(U, KAPPA, 1.0, bs[k].cpu().numpy(), xs[k].cpu().numpy())
        assert r / bn < 1e-11, k
    lat.close()
