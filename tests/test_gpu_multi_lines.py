"""The multi-system stencil takes one of two forms by precision, number of fields
and tiles.  Fields on both sides of each line, in every FP32 link form and in
FP16 storage: each result against the one-field stencil on the same input, and a
short batched solve (the fused reductions of the same form) to its true residual."""
import pytest

torch = pytest.importorskip("torch")

import synth
from gpu_checks import say

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1709_08785_amd as wc  # noqa: E402

KAPPA = 0.13
# against the one-field stencil: the rounding of the stored output
SAME = {wc.FP32: 1e-6, wc.FP16: 2e-3}
# lattice (tiles per parity), precision, link forms, numbers of fields
LINES = [
    ((16, 16, 16, 16), wc.FP32, (12,), (4, 8)),                 # 512
    ((16, 16, 16, 18), wc.FP32, (12, 8, 18), (3, 4, 5, 8, 9)),  # 576
    ((16, 16, 16, 24), wc.FP32, (12,), (4, 8)),                 # 768
    ((14, 16, 18, 34), wc.FP32, (12, 8, 18), (2, 4)),           # 1071
    ((14, 16, 20, 36), wc.FP32, (12,), (2, 4)),                 # 1260
    ((16, 16, 16, 72), wc.FP32, (12,), (2,)),                   # 2304
    ((12, 24, 24, 44), wc.FP32, (12,), (2,)),                   # 2376
    ((14, 14, 14, 16), wc.FP16, (12,), (2, 15)),                # 343
    ((16, 16, 16, 10), wc.FP16, (12,), (15,)),                  # 320
    ((16, 16, 16, 16), wc.FP16, (12,), (14, 15)),               # 512
    ((16, 16, 16, 18), wc.FP16, (12,), (7, 8, 12)),             # 576
    ((16, 16, 16, 28), wc.FP16, (12,), (12, 14)),               # 896
    ((12, 14, 16, 48), wc.FP16, (12,), (8, 11, 12)),            # 1008
    ((14, 16, 18, 34), wc.FP16, (12,), (5, 6)),                 # 1071
    ((16, 20, 20, 32), wc.FP16, (12,), (5, 6, 9)),              # 1600
    ((20, 20, 20, 30), wc.FP16, (12,), (9,)),                   # 1875
    ((18, 18, 20, 40), wc.FP16, (12,), (6, 9)),                 # 2025
    ((24, 24, 24, 24), wc.FP16, (12,), (6,)),                   # 2592
    ((24, 24, 24, 26), wc.FP16, (12,), (5, 6)),                 # 2808
    ((32, 32, 32, 32), wc.FP16, (12,), (6,)),                   # 8192
]


@pytest.mark.parametrize("dims,prec,recons,ns", LINES)
def test_both_sides_of_each_line(dims, prec, recons, ns):
    lat = wc.Lattice(dims)
    lat.load_links(torch.from_numpy(synth.random_links(dims, 0.3, 1990)).to("cuda"))
    lat.build_clover(KAPPA, 1.0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2990)
    lx, ly, lz, lt = dims
    nmax = max(ns)
    psis = [torch.randn((lt, lz, ly, lx, 4, 3), dtype=torch.complex128, device="cuda", generator=gen) for _ in range(nmax)]
    full = lat.new_eo(prec, 2)
    full.zero_()
    out = lat.parity_view(full, 0, prec)
    for recon in recons:
        if prec == wc.FP32:
            lat.set_link_recon(recon)
        ins = [lat.parity_view(lat.pack(p, prec), 0, prec).clone() for p in psis]

        def unpacked(src=None):
            if src is not None:
                out.copy_(src)
            return lat.unpack(full, prec)

        single = []
        for e in ins:
            lat.apply_Dee_oo(out, e, prec)
            single.append(unpacked())
        for n in ns:
            outs = [lat.new_eo(prec) for _ in range(n)]
            lat.apply_Dee_oo_batch(outs, ins[:n], prec)
            errs = [float((unpacked(o) - w).norm() / w.norm()) for o, w in zip(outs, single)]
            say(dims, "prec", prec, "links", recon, "fields", n, max(errs))
            assert max(errs) < SAME[prec]
        n = min(ns)
        xs, infos = lat.solve_batch(psis[:n], KAPPA, 1.0, 1e-9, inner_prec=prec)
        for i in infos:
            assert i["status"] == 0 and i["true_rel_residual"] <= 1e-9
    lat.close()
