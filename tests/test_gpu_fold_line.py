"""Where the reduction partials of the inner loop's updates are many for their
blocks, a fold kernel sums them once.  The line lies at 314 tiles for blocks of 64
threads and at 887 for 128 (1255 with FP16 storage, whose stencil then leaves a
partial per block), and at 2508 for 256.  Solves just below and above it against
the oracle's true residual, with exact iteration counts, and batches: several small
systems with one that needs the kernel, and systems (up to four count) that need it
together and not alone."""
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
# threads, the storage precisions of the inner solve, and lattices on both sides
LINE = [
    (64, (wc.FP32, wc.FP64, wc.FP16), ((14, 14, 20, 10), (12, 14, 20, 12))),   # 307, 315 tiles
    (128, (wc.FP32, wc.FP64, wc.FP16), ((14, 16, 18, 28), (16, 18, 18, 22))),  # 882, 891
    (128, (wc.FP16,), ((20, 20, 20, 20), (16, 18, 20, 28))),                   # 1250, 1260
    (256, (wc.FP32,), ((20, 20, 24, 32), (24, 24, 24, 24))),                   # 2400, 2592
]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def lattice(dims, seed, threads):
    U = synth.random_links(dims, 0.3, seed)
    lat = wc.Lattice(dims)
    lat.load_links(dev(U))
    lat.set_block_size(threads)
    return lat, U, synth.gaussian_source(dims, seed + 1000)


@pytest.mark.parametrize("threads,inner,dims", [(t, p, d) for t, ps, ds in LINE for p in ps for d in ds])
def test_solve_on_both_sides(threads, inner, dims):
    lat, U, b = lattice(dims, 1980, threads)
    x, info = lat.solve(dev(b), KAPPA, 1.0, 1e-12, inner_prec=inner)
    r, bn = oracle.residual(U, KAPPA, 1.0, b, x.cpu().numpy())
    say(threads, dims, inner, info["inner_iters_total"], r / bn)
    assert info["block_size"] == threads and r / bn < 1e-12
    # exactly the iterations asked for, whatever the chunks
    _, info = lat.solve(dev(b), KAPPA, 1.0, 1e-12, inner_prec=inner, fixed_work=11, check_every=4, outer_maxit=1,
                        raise_on_error=False)
    assert info["inner_iters_total"] == 11 * info["inner_calls"]
    lat.close()


@pytest.mark.parametrize("inner", [wc.FP32, wc.FP16])
@pytest.mark.parametrize("dims", [((8, 8, 8, 8), (12, 14, 20, 12)), ((12, 12, 12, 12),) * 2, ((12, 12, 12, 16),) * 2,
                                  ((12, 12, 12, 12),) * 4])
def test_batch_across_the_line(inner, dims):
    lats, Us, bs = zip(*(lattice(d, 1981 + k, 64) for k, d in enumerate(dims)))
    xs, infos = wc.solve_multi(lats, [dev(b) for b in bs], [KAPPA] * len(lats), [1.0] * len(lats), 1e-12, inner_prec=inner)
    for U, b, x, info in zip(Us, bs, xs, infos):
        r, bn = oracle.residual(U, KAPPA, 1.0, b, x.cpu().numpy())
        say(inner, info["inner_iters_total"], r / bn)
        assert r / bn < 1e-12
    for lat in lats:
        lat.close()
