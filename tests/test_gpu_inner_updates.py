"""The inner loop's updates sum the reduction partials themselves up to 1279 of
them and take them from a fold kernel above.  Solves on both sides of that
line, single and batched (a batch folds for every system as soon as one needs
it), against the oracle's true residual, with the iteration cap and the fixed
iteration count honoured exactly."""
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

BELOW, AT = (16, 16, 16, 36), (16, 16, 20, 32)  # 1152 and 1280 tiles per parity
KAPPA = 0.13


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def lattice(dims, seed):
    U = synth.random_links(dims, 0.3, seed)
    lat = wc.Lattice(dims)
    lat.load_links(dev(U))
    return lat, U, synth.gaussian_source(dims, seed + 1000)


@pytest.mark.parametrize("inner", [wc.FP32, wc.FP16, wc.FP64])
@pytest.mark.parametrize("dims", [BELOW, AT])
def test_solve_on_both_sides_of_the_fold(dims, inner):
    lat, U, b = lattice(dims, 1960)
    x, info = lat.solve(dev(b), KAPPA, 1.0, 1e-12, inner_prec=inner)
    r, bn = oracle.residual(U, KAPPA, 1.0, b, x.cpu().numpy())
    say(dims, inner, info["inner_iters_total"], r / bn)
    assert r / bn < 1e-12
    # exactly the iterations asked for, whatever the chunks
    _, info = lat.solve(dev(b), KAPPA, 1.0, 1e-12, inner_prec=inner, fixed_work=11, check_every=4, outer_maxit=1,
                        raise_on_error=False)
    assert info["inner_iters_total"] == 11 * info["inner_calls"]
    _, info = lat.solve(dev(b), KAPPA, 1.0, 1e-12, inner_prec=inner, inner_maxit=3, outer_maxit=1,
                        raise_on_error=False)
    assert info["rc"] == -5 and info["inner_iters_total"] == 3 * info["inner_calls"]
    lat.close()


def test_batch_with_and_without_fold_together():
    lats, Us, bs = zip(*(lattice(d, s) for d, s in (((8, 8, 8, 8), 1961), (AT, 1962))))
    xs, infos = wc.solve_multi(lats, [dev(b) for b in bs], [KAPPA] * 2, [1.0] * 2, 1e-12)
    for U, b, x, info in zip(Us, bs, xs, infos):
        r, bn = oracle.residual(U, KAPPA, 1.0, b, x.cpu().numpy())
        say(info["inner_iters_total"], r / bn)
        assert r / bn < 1e-12
    for lat in lats:
        lat.close()
