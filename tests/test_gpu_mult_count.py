"""info.dslash_count is the number of MULTs that ran.  The launched inner loop
notices a half-step exit after that iteration's second D-hat, and a full-step
exit at the host read that ends its chunk or, inside a chunk, after one D-hat
of the next iteration.  With a read after every iteration an inner solve
therefore runs four MULTs per iteration, exits of either kind included; with
one chunk for everything, two more for each full-step exit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from gpu_checks import say

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1709_08785_amd as wc  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("inner", [wc.FP32, wc.FP16])
@pytest.mark.parametrize("graph", [0, 1])
def test_mults_that_ran(inner, graph):
    dims = (8, 8, 8, 8)
    lat = wc.Lattice(dims)
    lat.load_links(dev(synth.random_links(dims, 0.3, 1970)))
    extra = {1: [], 500: []}
    calls = 0
    for seed in range(4):
        b = dev(synth.gaussian_source(dims, 2970 + seed))
        for every in (1, 500):
            _, info = lat.solve(b, 0.13, 1.0, 1e-10, inner_prec=inner, check_every=every, use_graph=graph)
            assert info["restarts"] == 0
            # outside the inner solves: two to set up, two per inner solve (the FP64
            # D-hat), three for x_o and the true residual
            extra[every].append(info["dslash_count"] - 5 - 2 * info["inner_calls"] - 4 * info["inner_iters_total"])
            if every == 1:
                calls += info["inner_calls"]
    say(extra, calls)
    assert extra[1] == [0] * 4
    assert all(e >= 0 and e % 2 == 0 for e in extra[500]) and sum(extra[500]) <= 2 * calls
    # exits of both kinds occur among these solves
    assert 0 < sum(extra[500]) < 2 * calls
    lat.close()


@pytest.mark.parametrize("every", [1, 500])
def test_mults_that_ran_in_the_pipelined_loop(every):
    # two D-hats to set up, two per iteration; a half-step exit comes before both
    # of its iteration's, a full-step exit between them
    dims = (8, 8, 8, 8)
    lat = wc.Lattice(dims)
    lat.load_links(dev(synth.random_links(dims, 0.3, 1971)))
    extra, calls = 0, 0
    for seed in range(4):
        b = dev(synth.gaussian_source(dims, 2975 + seed))
        _, info = lat.solve(b, 0.13, 1.0, 1e-10, inner_method=1, check_every=every)
        assert info["restarts"] == 0
        e = info["dslash_count"] - 5 - 2 * info["inner_calls"] - 4 * info["inner_iters_total"]
        assert e % 2 == 0 and 0 <= e <= 2 * info["inner_calls"]
        extra += e
        calls += info["inner_calls"]
    say(every, extra, calls)
    assert 0 < extra < 2 * calls
    # stopped by the iteration cap: nothing is left out
    _, info = lat.solve(b, 0.13, 1.0, 1e-10, inner_method=1, check_every=every, fixed_work=5, outer_maxit=1,
                        raise_on_error=False)
    rest = info["dslash_count"] - info["inner_calls"] * (4 + 4 * 5 + 2)
    assert rest == 5
    lat.close()


@pytest.mark.parametrize("inner,name", [(wc.FP32, "fp32"), (wc.FP16, "fp16")])
@pytest.mark.parametrize("every", [1, 500])
def test_kernel_table_has_the_launches_that_ran(inner, name, every):
    dims = (8, 8, 8, 8)
    lat = wc.Lattice(dims)
    lat.load_links(dev(synth.random_links(dims, 0.3, 1970)))
    seen = set()
    for seed in range(4):
        b = dev(synth.gaussian_source(dims, 2970 + seed))
        lat.solve(b, 0.13, 1.0, 1e-10, inner_prec=inner, check_every=every)
        lat.reset_kernel_stats()
        lat.set_timing(True)
        _, info = lat.solve(b, 0.13, 1.0, 1e-10, inner_prec=inner, check_every=every)
        lat.set_timing(False)
        st = lat.kernel_stats()
        hop, dh = st["mult_hopinv_" + name]["launches"], st["mult_dhat_" + name]["launches"]
        say(info, hop, dh)
        assert hop == dh and hop + dh == info["dslash_count"] - 5 - 2 * info["inner_calls"]
        seen.add(hop + dh - 4 * info["inner_iters_total"])
    assert seen == {0} if every == 1 else max(seen) > 0
    lat.close()
