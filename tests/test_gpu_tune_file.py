"""The tuner's results file and the two forms of the stencil: a stored shape is
taken only for the form that it was timed on.  Entries without the form field
come from the one-thread-per-site stencil; where a lattice's stencil gives each
tile four wavefronts they are left alone, and the first solve's shape follows
the lattice (64 threads and chunks of 64 tiles here)."""
import pytest

torch = pytest.importorskip("torch")

import synth
from gpu_checks import say

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1709_08785_amd as wc  # noqa: E402

SPLIT, SITES = (8, 8, 8, 16), (16, 16, 16, 36)  # FP16: four wavefronts a tile | one thread per site


def lattice(dims):
    lat = wc.Lattice(dims)
    lat.load_links(torch.from_numpy(synth.random_links(dims, 0.3, 1995)).to("cuda"))
    lat.build_clover(0.13, 1.0)
    return lat


def first_solve(dims, prec):
    lat = lattice(dims)
    b = torch.from_numpy(synth.gaussian_source(dims, 2995)).to("cuda")
    _, info = lat.solve(b, 0.13, 1.0, 1e-9, inner_prec=prec)
    shape = (info["block_size"], lat.xcd_chunk(prec))
    lat.close()
    return shape


@pytest.mark.parametrize("prec", [wc.FP32, wc.FP64])
@pytest.mark.parametrize("form,taken", [("1", True), ("0", False), (None, False)])
def test_split_form_takes_its_own_entries(tmp_path, prec, form, taken):
    path = tmp_path / "tune.txt"
    wc.set_tune_cache(str(path))
    try:
        lat = lattice(SPLIT)
        lat.tune_block_size(prec)
        lat.close()
        f = path.read_text().split()
        # wc-tune-v3 arch CUs Lx Ly Lz Lt prec recon pinned-cap threads chunk cap-mult cap-dhat us64 us128 us256 form
        assert len(f) == 18 and f[17] == "1"
        f[10], f[11] = "128", "8"
        path.write_text(" ".join(f[:17] + ([form] if form else [])) + "\n")
        shape = first_solve(SPLIT, prec)
        say(prec, form, shape)
        assert shape == ((128, 8) if taken else (64, 64))
    finally:
        wc.set_tune_cache(None)


@pytest.mark.parametrize("form,taken", [("0", True), (None, True), ("1", False)])
def test_site_form_takes_old_entries(tmp_path, form, taken):
    path = tmp_path / "tune.txt"
    wc.set_tune_cache(str(path))
    try:
        lat = lattice(SITES)
        lat.tune_block_size(wc.FP16)
        lat.close()
        f = path.read_text().split()
        assert len(f) == 18 and f[17] == "0"
        f[10], f[11] = "128", "0"  # a chunk that the tuner never stores
        path.write_text(" ".join(f[:17] + ([form] if form else [])) + "\n")
        shape = first_solve(SITES, wc.FP16)
        say(form, shape)
        assert (shape == (128, 0)) == taken
    finally:
        wc.set_tune_cache(None)


@pytest.mark.parametrize("dims,threads", [((16, 16, 16, 8), 64), ((12, 12, 12, 20), 256), ((16, 16, 16, 32), 256),
                                          ((14, 16, 18, 34), 64), ((16, 16, 20, 32), 64), ((16, 16, 16, 42), 256)])
def test_first_shape_follows_the_lattice(dims, threads):
    # 256, 270, 1024, 1071, 1280 and 1344 tiles
    assert first_solve(dims, wc.FP32) == (threads, 64 if dims[3] * dims[0] * dims[1] * dims[2] <= 1024 * 128 else 32)
