"""The one-level merge of small launches (at most 512 tiles with a seam between
merge groups) against the oracle, and both sides of that line (tolerance 0)."""
import numpy as np
import pytest

from oracle import oracle_label
from paper_1712_09789_amd import workloads as wl
from seam_atlas import Layout

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZE = {32: 1024, 64: 1024, 128: 2048}  # at most 512 tiles, by tile height
GROUP_PX = 256


@pytest.fixture(scope="module")
def ccl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_09789_amd.ccl as c
    return c


@pytest.mark.parametrize("rows", [32, 64, 128])
@pytest.mark.parametrize("conn", [4, 8])
def test_patterns_on_every_seam_kind(ccl, conn, rows):
    cols = ccl.tile_shape()[1]
    size = SIZE[rows]
    L = Layout(size, size, rows, cols, (GROUP_PX // rows, GROUP_PX // cols), conn, "cuda")
    for n in np.linspace(0, L.n_images - 1, 12).astype(int):
        pid = L.assemble(int(n))
        got = ccl.label(L.img.view(size, size), conn, tile_rows=rows).view(-1)
        bad = torch.nonzero(got != L.want)
        assert len(bad) == 0, f"image {n}: {L.describe(pid, int(bad[0]))}"


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("shape", [(2048, 2048), (2048, 2049), (1, 300), (300, 1), (129, 257)])
def test_both_sides_of_the_line(ccl, shape, conn):
    H, W = shape
    for img in (wl.serpentine(H, W), wl.bernoulli(H, W, 0.41 if conn == 8 else 0.6, seed=3)):
        want = oracle_label(img, conn)
        d = torch.from_numpy(img).cuda()
        assert np.array_equal(ccl.label(d, conn).cpu().numpy(), want)


@pytest.mark.parametrize("conn", [4, 8])
def test_small_images_merged_in_groups(ccl, conn):
    # beside an image of more than 512 tiles the same small images take the
    # two-level merge
    imgs = [wl.bernoulli(300, 517, 0.5, seed=1), wl.spiral(257, 600), wl.full(520, 130),
            wl.blobs(700, 301, 4.0, seed=2)]
    want = [oracle_label(im, conn) for im in imgs]
    d = [torch.from_numpy(im).cuda() for im in imgs]
    big = torch.zeros((2100, 2100), dtype=torch.uint8, device="cuda")
    alone = ccl.label_batch(d, conn)
    beside = ccl.label_batch(d + [big], conn)
    for w, a, b in zip(want, alone, beside):
        assert np.array_equal(a.cpu().numpy(), w)
        assert np.array_equal(b.cpu().numpy(), w)
