"""Launches of more tiles than the device holds workgroups of the split for
few tiles take the local step's split for many: small images of every kind of
edge, many of each in one batch, against the oracle (tolerance 0)."""
import numpy as np
import pytest

from oracle import oracle_label
from paper_1712_09789_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TILES = 9000  # more than 2048 or, at 32 rows, 4096 workgroups


@pytest.fixture(scope="module")
def ccl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_09789_amd.ccl as c
    return c


def images():
    yy, xx = np.indices((130, 200))
    # vertical dominoes: the most runs a strip can have and an edge per column
    # between strips (more edges than the edge list takes)
    yield ((yy // 2 + xx) % 2 == 0).astype(np.uint8)
    yield (xx % 2 == 0).astype(np.uint8)  # the most runs per row, no edges
    yield wl.checkerboard(127, 129, value=255)
    yield wl.full(64, 64)
    yield wl.serpentine(129, 131, width=1, vertical=True)
    for k, (shape, p) in enumerate((((1, 1), 1.0), ((1, 200), 0.6), ((200, 1), 0.6),
                                    ((31, 63), 0.4), ((64, 65), 0.5), ((65, 64), 0.6),
                                    ((130, 190), 0.55), ((128, 128), 0.7))):
        yield wl.bernoulli(*shape, p, seed=k)


@pytest.mark.parametrize("rows", [32, 64, 128])
@pytest.mark.parametrize("conn", [4, 8])
def test_small_images_in_a_large_batch(ccl, conn, rows):
    imgs = list(images())
    want = [torch.from_numpy(oracle_label(im, conn)).cuda() for im in imgs]
    dev = [torch.from_numpy(im).cuda() for im in imgs]
    tiles = sum(-(-h // rows) * -(-w // 64) for h, w in (im.shape for im in imgs))
    times = -(-TILES // tiles)
    got = ccl.label_batch(dev * times, conn, tile_rows=rows)
    for k, g in enumerate(got):
        assert torch.equal(g, want[k % len(want)]), f"image {k % len(want)}, copy {k // len(want)}"
