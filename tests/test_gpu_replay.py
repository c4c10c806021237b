"""Replays of the two per-tile kernels in any order (ccl_replay_last): after a
replayed local step the relabel writes each tile's own labels, as
ccl_label_local does with the same tile height."""
import numpy as np
import pytest

from oracle import oracle_label
from paper_1712_09789_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ccl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_09789_amd.ccl as c
    return c


# merge in groups (2256 tiles; one group of 16), across every seam, one tile
@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("shape", [(3001, 3003), (200, 250), (640, 480), (50, 60)])
def test_relabel_after_the_local_step(ccl, shape, conn):
    img = wl.bernoulli(*shape, 0.5, seed=3)
    d = torch.from_numpy(img).cuda()
    want, tiles = oracle_label(img, conn), ccl.label_local(d, conn).cpu().numpy()
    out = ccl.label(d, conn, tile_rows=64)
    for _ in range(2):
        ccl.replay_last("local", 2)
        ccl.replay_last("final", 2)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), tiles)
    ccl.label(d, conn, out=out, tile_rows=64)
    ccl.replay_last("final", 1)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)


def test_relabel_after_the_local_step_of_a_batch(ccl):
    imgs = [wl.bernoulli(H, W, 0.5, seed=H) for H, W in ((1500, 1600), (50, 60), (1300, 1700))]
    devs = [torch.from_numpy(im).cuda() for im in imgs]
    outs = ccl.label_batch(devs, 8, tile_rows=64)
    ccl.replay_last("local", 1)
    ccl.replay_last("final", 1)
    torch.cuda.synchronize()
    for o, d in zip(outs, devs):
        assert torch.equal(o, ccl.label_local(d, 8))
