"""The workspace path of ccl_label_3d (volumes of 32 rows or more) and the
rules beside it, against the 3-D oracle (tolerance 0)."""
import numpy as np
import pytest

from oracle import oracle_label3d
from paper_1712_09789_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ccl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_09789_amd.ccl as c
    return c


def check(ccl, vol, conn, view=None, out=None):
    d = torch.from_numpy(np.ascontiguousarray(vol)).cuda() if view is None else view
    got = ccl.label_3d(d, conn, out=out)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle_label3d(vol, conn))


# both sides of the line at 32 rows; one brick; then remainders 1, 15, 16 along
# y and z and 1, 63, 64 columns along x
@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("shape", [(1, 31, 130), (1, 32, 130), (31, 1, 65), (32, 1, 65),
                                   (2, 16, 129), (3, 11, 1), (8, 8, 64), (17, 17, 65),
                                   (2, 9, 5), (16, 16, 64), (15, 16, 63), (49, 64, 705),
                                   (63, 65, 640), (48, 79, 767), (64, 256, 192)])
def test_edges_of_bricks(ccl, shape, conn):
    for p in (0.15, 0.35, 0.6):
        check(ccl, wl.bernoulli3d(*shape, p, seed=sum(shape)), conn)


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("kind", ["checkerboard", "full", "empty", "lattice", "lattice2",
                                  "dominoes", "blobs"])
def test_contents(ccl, kind, conn):
    shape = (50, 130, 449)
    if kind == "dominoes":
        # 2 x 2 x 1 pieces: the most runs a bundle of rows can have, and more
        # edges between bundles than the edge list takes
        z, y, x = np.indices(shape)
        vol = ((z // 2 + y // 2 + x) % 2 == 0).astype(np.uint8)
    elif kind.startswith("lattice"):
        # isolated voxels: the most components a brick can have (26), and a
        # second lattice that joins some of them diagonally
        vol = np.zeros(shape, np.uint8)
        vol[::2, ::2, ::2] = 1
        if kind == "lattice2":
            odd = vol[1::2, 1::2, 1::2]
            odd[...] = wl.bernoulli3d(*odd.shape, 0.2, seed=3)
    else:
        vol = wl.make3d(kind, *shape, seed=2)
    check(ccl, vol, conn)


# more bricks than fit the card at once, along y and z and with ends of rows in
# two bricks each
@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("shape", [(737, 721, 3), (8209, 17, 65)])
def test_many_bricks(ccl, shape, conn):
    check(ccl, wl.bernoulli3d(*shape, 0.13 if conn == 26 else 0.35, seed=9), conn)


@pytest.mark.parametrize("conn", [6, 26])
def test_pitched_view_and_unaligned_labels(ccl, conn):
    big = wl.bernoulli3d(60, 150, 460, 0.3, seed=4) * np.uint8(200)
    view = torch.from_numpy(big).cuda()[1:58, 2:147, 5:454]
    flat = torch.full((57 * 145 * 449 + 1,), -1, dtype=torch.int32, device="cuda")
    check(ccl, big[1:58, 2:147, 5:454], conn, view=view, out=flat[1:].view(57, 145, 449))
    assert int(flat[0]) == -1


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("shape", [(64, 256, 192), (33, 41, 131)])
def test_capture_replays_in_place(ccl, shape, conn):
    """Under capture the call labels in place (nothing is allocated, and the
    graph holds no pointer into this stream's workspace)."""
    vol = wl.bernoulli3d(*shape, 0.3, seed=6)
    d = torch.from_numpy(vol).cuda()
    out = torch.zeros(vol.shape, dtype=torch.int32, device="cuda")
    want = [oracle_label3d(v, conn) for v in (vol, 1 - vol)]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ccl.label_3d(d, conn, out=out)
    ccl.release_workspace()
    for k in (0, 1, 0):
        d.copy_(torch.from_numpy(vol if k == 0 else 1 - vol))
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want[k])


def test_volumes_leave_the_image_workspace_alone(ccl):
    """A graph captured from an image call keeps its workspace when a volume
    that needs a larger one is labelled on the same stream."""
    from oracle import oracle_label
    img = wl.bernoulli(300, 500, 0.55, seed=1)
    vol = wl.bernoulli3d(100, 200, 400, 0.3, seed=2)
    d, dv = torch.from_numpy(img).cuda(), torch.from_numpy(vol).cuda()
    out = torch.zeros(img.shape, dtype=torch.int32, device="cuda")
    outv = torch.zeros(vol.shape, dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        ccl.label(d, 8, out=out)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ccl.label(d, 8, out=out)
        held = ccl.workspace_cached(s)
        for conn in (6, 26):
            ccl.label_3d(dv, conn, out=outv)
            assert ccl.workspace_cached(s) == held
            out.zero_()
            g.replay()
            s.synchronize()
            assert np.array_equal(out.cpu().numpy(), oracle_label(img, 8))
            assert np.array_equal(outv.cpu().numpy(), oracle_label3d(vol, conn))
