"""Volumes through both paths of ccl_label_3d against the 3-D oracle
(tolerance 0): in bricks of 64 x 16 x 16 voxels through a workspace, and in
bricks of 64 x 8 x 8 in place, which a call under stream capture takes."""
import numpy as np
import pytest

from oracle import oracle_label3d
from paper_1712_09789_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PATHS = ("workspace", "in_place")


@pytest.fixture(scope="module")
def ccl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_09789_amd.ccl as c
    return c


def check(ccl, path, vols, conn, view=lambda d: d, out=None):
    """Labels each of `vols` (of one shape), `view` of it on the device."""
    dev = torch.from_numpy(vols[0]).cuda()
    src = view(dev)
    if out is None:
        out = torch.empty(src.shape, dtype=torch.int32, device="cuda")
    run = lambda: ccl.label_3d(src, conn, out=out)  # noqa: E731
    if path == "in_place":
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            run()
        run = g.replay
    for k, vol in enumerate(vols):
        print(f"[volume] {path} {tuple(src.shape)} conn={conn} {k}", flush=True)
        dev.copy_(torch.from_numpy(vol))
        out.fill_(-1)
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        got, want = out.cpu().numpy(), oracle_label3d(np.ascontiguousarray(view(vol)), conn)
        bad = np.argwhere(got != want)
        assert len(bad) == 0, (k, len(bad), bad[0], got[tuple(bad[0])], want[tuple(bad[0])])


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("path", PATHS)
def test_every_corner_pattern_where_bricks_meet(ccl, path, conn):
    # Every 2 x 2 x 2 pattern, isolated by background, centred on points where
    # eight bricks meet, and on points where four or two do along each axis
    step = 16 if path == "workspace" else 8
    shape = (5 * step, 5 * step, 512)
    corners = [(z, y, x) for z in range(step, shape[0], step) for y in range(step, shape[1], step)
               for x in range(64, 512, 64)]
    shifts = [(a, b, c) for a in (0, 4) for b in (0, 4) for c in (0, 20) if (a, b, c) != (4, 4, 20)]
    perm = np.random.default_rng(5).permutation(256)
    vols = []
    for n0 in range(0, 256, len(corners)):
        vol = np.zeros(shape, np.uint8)
        for k, shift in enumerate(shifts):
            for i, corner in enumerate(corners):
                z, y, x = np.add(corner, shift)
                p = int(perm[(n0 + i + 37 * k) % 256])
                vol[z - 1:z + 1, y - 1:y + 1, x - 1:x + 1] = \
                    np.array([(p >> b) & 1 for b in range(8)], np.uint8).reshape(2, 2, 2)
        vols.append(vol)
    check(ccl, path, vols, conn)


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("shape", [(48, 64, 256), (33, 49, 193), (17, 15, 321)])
def test_contents(ccl, path, shape, conn):
    vols = [wl.bernoulli3d(*shape, p, seed=int(100 * p)) for p in (0.1, 0.3, 0.6)]
    vols += [wl.make3d(k, *shape, seed=1) for k in ("blobs", "checkerboard", "full", "slabs")]
    check(ccl, path, vols, conn)


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("off", [0, 1, 2])
def test_strided_view_and_unaligned_labels(ccl, path, off, conn):
    vols = [wl.bernoulli3d(40, 70, 300, p, seed=4) * np.uint8(200) for p in (0.15, 0.3, 0.5)]
    flat = torch.empty(37 * 60 * 290 + off, dtype=torch.int32, device="cuda")
    check(ccl, path, vols, conn, lambda d: d[1:38, 3:63, 5:295], flat[off:].view(37, 60, 290))


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("path", PATHS)
def test_repeated_merges(ccl, path, conn):
    # the merge races on its forest or on the label map: the same volume again
    # and again
    check(ccl, path, [wl.bernoulli3d(64, 96, 160, 0.35 if conn == 6 else 0.12, seed=9)] * 20, conn)


# the line of thin volumes: up to 4096 bricks of 64 x 16 x 16, an eighth full,
# through a workspace, more of them in place; bricks over a third full stay with
# the workspace
@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("shape", [(2, 16, 64 * 4096), (2, 16, 64 * 4096 + 1), (6, 16, 64 * 4096 + 1)])
def test_thin_volumes(ccl, shape, conn):
    check(ccl, "eager", [wl.bernoulli3d(*shape, 0.35 if conn == 6 else 0.15, seed=2)], conn)
