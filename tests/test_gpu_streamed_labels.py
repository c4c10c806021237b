"""Label maps of at least 128 MiB whose rows are whole 128-byte lines are
written around the caches; neighbours of that rule are not.  Against closed
forms and the oracle (tolerance 0)."""
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


# streamed: whole tiles, a tile cut at 32 columns, few rows; not streamed:
# rows off 128 bytes, a map under 128 MiB
@pytest.mark.parametrize("shape", [(5800, 5824), (5823, 5792), (33, 1 << 20), (5800, 5796),
                                   (5776, 5792)])
@pytest.mark.parametrize("conn", [4, 8])
def test_large_maps(ccl, shape, conn):
    img = wl.bernoulli(*shape, 0.6 if conn == 4 else 0.4, seed=shape[0])
    d = torch.from_numpy(img).cuda()
    flat = torch.full((img.size + 96,), -1, dtype=torch.int32, device="cuda")
    want = torch.from_numpy(oracle_label(img, conn)).cuda()
    for off in (32, 33):  # on a 128-byte line, and off it
        out = flat[off:off + img.size].view(shape)
        ccl.label(d, conn, out=out)
        assert torch.equal(out, want)
        assert int(flat[off - 1]) == -1 and int(flat[off + img.size]) == -1
        flat.fill_(-1)


# maps of 256 MiB or more off 128-byte lines: tiles taken in pairs, with a last
# span of fewer than sixteen; one column less than the line; explicit heights
@pytest.mark.parametrize("shape,rows", [((8193, 8193), None), ((70, 958_700), None),
                                        ((8191, 8193), None), ((8193, 8195), 32),
                                        ((8193, 8195), 64)])
@pytest.mark.parametrize("conn", [4, 8])
def test_paired_tiles(ccl, shape, rows, conn):
    img = wl.bernoulli(*shape, 0.55 if conn == 4 else 0.4, seed=shape[0])
    d = torch.from_numpy(img).cuda()
    out = torch.full((img.size + 32,), -1, dtype=torch.int32, device="cuda")
    got = out[:img.size].view(shape)
    ccl.label(d, conn, out=got, **({"tile_rows": rows} if rows else {}))
    assert torch.equal(got, torch.from_numpy(oracle_label(img, conn)).cuda())
    assert int(out[img.size]) == -1


def test_batch_of_both_kinds(ccl):
    imgs = [wl.bernoulli(4000, 4096, 0.4, seed=1), wl.bernoulli(4100, 4001, 0.4, seed=2),
            wl.blobs(700, 96, 4.0, seed=3), wl.full(70, 64)]
    got = ccl.label_batch([torch.from_numpy(i).cuda() for i in imgs], 8)
    for im, g in zip(imgs, got):
        assert np.array_equal(g.cpu().numpy(), oracle_label(im, 8))
