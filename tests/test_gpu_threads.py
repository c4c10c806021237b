"""Several host threads calling the library on one stream, whose cached
workspaces they share, against the oracle (tolerance 0)."""
import threading

import numpy as np
import pytest

from oracle import oracle_label, oracle_label3d
from paper_1712_09789_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CALLS = 24


@pytest.fixture(scope="module")
def ccl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1712_09789_amd.ccl as c
    return c


def label_all(ccl, call, inputs):
    """Labels every input CALLS times, each in a thread of its own, all on the
    default stream."""
    devs = [torch.from_numpy(v).cuda() for v in inputs]
    outs = [[torch.full(v.shape, -1, dtype=torch.int32, device="cuda") for _ in range(CALLS)]
            for v in inputs]
    ccl.release_workspace()
    torch.cuda.synchronize()
    errors = []

    def work(i):
        try:
            for o in outs[i]:
                call(devs[i], o)
        except Exception as e:  # noqa: BLE001 (raised in the test's own thread below)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(inputs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    return outs


@pytest.mark.parametrize("conn", [6, 26])
def test_volumes(ccl, conn):
    # the second and third need larger workspaces than the first
    vols = [wl.bernoulli3d(*s, 0.3 if conn == 6 else 0.15, seed=s[2])
            for s in ((40, 50, 70), (64, 96, 200), (100, 120, 300))]
    outs = label_all(ccl, lambda d, o: ccl.label_3d(d, conn, out=o), vols)
    for v, got in zip(vols, outs):
        want = torch.from_numpy(oracle_label3d(v, conn)).cuda()
        assert all(torch.equal(o, want) for o in got), v.shape


@pytest.mark.parametrize("conn", [4, 8])
def test_images(ccl, conn):
    imgs = [wl.bernoulli(*s, 0.5, seed=s[1]) for s in ((200, 300), (700, 900), (1700, 2100))]
    outs = label_all(ccl, lambda d, o: ccl.label(d, conn, out=o), imgs)
    for im, got in zip(imgs, outs):
        want = torch.from_numpy(np.ascontiguousarray(oracle_label(im, conn))).cuda()
        assert all(torch.equal(o, want) for o in got), im.shape
