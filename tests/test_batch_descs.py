"""The two builders of batch descriptors in the binding: the fast one gives the
bytes of the general one, or leaves the call to it."""
import numpy as np
import pytest
import torch

import paper_1712_09789_amd.ccl as ccl


class _FakeDeviceTensor:
    """The tensor properties the descriptor builders read, for a tensor that
    claims to be on a device."""

    def __init__(self, t):
        self._t = t
        self.shape, self.dtype, self.is_cuda, self.device = t.shape, t.dtype, True, "dev"

    def get_device(self):
        return 0

    def __getattr__(self, name):
        return getattr(self._t, name)


@pytest.mark.parametrize("conn", [8, [4, 8, 4, 8]])
def test_batch_descriptors_fast_and_general(conn):
    base = torch.zeros((40, 60), dtype=torch.uint8)
    imgs = [base, base[3:9, 5:50], base[7:8, 1:2], base[2:3, :]]
    outs = [torch.zeros(i.shape, dtype=torch.int32) for i in imgs]
    fi, fo = [_FakeDeviceTensor(i) for i in imgs], [_FakeDeviceTensor(o) for o in outs]
    assert bytes(ccl._plain_descs(fi, fo, conn)) == bytes(ccl.make_descs(fi, fo, conn))
    # whatever the general path checks or refuses is left to it
    wide = _FakeDeviceTensor(torch.zeros((4, 8), dtype=torch.int32)[:, ::2])
    o4 = _FakeDeviceTensor(torch.zeros((4, 4), dtype=torch.int32))
    img = _FakeDeviceTensor(torch.zeros((4, 4), dtype=torch.uint8))
    for im, o, c in ((_FakeDeviceTensor(torch.zeros((4, 8), dtype=torch.uint8)[:, ::2]), o4, 8),
                     (_FakeDeviceTensor(torch.zeros((1, 4), dtype=torch.uint8).expand(4, 4)), o4, 8),
                     (_FakeDeviceTensor(torch.zeros((4, 4), dtype=torch.int8)), o4, 8),
                     (_FakeDeviceTensor(torch.zeros((0, 4), dtype=torch.uint8)),
                      _FakeDeviceTensor(torch.zeros((0, 4), dtype=torch.int32)), 8),
                     (torch.zeros((4, 4), dtype=torch.uint8), o4, 8),
                     (img, torch.zeros((4, 4), dtype=torch.int32), 8),
                     (img, wide, 8), (img, _FakeDeviceTensor(torch.zeros((4, 4))), 8),
                     (img, o4, "x"), (np.zeros((4, 4), np.uint8), o4, 8)):
        assert ccl._plain_descs([im], [o], c) is None
    assert ccl._plain_descs([img], [], 8) is None and ccl._plain_descs([], [], 8) is None
