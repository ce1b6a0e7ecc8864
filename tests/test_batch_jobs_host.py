"""The job table of a batch compression (lopc.py), written as packed bytes: the
same members as stores to them one by one, also for modes that do not fit 32
bits, which a C int takes modulo 2^32 as the single-field call does."""
import ctypes

import pytest
import torch

from paper_2603_26968_amd import lopc


class Field:
    """What _compress_jobs asks of a device tensor."""
    is_cuda, device, dtype = True, torch.device("cuda:0"), torch.float32

    def __init__(self, shape, dtype=torch.float32):
        self.shape, self.dtype = torch.Size(shape), dtype

    def dim(self):
        return len(self.shape)

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 0x7000000 + 16 * self.shape[0]


class Out:
    def numel(self):
        return 1 << 40

    def data_ptr(self):
        return 0x9000000


@pytest.mark.parametrize("mode", [0, 1, "noa", "ABS", 3, -1, 2**31, 2**32, 2**32 + 1, -2**31 - 1, True])
def test_jobs_hold_what_was_given(monkeypatch, mode):
    monkeypatch.setattr(lopc, "lopc_ctx_get_option", lambda ctx, option: 0)
    fields = [Field((70, 61)), Field((9, 10, 11), torch.float64)]
    jobs, _, offs, _, _ = lopc._compress_jobs(fields, [1e-3, 2], mode, Out(), 0)
    for j, x, eb, off in zip(jobs, fields, (1e-3, 2.0), offs):
        want = lopc.Job()
        want.d_in, want.d_out = x.data_ptr(), 0x9000000 + off
        want.out_cap = lopc.lopc_compress_bound(x.shape, x.dtype)
        want.dtype, want.ndim = int(x.dtype == torch.float64), x.dim()
        for i, d in enumerate(x.shape):
            want.dims[i] = d
        want.error_bound = eb
        want.mode = lopc._mode(mode)
        assert bytes(j) == bytes(want)
        assert ctypes.sizeof(j) == ctypes.sizeof(want)
