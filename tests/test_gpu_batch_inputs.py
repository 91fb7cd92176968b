"""What pmc_batch_compress refuses as an input, pmc_batch_tune refuses too: both
hand the pointers to the same kernels."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


def test_bad_input_pointers_are_refused():
    import torch

    from paper_2308_11759_amd import pmc

    ctx = pmc.Context(0)
    xs = [torch.rand(8, 8, 8, device="cuda:0"), torch.rand(5, 6, 7, device="cuda:0")]
    batch = ctx.batch([(tuple(x.shape), x.dtype) for x in xs], [[0.1, 0.01]] * 2)
    room = torch.zeros(8 * 8 * 8 + 16, device="cuda:0")
    vp = ctypes.c_void_p
    for bad in (None, room.data_ptr() + 4):
        for i in range(2):
            ptrs = [x.data_ptr() for x in xs]
            ptrs[i] = bad
            arr = (vp * 2)(*ptrs)
            ms, out = ctypes.c_float(), (vp * 2)()
            buf = (vp(batch.ws.data_ptr()), batch.ws.numel(), vp(batch.streams.data_ptr()), batch.streams.numel())
            assert ctx.lib.pmc_batch_tune(batch.handle, arr, *buf, ctypes.byref(ms)) == pmc.E_ARG
            assert ctx.lib.pmc_batch_compress(batch.handle, arr, *buf, out) == pmc.E_ARG
    batch.tune(xs)
    for s, x in zip(batch.compress(xs), xs):
        assert float((ctx.retrieve(s, 2) - x).abs().max()) <= 0.01
