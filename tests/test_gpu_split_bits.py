"""Retrievals and refinements with one wave per component and with one wave for
all of them give the same bits, the sign of zero included: each later
component is decoded onto -0 there, the neutral element of the sum."""
import numpy as np
import pytest

from paper_2308_11759_amd import inputs

pytestmark = pytest.mark.gpu


def bits(t):
    a = t.cpu().numpy()
    return a.view(np.uint32 if a.dtype == np.float32 else np.uint64)


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("step", [8.0, 300.0])
def test_same_bits_on_both_forms(step, dtype, codec):
    import torch

    from paper_2308_11759_amd import pmc

    n, shape = 6, (30, 37, 61)
    x = inputs.spectral_field(shape, seed=n, dtype=dtype)
    x[:8] = 0  # empty blocks in every component
    x[8:12] = -0.0
    print("split bits case", step, dtype.__name__, codec, flush=True)
    ctx = pmc.Context(0)
    ctx.set_option(pmc.OPT_CODEC, codec)
    store = ctx.compress(torch.from_numpy(x).to("cuda:0"), [step ** (0.3 - i) for i in range(n)],
                         allow_bound_miss=True)
    start = ctx.retrieve(store, 1)
    start.view(-1)[::3] = -0.0
    seen = {}
    for fused in (1, 0):  # (one component per launch: never split)
        ctx.set_option(pmc.OPT_FUSED_DECODE, fused)
        for k in range(2, n + 1):
            out = start.clone()
            ctx.refine(store, 1, k, out)
            got = (bits(ctx.retrieve(store, k)), bits(out))
            if fused:
                seen[k] = got
            else:
                assert all(np.array_equal(a, b) for a, b in zip(got, seen[k])), k
    # the negative zeros of empty blocks are still there, others became sums
    zeros = bits(start) == bits(torch.tensor([-0.0], dtype=start.dtype))[0]
    kept = seen[n][1][zeros] == bits(torch.tensor([-0.0], dtype=start.dtype))[0]
    assert kept.any() and not kept.all()
