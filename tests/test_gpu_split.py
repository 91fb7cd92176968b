"""Retrievals that decode one component per wave, and the float64 routes of
both kernels: every prefix, refinement and box against the oracle's decoding of
the same streams, bit for bit, on both sides of each rule (components per
launch, waves per launch, high-half words or not, words that fit LDS or not)."""
import numpy as np
import pytest

from oracle import driver
from paper_2308_11759_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    ((4, 4, 4), 2, 8.0, False),       # one block, two waves
    ((30, 37, 61), 8, 8.0, False),    # eight waves; float64 on the high-half routes
    ((30, 37, 61), 8, 300.0, False),  # wide residuals: off those routes, float64 four and four
    ((18, 22, 71), 9, 4.0, False),    # two launches of five and four
    ((17, 30, 61), 6, 6.0, True),     # raw blocks and wide first words; spans beyond LDS
    ((132, 132, 128), 3, 8.0, False),  # 545 waves: float64 decodes all components in one wave
]


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape,n,step,wild", CASES)
def test_retrievals_equal_the_oracle(shape, n, step, wild, dtype, codec):
    import torch

    from paper_2308_11759_amd import pmc

    print("split case", shape, n, step, dtype.__name__, codec, flush=True)
    ctx = pmc.Context(0)
    ctx.set_option(pmc.OPT_CODEC, codec)
    ctx.set_option(pmc.OPT_SYNC_CHECK, 1)
    x = inputs.spectral_field(shape, seed=n, dtype=dtype)
    if wild:
        x.reshape(-1)[::211] *= dtype(2.0) ** 60
        x.reshape(-1)[5::1009] = -0.0
    store = ctx.compress(torch.from_numpy(x).to("cuda:0"), [step ** (0.3 - i) for i in range(n)],
                         allow_bound_miss=True)
    loaded = ctx.deserialize(store.serialize())
    dec = driver.PredictionCodec() if codec else driver.BlockCodec()
    part = [np.zeros(shape, dtype)]
    for i in range(n):
        part.append(part[-1] + dec.decode(store.stream(i).cpu().numpy(), shape, dtype))
    nz, ny, nx = shape
    boxes = [((0, 0, 0), (nx, ny, nz)), ((1, 2, 3), (nx - 1, ny - 1, nz)), ((nx // 2, 1, 0), (nx // 2 + 1, 4, 2))]
    for k in range(1, n + 1):
        for st in (store, loaded):
            assert np.array_equal(ctx.retrieve(st, k).cpu().numpy(), part[k]), k
        for lo, hi in boxes:
            got = ctx.retrieve_box(store, k, lo, hi).cpu().numpy()
            assert np.array_equal(got, part[k][lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]]), (k, lo, hi)
        out = ctx.retrieve(store, k)
        ctx.refine(store, k, n, out)
        assert np.array_equal(out.cpu().numpy(), part[n]), k
