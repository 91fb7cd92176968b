"""Stores brought back from blobs: the rebuilt block indexes and decode routes
on every launch shape of the index rebuild (few or many chunks per wave, chunks
longer than any encoder writes), against the store that was saved."""
import numpy as np
import pytest

from oracle import driver
from paper_2308_11759_amd import inputs

from helpers import oracle_run, store_blob

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape,n", [((3, 5, 4), 2), ((17, 30, 61), 5), ((128, 128, 132), 8), ((127, 129, 130), 9)])
def test_loaded_store_equals_saved(shape, n, dtype, codec):
    import torch

    from paper_2308_11759_amd import pmc

    print("load case", shape, n, dtype.__name__, codec, flush=True)
    ctx = pmc.Context(0)
    ctx.set_option(pmc.OPT_CODEC, codec)
    ctx.set_option(pmc.OPT_SYNC_CHECK, 1)
    x = inputs.spectral_field(shape, seed=n, dtype=dtype)
    x.reshape(-1)[::997] *= 2.0 ** 40  # raw and wide blocks among them
    store = ctx.compress(torch.from_numpy(x).to("cuda:0"), [2.0 ** (2 - 2.5 * i) for i in range(n)],
                         allow_bound_miss=True)
    loaded = ctx.deserialize(store.serialize())
    for k in (1, n):
        assert torch.equal(ctx.retrieve(loaded, k), ctx.retrieve(store, k))
    for a, b in zip(loaded.info, store.info):
        assert a == b


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("extra", [3000, 20000])
def test_chunks_longer_than_an_encoder_writes(extra, codec):
    """Words behind a chunk's last block belong to the chunk and are not read:
    beyond the staging buffers the unstaged readers take over."""
    import torch

    from paper_2308_11759_amd import pmc

    x = inputs.spectral_field((9, 18, 70), seed=6, dtype=np.float32)
    taus = [0.1, 0.004]
    comps, meta, recon = oracle_run(x, taus, driver.PredictionCodec() if codec else None)
    long = []
    for c in comps:
        c = np.concatenate([c, np.full(4 * extra, 0x5A, np.uint8)])
        c[56:64] = np.frombuffer(np.uint64(int(c[56:64].view(np.uint64)[0]) + extra).tobytes(), np.uint8)
        long.append(c)
    ctx = pmc.Context(0)
    ctx.set_option(pmc.OPT_SYNC_CHECK, 1)
    store = ctx.deserialize(store_blob(x.shape, x.dtype, long, meta, codec))
    for k in (1, 2):
        assert np.array_equal(ctx.retrieve(store, k).cpu().numpy(), recon[k - 1])
