"""Compression of data whose components outgrow the staging slots: the launches
after the first go on from the components in place instead of beginning again.
Streams, measured errors and counts equal the oracle's, whatever wave gives up
at whatever component, and the launches stay few."""
import re

import numpy as np
import pytest

from oracle import driver
from paper_2308_11759_amd import inputs
from test_gpu_staging import oracle_streams, same, wide_field, wide_taus

pytestmark = pytest.mark.gpu


def setup(codec=0):
    from paper_2308_11759_amd import pmc

    ctx = pmc.Context(0)
    ctx.set_option(pmc.OPT_CODEC, codec)
    ctx.set_option(pmc.OPT_PROFILE, 1)
    return ctx


def launches(ctx, prefix):
    return sum(v[0] for k, v in ctx.prof_read(reset=True).items() if k.startswith(prefix))


def mixed_field(shape, dtype):
    """Waves that outgrow their slot early, late and not at all."""
    x = inputs.spectral_field(shape, seed=9, dtype=dtype)
    z = shape[0] // 3
    x[:z] = wide_field((z,) + shape[1:], dtype, 6)
    x[z:2 * z] = wide_field((z,) + shape[1:], dtype, 7) * dtype(2.0 ** -20)
    return x


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(24, 16, 64), (25, 18, 70), (4, 4, 4)])
def test_few_launches_and_the_oracles_streams(shape, dtype, codec):
    import torch

    from paper_2308_11759_amd import pmc

    x = mixed_field(shape, dtype) if shape != (4, 4, 4) else wide_field(shape, dtype, 8)
    taus = wide_taus(dtype)
    print("resume case", shape, dtype.__name__, codec, flush=True)
    comps, meta = oracle_streams(x, taus, codec)
    xd = torch.from_numpy(x).to("cuda:0")
    ctx = setup(codec)
    for fused in (1, 0):
        ctx.set_option(pmc.OPT_FUSED_DECODE, fused)
        launches(ctx, "")
        same(ctx.compress(xd, taus, allow_bound_miss=True), comps, meta, "mixed")
        # (a launch adds at least the room of its slots less one raw component:
        # 31 of 64 bits per value, 62 in float64)
        assert launches(ctx, "k_encode") <= 1 + len(taus) // 4
    same(ctx.compress_static(xd, taus), comps, meta, "static")


def test_stream_buffer_too_small_reports_the_size():
    import torch

    from paper_2308_11759_amd import pmc

    x, taus = wide_field((9, 10, 70), np.float32, 5), wide_taus(np.float32)
    comps, meta = oracle_streams(x, taus, 0)
    xd = torch.from_numpy(x).to("cuda:0")
    ctx = setup()
    blocks = 3 * 3 * 18
    need = len(taus) * ((4 * blocks + 255) // 256 * 256)
    for c in comps:
        need = (need + 255) // 256 * 256 + len(c)
    for cap in (need - 1, need // 2, need // 4):
        buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda:0")
        with pytest.raises(pmc.PmcError) as err:
            ctx.compress(xd, taus, streams=buf[:cap])
        assert int(re.search(r"need (\d+) bytes", str(err.value)).group(1)) == need
        assert bool((buf[cap:] == 0xA5).all())
    same(ctx.compress(xd, taus, streams=buf[:need]), comps, meta, "exact capacity")


def test_batch_goes_on_with_the_fields_that_need_it():
    import torch

    cases = [(inputs.spectral_field((20, 21, 22), seed=1, dtype=np.float32), [0.1, 0.01, 0.001]),
             (mixed_field((25, 18, 70), np.float32), wide_taus(np.float32)),
             (inputs.spectral_field((8, 8, 8), seed=2, dtype=np.float64), [0.125]),
             (wide_field((9, 10, 70), np.float64, 3), wide_taus(np.float64)),
             (wide_field((8, 8, 16), np.float32, 4), wide_taus(np.float32)[:20])]
    want = [oracle_streams(x, taus, 0) for x, taus in cases]
    ctx = setup()
    batch = ctx.batch([(x.shape, torch.from_numpy(x).dtype) for x, _ in cases], [t for _, t in cases])
    xs = [torch.from_numpy(x).to("cuda:0") for x, _ in cases]
    for order in (0, 1, 2):
        batch.schedule(2, order)
        launches(ctx, "")
        stores = batch.compress(xs)
        assert 1 <= launches(ctx, "batch_resumed") <= 8  # (a quarter of the most components)
        for store, (comps, meta) in zip(stores, want):
            same(store, comps, meta, "batch")
            k = len(comps)
            got = ctx.retrieve(store, k).cpu().numpy()
            assert np.array_equal(got, driver.reconstruct(comps, k, got.shape, got.dtype))
