"""Compression's staging and pack, where they can go wrong: component counts
around the workspace's layouts, spans of one and of several emission windows,
spans that outgrow their slot together (the components then run one launch
each), and fields on both sides of the pack's small-field limit.  Streams,
measured errors and block counts equal the oracle's byte for byte."""
import numpy as np
import pytest

from oracle import driver
from paper_2308_11759_amd import inputs

pytestmark = pytest.mark.gpu


def wide_field(shape, dtype, seed):
    """Magnitudes log-uniform over a range that no block exponent spans: every
    component codes its share of bits for all samples."""
    rng = np.random.Generator(np.random.PCG64(seed))
    span = 50 if dtype == np.float32 else 150
    return (rng.choice([-1.0, 1.0], size=shape) * 2.0 ** rng.uniform(-span, span, size=shape)).astype(dtype)


def wide_taus(dtype):
    return [2.0 ** (46 - 4 * i) for i in range(28)] if dtype == np.float32 else [2.0 ** (142 - 9 * i) for i in range(32)]


def oracle_streams(x, taus, codec):
    return driver.compress(x, taus, driver.PredictionCodec() if codec else None)


def same(store, comps, meta, label):
    for i in range(len(comps)):
        got = store.stream(i).cpu().numpy()
        assert got.size == comps[i].size and np.array_equal(got, comps[i]), "%s: stream %d" % (label, i)
        info = store.info[i]
        assert info["linf"] == meta[i]["linf"], (label, i)
        for key in ("nempty", "ncoded", "nraw", "nesc", "nmiss"):
            assert info[key] == meta[i][key], (label, i, key)


def compress(x, taus, codec=0):
    import torch

    from paper_2308_11759_amd import pmc

    print("staging case", x.shape, x.dtype, len(taus), codec, flush=True)
    ctx = pmc.Context(0)
    ctx.set_option(pmc.OPT_CODEC, codec)
    return ctx.compress(torch.from_numpy(x).to("cuda:0"), taus, allow_bound_miss=True)


@pytest.mark.parametrize("codec", [0, 1])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(9, 10, 70), (8, 16, 128)])
def test_spans_beyond_the_slot(shape, dtype, codec):
    x, taus = wide_field(shape, dtype, 5), wide_taus(dtype)
    comps, meta = oracle_streams(x, taus, codec)
    blocks = np.prod([(d + 3) // 4 for d in shape])
    payload = sum(c.size - 64 - 4 * ((blocks + 15) // 16) for c in comps)
    assert payload > blocks * 64 * 3 * np.dtype(dtype).itemsize + 4096  # more than three raw components
    same(compress(x, taus, codec), comps, meta, "wide")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 32])
def test_component_counts(n, dtype):
    x = inputs.spectral_field((13, 9, 35), seed=3, dtype=dtype)
    x[0, 0, :8] = wide_field((8,), dtype, 1)  # raw blocks among them
    taus = [2.0 ** (-1 - 0.75 * i) for i in range(n)]
    comps, meta = oracle_streams(x, taus, 0)
    same(compress(x, taus), comps, meta, "n=%d" % n)


@pytest.mark.parametrize("shape", [(4, 512, 512), (4, 512, 516), (5, 511, 514)])
def test_small_field_limit_of_the_pack(shape):
    x = inputs.spectral_field(shape, seed=4, dtype=np.float32)
    taus = [0.25, 0.01]
    comps, meta = oracle_streams(x, taus, 0)
    same(compress(x, taus), comps, meta, "pack %s" % (shape,))


@pytest.mark.parametrize("bits", [5, 7, 9, 20])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_spans_of_several_windows(dtype, bits):
    rng = np.random.Generator(np.random.PCG64(bits))
    x = rng.uniform(-1.0, 1.0, size=(12, 12, 48)).astype(dtype)
    taus = [2.0 ** -bits, 2.0 ** -(bits + 3)]
    comps, meta = oracle_streams(x, taus, 0)
    same(compress(x, taus), comps, meta, "bits=%d" % bits)


def test_batch_with_a_field_beyond_its_slot():
    import torch

    from paper_2308_11759_amd import pmc

    cases = [(inputs.spectral_field((20, 21, 22), seed=1, dtype=np.float32), [0.1, 0.01, 0.001]),
             (wide_field((9, 10, 70), np.float32, 5), wide_taus(np.float32)),
             (inputs.spectral_field((8, 8, 8), seed=2, dtype=np.float64), [0.125])]
    ctx = pmc.Context(0)
    batch = ctx.batch([(x.shape, torch.from_numpy(x).dtype) for x, _ in cases], [t for _, t in cases])
    xs = [torch.from_numpy(x).to("cuda:0") for x, _ in cases]
    for _ in range(2):  # the graph after a call that left it, too
        stores = batch.compress(xs)
        for store, (x, taus) in zip(stores, cases):
            comps, meta = oracle_streams(x, taus, 0)
            same(store, comps, meta, "batch")
