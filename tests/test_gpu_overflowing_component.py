"""A stored component whose decoded values pass the largest double: they are
infinite before they are added, on every decode route, as in the oracle (an
encoder never accepts such a component, but a stream may hold one)."""
import struct

import numpy as np
import pytest

from helpers import store_blob
from oracle import driver, lib

pytestmark = pytest.mark.gpu

BIG = 1.2e308


def overflowing_stream(first, shape, blocks, tau, seed):
    """A stream like `first` whose blocks code random top ten planes at the
    largest exponent; tau = 2^1022 makes that ten planes."""
    rng = np.random.Generator(np.random.PCG64(seed))
    chunks, index = [], []
    for c in range(0, blocks, 16):
        bits = []
        for _ in range(c, min(c + 16, blocks)):
            u = rng.integers(0, 1 << 63, size=64, dtype=np.uint64) << np.uint64(1)
            buf, n = lib.encode_planes(u & ~np.uint64((1 << 54) - 1), 64, 10)
            bits += [1, 0, 0] + [(1024 + 1023 >> i) & 1 for i in range(11)]  # nonempty, coded, no escalation, emax
            bits += list(np.unpackbits(buf, bitorder="little")[:n])
        bits += [0] * (-len(bits) % 32)
        index.append(sum(len(w) for w in chunks) // 4)
        chunks.append(np.packbits(np.array(bits, np.uint8), bitorder="little").tobytes())
    payload = b"".join(chunks)
    head = bytearray(first[:64])
    head[32:44] = struct.pack("<di", tau, 1022)
    head[56:64] = struct.pack("<Q", len(payload) // 4)
    return np.frombuffer(bytes(head) + struct.pack("<%dI" % len(index), *index) + payload, np.uint8)


@pytest.mark.parametrize("shape", [(4, 4, 8), (12, 13, 70)])
def test_every_route_gives_the_oracles_infinities(shape):
    from paper_2308_11759_amd import pmc

    blocks = int(np.prod([(d + 3) // 4 for d in shape]))
    taus = [1.5 * 2.0 ** 1023, 2.0 ** 1022]
    x = np.full(shape, -BIG)
    x[..., 1::2] = BIG
    comps, _ = driver.compress(x, taus[:1])
    second = overflowing_stream(np.asarray(comps[0]).tobytes(), shape, blocks, taus[1], 3)
    with np.errstate(over="ignore"):
        want = np.zeros(shape) + lib.decode(np.asarray(comps[0]), shape, np.float64)
        added = lib.decode(second, shape, np.float64)
        want = want + added
        # some products overflow where their fused sum with x~_1 would not
        assert np.any(np.isinf(added) & (np.abs(x + np.clip(added, -1.7e308, 1.7e308)) < 1.7e308))
    print("overflow case", shape, int(np.isinf(want).sum()), flush=True)
    ctx = pmc.Context(0)
    blob = store_blob(shape, np.float64, [np.asarray(comps[0]), second], [dict(tau=t, linf=t) for t in taus])
    store = ctx.deserialize(blob)
    nz, ny, nx = shape
    for fused in (1, 0):
        ctx.set_option(pmc.OPT_FUSED_DECODE, fused)
        assert np.array_equal(ctx.retrieve(store, 2).cpu().numpy(), want, equal_nan=True), fused
    out = ctx.retrieve(store, 1)
    ctx.refine(store, 1, 2, out)
    assert np.array_equal(out.cpu().numpy(), want, equal_nan=True)
    assert np.array_equal(ctx.retrieve_box(store, 2, (0, 0, 0), (nx, ny, nz)).cpu().numpy(), want, equal_nan=True)
