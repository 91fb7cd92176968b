"""A plane in which all 64 coefficients become significant at once: its section
is the longest the coder has, 127 bits, with the last terminator implied."""
import numpy as np
import pytest

from oracle import driver, lib

pytestmark = pytest.mark.gpu


def opens_full(block, dtype):
    """The block's first non-empty plane has a one for every coefficient."""
    _, _, u = lib.block_coeffs(block, dtype, 3)
    top = int(np.bitwise_or.reduce(u)).bit_length() - 1
    return top >= 0 and all((int(v) >> top) & 1 for v in u)


def full_plane_blocks(dtype, count, seed):
    """Blocks whose coefficients all have the same top plane, by decoding such
    coefficients (the transform loses only low bits of them)."""
    P = 32 if dtype == np.float32 else 64
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    while len(out) < count:
        top = int(rng.integers(P - 14, P - 4))
        u = (np.uint64(1) << np.uint64(top)) | rng.integers(0, 1 << (top - 2), size=64, dtype=np.uint64)
        block = lib.block_values(u, 1, dtype, 3).astype(dtype)
        if opens_full(block.astype(np.float64), dtype):
            out.append(block.reshape(4, 4, 4))
    return out


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(8, 8, 64), (9, 10, 70)])
def test_streams_equal_the_oracles(shape, dtype):
    import torch

    from paper_2308_11759_amd import pmc

    x = np.zeros(shape, dtype)
    blocks = full_plane_blocks(dtype, 24, 1)
    for j, b in enumerate(blocks):  # in the field's whole blocks, spread over the waves
        k = 5 * j + 1
        bx, by, bz = k % (shape[2] // 4), k // (shape[2] // 4) % (shape[1] // 4), j % (shape[0] // 4)
        x[4 * bz:4 * bz + 4, 4 * by:4 * by + 4, 4 * bx:4 * bx + 4] = b
    top = float(np.abs(x).max())
    taus = [top * 2.0 ** -(6 + 5 * i) for i in range(4)]
    print("full plane case", shape, dtype.__name__, flush=True)
    comps, meta = driver.compress(x, taus)
    xd = torch.from_numpy(x).to("cuda:0")
    ctx = pmc.Context(0)
    batch = ctx.batch([(shape, xd.dtype)], [taus])
    for store in (ctx.compress(xd, taus), batch.compress([xd])[0]):
        for i in range(len(taus)):
            assert np.array_equal(store.stream(i).cpu().numpy(), comps[i]), i
        out = ctx.retrieve(store, len(taus)).cpu().numpy()
        assert np.array_equal(out, driver.reconstruct(comps, len(taus), shape, x.dtype))
        assert float(np.abs(x.astype(np.float64) - out.astype(np.float64)).max()) <= taus[-1]
