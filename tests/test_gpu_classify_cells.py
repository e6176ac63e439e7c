"""The empty-space classification bit by bit: the occupancy words, read from the
metadata region that the caller owns (they are its last array), against every
cell's corners.  Bricks cross the places where the kernel's work is divided: 16
cells along y to a wave, 64 to a workgroup, the row above taken from the next
wave or the next tile, walks along z of 4 words and more."""
import numpy as np
import pytest

from oracle import encoders
from paper_1205_0282_amd import binding, synth

pytestmark = pytest.mark.gpu


def _align(n):
    return (n + 255) // 256 * 256


def _expected(g, so, storage, op, matters, K, sc, bi):
    """Occupancy bit of each cell of a ghosted brick's decoded values [z][y][x]."""
    f = np.float32

    def fma(a, b, c):
        return (a.astype(np.float64) * np.float64(b) + np.float64(c)).astype(f)
    csc, cbi = sc, bi
    if storage == "fp8":
        if op == "mip":
            g = fma(g, so[0], so[1])
        else:
            csc, cbi = f(sc * so[0]), fma(so[1:2], sc, bi)[0]
    n = [s - 1 for s in g.shape]
    c = np.stack([g[z:n[0] + z, y:n[1] + y, x:n[2] + x] for z in (0, 1) for y in (0, 1) for x in (0, 1)])
    mn, mx = c.min(0), c.max(0)
    m = fma(np.maximum(abs(mn), abs(mx)), f(2.0 ** -20), f(1e-30))
    il = np.minimum(np.clip(fma(mn - m, csc, cbi), 0, K - 1).astype(int), K - 2)
    ih = np.minimum(np.clip(fma(mx + m, csc, cbi), 0, K - 1).astype(int), K - 2) + 1
    count = np.concatenate([[0], np.cumsum(matters)])
    return count[ih + 1] - count[0 if op == "mip" else il] > 0


@pytest.mark.parametrize("storage", ["f32", "f16", "fp8"])
@pytest.mark.parametrize("dims,brick,K,op", [
    ((7, 15, 9), (8, 16, 16), 64, "composite"),             # 16 cells along y
    ((13, 31, 10), (13, 16, 10), 300, "composite"),         # 17, then 16
    ((70, 127, 6), (67, 64, 6), 37, "composite"),           # 65, then 64; 68 and 4 along x
    ((9, 62, 70), (9, 62, 70), 1025, "composite"),          # 63; 71 along z
    ((5, 129, 141), (5, 129, 141), 256, "mip"),             # 130; 142 along z
    ((34, 256, 3), (17, 128, 3), 4096, "composite"),        # 129 twice
    ((133, 17, 35), (133, 17, 35), 100, "mip"),             # 18; 134 along x
    ((340, 340, 139), (17, 17, 139), 64, "composite"),      # 400 bricks: walks of 8 words
    ((333, 333, 139), (9, 9, 139), 50, "mip"),              # 1369 bricks: walks of 32 words
])
def test_every_cell(storage, dims, brick, K, op):
    import torch
    rng = np.random.default_rng(K + dims[1])
    vol = rng.standard_normal(dims[::-1]).astype(np.float32)
    vmin, vmax = -2.0, 2.5
    tf = synth.random_tf(rng, K, 0.01)
    if op == "mip":
        tf[: K // 2] = tf[0]                                # a leading run of equal entries
        matters = (tf != tf[0]).any(1)
    else:
        tf[rng.uniform(size=K) < 0.7, 3] = 0.0              # holes: most entries transparent
        matters = tf[:, 3] != 0
    bc = binding.BrickCaster(0)
    bc.plan(dims, brick, storage=storage, max_w=16, max_h=16, max_tiles=64 * 1369)
    bc.bind()
    bc.load(torch.from_numpy(vol).cuda())
    bc.set_operator(op, "fixed")
    bc.set_transfer_function(tf, vmin, vmax)
    bc.set_views([synth.orbit_view(dims, 0, width=16, height=16)])
    bc.render()
    torch.cuda.synchronize()
    lohi, so, _ = bc.bricks()
    words = [[(n + 1 + 3) // 4, (m + 1 + 3) // 4, (k + 1 + 1) // 2] for n, m, k in (lohi[:, 3:] - lohi[:, :3])]
    total = sum(a * b * c for a, b, c in words)
    end = bc.planned_sizes[1]
    occ = bc.regions[1][end - _align(4 * total):][:4 * total].cpu().numpy().view(np.uint32)
    sc, bi = np.float32((K - 1) / (vmax - vmin)), np.float32(-vmin * ((K - 1) / (vmax - vmin)))
    e4m3 = encoders.e4m3_value(np.arange(256)).astype(np.float32)
    at = set_bits = cells = 0
    for k, (wx, wy, wz) in enumerate(words):
        lo, n = lohi[k, :3], lohi[k, 3:] - lohi[k, :3]
        if storage == "fp8" or k == 0:
            buf, padded = bc.read_brick(k)
            g = binding.unswizzle(buf, padded)[: n[2] + 2, : n[1] + 2, : n[0] + 2]
            g = e4m3[g] if storage == "fp8" else (g.view(np.float16).astype(np.float32) if storage == "f16" else g)
        else:
            ix = [np.clip(np.arange(lo[a] - 1, lo[a] + n[a] + 1), 0, dims[a] - 1) for a in (2, 1, 0)]
            g = vol[np.ix_(*ix)]
            if storage == "f16":
                g = g.astype(np.float16).astype(np.float32)
        want = _expected(g, so[k], storage, op, matters, K, sc, bi)
        w = occ[at:at + wx * wy * wz].reshape(wz, wy, wx)
        at += wx * wy * wz
        bit = np.arange(32)
        bits = (w[..., None] >> bit.astype(np.uint32)) & 1                        # [wz][wy][wx][z%2, y%4, x%4]
        got = bits.reshape(wz, wy, wx, 2, 4, 4).transpose(0, 3, 1, 4, 2, 5).reshape(2 * wz, 4 * wy, 4 * wx).astype(bool)
        cz, cy, cx = want.shape
        assert np.array_equal(got[:cz, :cy, :cx], want), k
        assert got.sum() == want.sum(), k                                         # nothing set past the cells
        set_bits += int(want.sum())
        cells += want.size
    assert 0 < set_bits < cells
    bc.close()
