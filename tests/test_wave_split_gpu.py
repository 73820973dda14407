"""The automatic form of the GEMMs (wave-split kernel) on the GPU: plain, with
the fused epilogues and grouped, at the sizes where its tile or K split
changes and at the edges of those tiles, against the oracle, and against an
explicit tiled configuration on every output.

Bounds.  A weight is rounded to binary16 once (relative 2^-11), the sum of K
products runs in binary32 and the result is rounded to binary16 once.  With
A = sum |x||w| of an output:
    |y - ref| <= (2^-11 + K 2^-24) A + 2^-11 |ref| + 2^-25
(2^-25: half the spacing of subnormal results).  Two kernels use the same
rounded weights and differ by the order of their sums and the last rounding:
    |y1 - y2| <= 2 K 2^-24 A + 2^-10 |y| + 2^-24."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_10076_amd as Q
from gpu_util import Packed, f16_values, from_dev_y, rand_case, say, to_dev_x

pytestmark = pytest.mark.gpu

U16, U32 = 2.0 ** -11, 2.0 ** -24


def _sample(N):
    """Columns of the first and last n-tiles and of some between."""
    return np.unique(np.concatenate([np.arange(min(16, N)), np.arange(N - 16, N),
                                     np.linspace(0, N - 1, 24).astype(int)]))


def _reference(x, q, z, s, cols):
    """(oracle result, A) on `cols`."""
    W = oracle.dequant(q[:, cols], z[:, cols], s[:, cols])
    return oracle.gemm(x, q, z, s, cols=cols), np.abs(f16_values(x)) @ np.abs(W)


def _check(y, ref, bound):
    assert np.all(np.isfinite(y))
    worst = float(np.max(np.abs(y - ref) / bound))
    say("  worst error / bound %.3f" % worst)
    assert worst <= 1.0


# (M, N, K): rows at the edges of tiles of 16 to 128 rows, ragged columns, one
# k-group (waves without any), odd numbers of k-groups, two and more K slices
SIZES = [(3, 9744, 11008), (16, 5120, 5120), (9, 6144, 1024), (16, 12288, 512), (9, 528, 128), (13, 15360, 640),
         (17, 16, 128), (17, 16, 384), (17, 16, 11008), (31, 48, 128), (33, 272, 11008), (63, 528, 11008),
         (33, 528, 11008), (33, 2032, 11008), (97, 1040, 896), (97, 1040, 384), (65, 784, 11008), (49, 528, 11008),
         (129, 1360, 11008), (200, 1648, 4224), (112, 1376, 11008), (257, 1808, 384), (129, 1648, 1152),
         (97, 1040, 11008), (333, 2960, 640), (257, 1648, 11008), (449, 3088, 11008), (1025, 240, 1152),
         (333, 80, 11008), (1025, 464, 384), (257, 784, 11008), (1025, 912, 384), (333, 2960, 384), (200, 1664, 11008),
         (97, 1552, 11008), (257, 1824, 896), (65, 688, 11008), (449, 2432, 4224), (449, 4112, 384), (449, 2416, 11008),
         (257, 2464, 4224), (1347, 1424, 640), (129, 2736, 11008), (1025, 4448, 1664), (641, 4432, 384),
         (257, 2464, 11008), (641, 5424, 896), (333, 2704, 11008), (449, 12320, 4224), (1025, 9632, 384),
         (641, 4624, 384), (641, 5392, 384), (641, 6976, 4224), (1025, 7232, 384), (1347, 8880, 384),
         (449, 6576, 384), (1025, 6432, 384), (1025, 4944, 4224), (1347, 7312, 384), (1347, 9904, 384)]


# ... chosen so that with the ones above every tile of the form runs (checked
# without a GPU in test_launch_plan.py), those of one K range with an odd number
# of k-groups that goes round the rings of weights and activations several times
SIZES += [(17, 32, 1152), (17, 32, 5504), (97, 2736, 1152), (129, 5456, 1152), (225, 4112, 1152), (129, 4096, 1152),
          (333, 8208, 1152), (449, 6544, 1152), (897, 8224, 1152), (513, 8080, 1152), (897, 8208, 1152),
          (1347, 8848, 1152), (700, 9232, 1152), (1025, 9616, 1152), (1347, 9744, 1152)]


@pytest.mark.parametrize("M,N,K", SIZES)
def test_automatic_form(M, N, K):
    x, q, z, s = rand_case(M * 7 + N + K, M, K, N)
    say("automatic M=%d N=%d K=%d" % (M, N, K))
    p = Packed(q, z, s)
    xd = to_dev_x(x)
    y = p.gemm(xd)
    tiled = p.gemm(xd, cfg=Q.make_config(variant=2, split_k=1, tile_m=64 if M > 16 else 16, tile_n=32))
    torch.cuda.synchronize()
    cols = _sample(N)
    ref, A = _reference(x, q, z, s, cols)
    _check(f16_values(from_dev_y(y))[:, cols], ref, (U16 + K * U32) * A + U16 * np.abs(ref) + 2.0 ** -25)
    # every output; A <= |x row| |w column|, |w| <= 15 s
    xn = xd.float().norm(dim=1)
    wn = torch.from_numpy((f16_values(s) ** 2).sum(axis=0) * 128).sqrt().float().cuda() * 15
    bound = 2 * K * U32 * xn[:, None] * wn[None, :] + 2 * U16 * tiled.float().abs() + 2.0 ** -24
    assert bool(((y.float() - tiled.float()).abs() <= bound).all())
    # repeated: the same bits (the order of every sum is fixed)
    assert torch.equal(p.gemm(xd), y)


EPILOGUES = [(16, 12288, 512), (17, 32, 128), (33, 2048, 11008), (65, 672, 11008),
             (97, 1056, 384), (129, 1632, 1152), (48, 20512, 256), (128, 10272, 384),
             (33, 2080, 5504), (65, 2080, 11008), (257, 6560, 1152), (700, 9248, 1152)]


@pytest.mark.parametrize("M,N,K", EPILOGUES)
def test_automatic_form_with_epilogues(M, N, K):
    """Bias, and bias with the gated SiLU (a gate tile and its up tile end up
    in one wave whatever the tile), with one K slice, with the reduction pass and
    (33 and 65 rows) in the last of two slices to arrive.  With h the GEMM's bound E: silu' <= 1.1,
    |silu(g)| <= |g|, so the product moves by 1.1 E |u| + |g| E + 1.1 E^2 at most."""
    x, q, z, s = rand_case(M + 3 * N + K, M, K, N)
    b = np.random.Generator(np.random.PCG64(M)).uniform(-2, 2, N).astype(np.float16).view(np.uint16)
    bd = torch.from_numpy(b.view(np.int16)).cuda().view(torch.float16)
    p = Packed(q, z, s)
    xd = to_dev_x(x)
    cols = np.unique(np.concatenate([np.arange(32), np.arange(N - 32, N)]))
    ref, A = _reference(x, q, z, s, cols)
    h = ref + f16_values(b)[cols]
    E = (U16 + K * U32) * A + U32 * np.abs(h) + 2.0 ** -25
    say("epilogues M=%d N=%d K=%d" % (M, N, K))
    y = Q.gemm_fused(xd, p.dw, p.ds, p.dz, N, bias=bd)
    _check(f16_values(from_dev_y(y))[:, cols], h, E + U16 * np.abs(h))
    y = f16_values(from_dev_y(Q.gemm_fused(xd, p.dw, p.ds, p.dz, N, bias=bd, activation=Q.ACT_SILU_GATE)))
    for t in np.unique(cols // 32):   # pairs of tiles
        gi, ui = np.nonzero((cols // 16) == 2 * t)[0], np.nonzero((cols // 16) == 2 * t + 1)[0]
        g, u, Eg, Eu = h[:, gi], h[:, ui], E[:, gi], E[:, ui]
        want = g / (1 + np.exp(-g)) * u
        # 2^-20: the device's exponential and divide
        _check(y[:, 16 * t:16 * t + 16], want,
               1.1 * Eg * np.abs(u) + np.abs(g) * Eu + 1.1 * Eg * Eu + (U16 + 2.0 ** -20) * np.abs(want) + 2.0 ** -25)


# (rows of each expert, N, K): empty experts, one row, tiles that just fit and
# just do not, rows that fill several tiles unevenly
GROUPS = [((1, 0, 0), 32, 1152), ((0, 17, 16, 1, 33), 1040, 384), ((64, 65, 86), 1040, 1152), ((0, 2), 16, 640),
          ((129, 0, 469), 5952, 384), ((314, 600, 30), 5952, 384), ((97, 1003, 96), 7888, 384),
          ((300, 81, 89), 8576, 1152), ((128, 1, 1199), 8752, 384),
          # full and lower tiles of the other shapes
          ((77, 32), 6544, 4096), ((1047, 12), 208, 1152), ((733, 31), 16, 384), ((1160, 26), 3232, 384),
          ((219, 80), 16, 384), ((1120, 80), 4992, 1152)]


@pytest.mark.parametrize("counts,N,K", GROUPS, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_automatic_grouped_form(counts, N, K):
    T, E = 150, len(counts)
    rng = np.random.Generator(np.random.PCG64(sum(counts) + N))
    experts = [rand_case(1000 + e + N, 1, K, N)[1:] for e in range(E)]
    x = rand_case(N + K, T, K, 16)[0]
    rows = np.concatenate([np.sort(rng.integers(0, T, c)) for c in counts]).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    d = Q.to_device(*Q.pack_experts(experts))
    say("grouped counts=%s N=%d K=%d" % (counts, N, K))
    y = Q.grouped_gemm(to_dev_x(x), torch.from_numpy(offsets).cuda(), *d, N, rows=torch.from_numpy(rows).cuda())
    y = f16_values(from_dev_y(y))
    cols = _sample(N)
    for e in range(E):
        lo, hi = offsets[e], offsets[e + 1]
        if hi > lo:
            ref, A = _reference(x[rows[lo:hi]], *experts[e], cols)
            _check(y[lo:hi][:, cols], ref, (U16 + K * U32) * A + U16 * np.abs(ref) + 2.0 ** -25)
