"""GPU parity: every step of the hot path, through the C-ABI, against the CPU oracle.

Tolerances
  dequant / pack / index .......... bit-exact
  qlinear (GEMV and GEMM) ......... max |y - r| / max(|r|, rms_n r[m,:]) <= 2e-3, y the fp16 output,
                                    r the oracle's fp64 result (pure element-wise relative error is
                                    unbounded where r ~ 0)
  token NLL ....................... |per-sequence mean| <= 1e-3, per token <= 2e-3
"""
import math

import numpy as np
import pytest

import fq_synth
import oracle

pytestmark = pytest.mark.gpu

BITS = (2, 3, 4, 8)
TOL = 2e-3


@pytest.fixture(scope="module")
def fq():
    import paper_2501_07139_amd as mod

    return mod


@pytest.fixture(scope="module")
def torch():
    import torch as t

    assert t.cuda.is_available()
    return t


def qerr(y, r):
    """The qlinear error measure: |y - r| over max(|r|, row rms of r)."""
    y = np.asarray(y, dtype=np.float64)
    rms = np.sqrt(np.mean(r * r, axis=1, keepdims=True))
    den = np.maximum(np.abs(r), np.maximum(rms, 1e-30))
    return float(np.max(np.abs(y - r) / den))


def make_matrix(fq, seed, N, K, bits):
    W = fq_synth.weights(seed, N, K)
    codes, s, z = oracle.quantize_rtn(W, bits)
    return fq.PackedMatrix.from_host(codes, s, z, bits), codes, s, z


def dev(torch, a):
    if a.dtype == np.float16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.float16)
    return torch.from_numpy(a).cuda()


def host16(t):
    import torch as _t

    return t.cpu().view(_t.int16).numpy().view(np.float16)


# ------------------------------------------------------------------- dequant
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("shape", [(512, 512), (200, 384), (70, 256), (4096, 1024)])
def test_dequant_bit_exact(fq, torch, bits, shape):
    N, K = shape
    w, codes, s, z = make_matrix(fq, 7, N, K, bits)
    want = oracle.dequant(codes, s, z)
    got = fq.fq_dequant(w).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    got16 = host16(fq.fq_dequant(w, fp16=True))
    assert np.array_equal(got16.view(np.uint16), oracle.round_f16(want.astype(np.float64)).view(np.uint16))


@pytest.mark.parametrize("bits", BITS)
def test_dequant_arbitrary_codes_and_fractional_zeros(fq, torch, bits):
    N, K = 128, 512
    codes = fq_synth.codes(3, N, K, bits)
    s = (np.abs(fq_synth.activations(4, N, K // 128).astype(np.float32)) * 0.01 + 1e-4).astype(np.float16)
    z = (fq_synth.codes(5, N, K // 128, bits).astype(np.float32) / 16).astype(np.float16)
    w = fq.PackedMatrix.from_host(codes, s, z, bits)
    got = fq.fq_dequant(w).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), oracle.dequant(codes, s, z).view(np.uint32))


class Guarded:
    """A device buffer of `nbytes` with 4 KiB of a known pattern on either side."""
    PAD = 4096

    def __init__(self, torch, nbytes, fill=0xA5):
        self.torch, self.n = torch, nbytes
        self.raw = torch.full((nbytes + 2 * self.PAD,), fill, dtype=torch.uint8, device="cuda")
        self.fill = fill

    def bytes(self):
        return self.raw[self.PAD:self.PAD + self.n]

    def half(self, *shape):
        return self.bytes().view(self.torch.float16).view(*shape)

    def f32(self, *shape):
        return self.bytes().view(self.torch.float32).view(*shape)

    def intact(self):
        lo, hi = self.raw[:self.PAD], self.raw[self.PAD + self.n:]
        return bool((lo == self.fill).all().item()) and bool((hi == self.fill).all().item())


# ------------------------------------------------------------------- qlinear
GEMV_CASES = [(1, 512, 512), (16, 512, 512), (3, 200, 384), (1, 4096, 4096), (5, 70, 256), (1, 1, 128),
              (1, 160, 11008), (3, 96, 11008)]  # rows longer than one pass of the staging
GEMM_CASES = [(17, 512, 512), (64, 512, 512), (300, 200, 384), (520, 384, 1024), (33, 70, 256), (256, 64, 128)]


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", GEMV_CASES + GEMM_CASES, ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_against_oracle(fq, torch, bits, case):
    M, N, K = case
    w, codes, s, z = make_matrix(fq, 100 + bits, N, K, bits)
    X = fq_synth.activations(9, M, K)
    r = oracle.qlinear(X, oracle.dequant(codes, s, z))
    y = host16(fq.fq_qlinear(dev(torch, X), w))
    assert y.shape == (M, N)
    assert qerr(y, r) <= TOL
    # plain max-norm figure as well, for the record
    assert np.max(np.abs(y.astype(np.float64) - r)) / np.max(np.abs(r)) <= TOL


# The 256-row kernel (two halves of K per workgroup) in tiles of 8 blocks of sixteen rows, what matrices of so few columns are cut into: one group,
# odd and even group counts, ragged rows and columns
TALL_CASES = [(256, 128, 128), (300, 200, 384), (520, 384, 1024), (17, 70, 256), (512, 1030, 640), (700, 264, 2816)]


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", TALL_CASES, ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_tall_tiles_against_oracle(fq, torch, bits, case):
    M, N, K = case
    w, codes, s, z = make_matrix(fq, 120 + bits, N, K, bits)
    X = fq_synth.activations(11, M, K)
    r = oracle.qlinear(X, oracle.dequant(codes, s, z))
    out = Guarded(torch, M * N * 2)
    fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N), tile_rows=256)
    torch.cuda.synchronize()
    assert out.intact()
    y = host16(out.half(M, N))
    assert qerr(y, r) <= TOL
    # the 128-row kernel on the same inputs: same products, fp32 sums in another order
    y128 = host16(fq.fq_qlinear(dev(torch, X), w, tile_rows=128))
    assert qerr(y, y128.astype(np.float64)) <= 1e-3


# Few columns: their tiles fill one round however low, so the rows are cut into tiles of 8, 10 or 12 blocks of sixteen; whole blocks and ragged ones,
# in one row tile and in several
TALL_LOW = {121: (1, 128), 144: (1, 160), 150: (1, 160), 161: (1, 192), 177: (1, 192), 192: (1, 192), 208: (2, 128), 209: (2, 128), 225: (2, 128),
            240: (2, 128), 241: (2, 128), 300: (3, 128), 403: (4, 128), 611: (5, 128), 1200: (10, 128)}


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("M", TALL_LOW)
def test_qlinear_low_tall_tiles(fq, torch, bits, M):
    """Integer and fractional zeros (their loops differ); the last column of tiles is ragged."""
    N, K = 130, 384
    tiles, _, _, worked = fq.fq_qlinear_tall_tile(M, N, bits, K)
    assert (tiles, worked) == TALL_LOW[M]
    codes = fq_synth.codes(121, N, K, bits)
    s = np.random.default_rng(122).uniform(0.01, 0.02, (N, K // 128)).astype(np.float16)
    X = fq_synth.activations(123, M, K)
    for fraction in (0.0, 0.25):
        z = (fq_synth.codes(124, N, K // 128, bits).astype(np.float32) + fraction).astype(np.float16)
        r = oracle.qlinear(X, oracle.dequant(codes, s, z))
        out = Guarded(torch, M * N * 2)
        fq.fq_qlinear(dev(torch, X), fq.PackedMatrix.from_host(codes, s, z, bits), out=out.half(M, N), tile_rows=256)
        torch.cuda.synchronize()
        assert out.intact()
        assert qerr(host16(out.half(M, N)), r) <= TOL


# 256 columns of tiles: a row tile is a round of its own, so the tiles are as few and high as can be.  Every height, in one row tile and in
# several, that differ by a block too; whole blocks and ragged ones
TALL_WIDE = {119: (128,), 135: (160,), 151: (160,), 167: (192,), 183: (192,), 199: (208,), 208: (208,), 215: (224,), 231: (240,), 247: (256,), 256: (256,),
             281: (160, 160), 345: (192, 192), 397: (208, 192), 409: (208, 208), 429: (224, 208), 441: (224, 224), 461: (240, 224), 473: (240, 240),
             493: (256, 240), 505: (256, 256), 749: (256, 256, 240)}


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("K", [128, 384, 640])
@pytest.mark.parametrize("fraction", [0.0, 0.25])
def test_qlinear_tall_tiles_of_every_height(fq, torch, bits, K, fraction):
    """The first and last columns and sampled ones against the oracle, all of them against the 128-row kernel; one group and odd numbers of
    them, integer and fractional zeros, a last column of tiles that is ragged, guard bytes.

    The oracle takes the weights as the kernel has them, rounded to fp16 once (code - zero, of at most ten bits here, is exact): what is left is the
    result's own rounding, 2^-11 = 4.9e-4, and fp32 sums of 640 products, below 640 * 2^-24 = 4e-5 of sum |x w|, in practice 1e-6 of the rms."""
    N = 32707
    assert {h for heights in TALL_WIDE.values() for h in heights} == {128, 160, 192, 208, 224, 240, 256}
    rng = np.random.default_rng(125)
    codes = fq_synth.codes(126, N, K, bits)
    s = rng.uniform(0.01, 0.02, (N, K // 128)).astype(np.float16)
    z = (fq_synth.codes(127, N, K // 128, bits).astype(np.float32) + fraction).astype(np.float16)
    w = fq.PackedMatrix.from_host(codes, s, z, bits)
    cols = np.unique(np.concatenate([rng.integers(0, N, size=64), np.arange(128), np.arange(N - 80, N)]))
    sampled = oracle.dequant(codes[cols], s[cols], z[cols])
    X = fq_synth.activations(128, max(TALL_WIDE), K)
    r = oracle.qlinear(X, oracle.round_f16(sampled.astype(np.float64)).astype(np.float32))
    Xd, index = dev(torch, X), torch.from_numpy(cols).cuda()
    for M, heights in TALL_WIDE.items():
        tiles = [fq.fq_qlinear_tall_tile(M, N, bits, K, t) for t in range(len(heights))]
        assert tuple(t[3] for t in tiles) == heights and tiles[0][0] == len(heights), M
        out = Guarded(torch, M * N * 2)
        fq.fq_qlinear(Xd[:M], w, out=out.half(M, N), tile_rows=256)
        torch.cuda.synchronize()
        assert out.intact(), M
        assert qerr(host16(out.half(M, N)[:, index]), r[:M]) <= 5.2e-4, M
        # the 128-row kernel on the same inputs: same products, fp32 sums in another order
        y, y128 = out.half(M, N).float(), fq.fq_qlinear(Xd[:M], w, tile_rows=128).float()
        rms = y128.square().mean(1, keepdim=True).sqrt()
        assert float(((y - y128).abs() / torch.maximum(y128.abs(), rms)).max()) <= 1e-3, M


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", [(1, 5000, 128), (2, 5000, 1152), (1, 5120, 640), (3, 4100, 384), (1, 200, 8320)],
                         ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_decode_units_against_oracle(fq, torch, bits, case):
    """Between 4096 and 8192 rows the decode kernel hands 3-bit supertile rows out by halves; rows that end inside a
    half, K of fewer groups than wavefronts and of whole and broken turns of their ring, long rows of 4 bits."""
    M, N, K = case
    w, codes, s, z = make_matrix(fq, 80, N, K, bits)
    X = fq_synth.activations(81, M, K)
    out = Guarded(torch, M * N * 2)
    fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N))
    assert out.intact()
    # One rounding to fp16 (2^-11), and the kernel's codes carry a bias of 1024 that leaves each group's sum by
    # subtraction: its roundings in fp32 are 2^-24 of 1024 sum |x|, against 2-bit codes and K = 128 up to 5e-4 of the
    # row's rms each, a few of them per group.
    r = oracle.qlinear(X, oracle.dequant(codes, s, z))
    assert qerr(host16(out.half(M, N)), r) <= TOL


# Shapes of the few-row kernel: its tiles of up to 64 rows (16/32/48/64 rows x 16/32/64 columns) at every width, as the library
# chooses them (tests/test_host.py holds this list and the next against the rule), row tiles that end inside a block of sixteen, column
# counts that end inside a tile or a block, K of one group, of fewer groups than wavefronts, of one more than a whole
# turn of them, and of several turns.
SKINNY_CASES = [(4, 512, 128), (16, 70, 1152), (9, 11008, 384), (17, 4096, 1152), (17, 8200, 1152), (33, 4096, 1152),
                (48, 11008, 384), (60, 4096, 2176), (64, 11008, 1152), (77, 4096, 1152), (100, 201, 256),
                (128, 4096, 1152), (200, 4096, 1152), (250, 1030, 1280), (5, 4150, 384), (1036, 98, 128), (620, 230, 896),
                (1045, 193, 128),
                # one block a tile, where wavefronts have no group: one of them, most, none
                (20, 70, 896), (21, 68, 256), (33, 40, 1024)]


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", SKINNY_CASES, ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_few_rows_against_oracle(fq, torch, bits, case):
    """Integer zeros, then zeros with fractions in some groups (the kernel unpacks those differently).

    Bound: one rounding of the output to fp16 (2^-11 |r|), and where the tile scales its weights in fp16 one more of
    each weight, at worst 2^-11 sum |x||w|; differences of a code and a fractional zero are exact here, fp32 sums add
    1e-6 sum |x||w|.  The scales spread over an order of magnitude, so the largest of half a million errors is well over the
    2e-3 of the row's rms that evenly scaled weights stay below; rounding errors being independent, the rms over
    all outputs has to stay at sqrt(2) of one rounding (2^-11 / sqrt(3) at most), 4e-4."""
    M, N, K = case
    codes = fq_synth.codes(60, N, K, bits)
    s = (np.abs(fq_synth.activations(61, N, K // 128).astype(np.float32)) * 0.01 + 1e-3).astype(np.float16)
    X = fq_synth.activations(62, M, K)
    for frac in (0, 1):
        z = fq_synth.codes(63, N, K // 128, bits).astype(np.float32)
        if frac:
            z[::3, ::2] += 0.25
        z = z.astype(np.float16)
        w = fq.PackedMatrix.from_host(codes, s, z, bits)
        out = Guarded(torch, M * N * 2)
        assert fq.fq_qlinear_route(M, N, bits, K)[0] == "few_rows"
        fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N))
        assert out.intact()
        W = oracle.dequant(codes, s, z)
        r, size = oracle.qlinear(X, W), oracle.qlinear(np.abs(X), np.abs(W))
        err = np.abs(host16(out.half(M, N)).astype(np.float64) - r)
        assert np.all(err <= 2.0 ** -11 * (np.abs(r) + size) + 1e-6 * size)
        assert np.sqrt(np.mean(err ** 2)) <= 4e-4 * np.sqrt(np.mean(r ** 2))


# Tiles of 64 columns that take two to eight row blocks at once: (M, N, K) and the blocks; the last row block full, with one row,
# and with most; columns at and beside a multiple of 64; fewer groups than wavefronts, one turn, a second one for
# some, several.
WIDE_CASES = [((30, 11000, 1152), 2), ((48, 11008, 384), 3), ((200, 4096, 1152), 4), ((65, 8200, 1152), 5), ((80, 8250, 1152), 5),
              ((81, 10001, 1152), 6), ((96, 11008, 1152), 6), ((110, 9100, 1152), 7), ((112, 8300, 2176), 7), ((128, 11008, 1152), 8),
              ((113, 8200, 3200), 8)]


# 8-bit matrices take at most five row blocks
@pytest.mark.parametrize("bits, case, blocks", [(b, c, n) for c, n in WIDE_CASES for b in BITS if b < 8 or n <= 5],
                         ids=lambda c: "M%d_N%d_K%d" % c if isinstance(c, tuple) else str(c))
def test_qlinear_wide_few_row_tiles_against_oracle(fq, torch, bits, case, blocks):
    """Integer zeros, then fractions in some groups.  Bound: one rounding of the output (2^-11 |r|) and fp32 sums, 1e-6 sum
    |x||w|; code - zero is exact here and the scale is applied in fp32.  2^-24: subnormal results."""
    M, N, K = case
    codes = fq_synth.codes(70, N, K, bits)
    s = (np.abs(fq_synth.activations(71, N, K // 128).astype(np.float32)) * 0.01 + 1e-3).astype(np.float16)
    X = fq_synth.activations(72, M, K)
    assert fq.fq_qlinear_route(M, N, bits, K) == ("few_rows", 16 * blocks, 64)
    for frac in (0, 1):
        z = fq_synth.codes(73, N, K // 128, bits).astype(np.float32)
        if frac:
            z[::3, ::2] += 0.25
        z = z.astype(np.float16)
        out = Guarded(torch, M * N * 2)
        fq.fq_qlinear(dev(torch, X), fq.PackedMatrix.from_host(codes, s, z, bits), out=out.half(M, N))
        assert out.intact()
        W = oracle.dequant(codes, s, z)
        r, size = oracle.qlinear(X, W), oracle.qlinear(np.abs(X), np.abs(W))
        err = np.abs(host16(out.half(M, N)).astype(np.float64) - r)
        assert np.all(err <= 2.0 ** -11 * np.abs(r) + 1e-6 * size + 2.0 ** -24)


def sampled_columns(rng, N, count):
    """Columns of a matrix of N rows: some at random, and those on either side of the blocks of 16 and 64 at its ends."""
    edges = [n for n in (0, 15, 16, 63, 64, (N - 1) // 64 * 64 - 1, (N - 1) // 64 * 64, (N - 1) // 16 * 16, N - 1) if 0 <= n < N]
    return np.unique(np.concatenate([rng.integers(0, N, size=count), edges]))


# The same tiles over rows of more than 32 groups, where a wavefront's slots for scales and zeros are filled again: (M, N, K) and the
# blocks, on both sides of every difference between the bodies.
LONG_WIDE_CASES = [((600, 830, 5248), 2), ((620, 830, 5248), 3), ((640, 1180, 5248), 4), ((600, 1635, 5248), 5), ((600, 2055, 5248), 6),
                   ((600, 2335, 4224), 7), ((600, 2720, 5248), 8), ((600, 620, 11008), 2), ((600, 1635, 11008), 5)]


@pytest.mark.parametrize("bits, case, blocks", [(b, c, n) for c, n in LONG_WIDE_CASES for b in BITS if b < 8 or n <= 5],
                         ids=lambda c: "M%d_N%d_K%d" % c if isinstance(c, tuple) else str(c))
def test_qlinear_wide_few_row_tiles_over_long_rows(fq, torch, bits, case, blocks):
    """Scales and zeros differ from group to group; sampled columns, and the bound of the test above."""
    M, N, K = case
    assert fq.fq_qlinear_route(M, N, bits, K) == ("few_rows", 16 * blocks, 64)
    codes = fq_synth.codes(74, N, K, bits)
    s = (np.abs(fq_synth.activations(75, N, K // 128).astype(np.float32)) * 0.01 + 1e-3).astype(np.float16)
    X = fq_synth.activations(76, M, K)
    cols = sampled_columns(np.random.default_rng(3), N, 60)
    for frac in (0, 1):
        z = fq_synth.codes(77, N, K // 128, bits).astype(np.float32)
        if frac:
            z[::3, ::2] += 0.25
        z = z.astype(np.float16)
        out = Guarded(torch, M * N * 2)
        fq.fq_qlinear(dev(torch, X), fq.PackedMatrix.from_host(codes, s, z, bits), out=out.half(M, N))
        assert out.intact()
        W = oracle.dequant(codes[cols], s[cols], z[cols])
        r, size = oracle.qlinear(X, W), oracle.qlinear(np.abs(X), np.abs(W))
        err = np.abs(host16(out.half(M, N))[:, cols].astype(np.float64) - r)
        assert np.all(err <= 2.0 ** -11 * np.abs(r) + 1e-6 * size + 2.0 ** -24)


# Launches of several matrices: odd column offsets, a row pitch that is not a matrix's own N, matrices of few and many tiles in
# every place, and one of 8 bits, which keeps all of the launch to five blocks.
@pytest.mark.parametrize("M, rows, runs", [(77, 32, [(2433, 2), (1231, 3), (432, 4)]), (100, 48, [(2433, 2), (1231, 3), (432, 4)]),
                                           (200, 80, [(2433, 2), (1231, 3), (432, 4)]), (300, 112, [(2433, 2), (1231, 3), (432, 4)]),
                                           (300, 48, [(1231, 8), (2433, 2), (400, 4)]), (200, 80, [(2433, 2), (400, 4), (1231, 8)]),
                                           (512, 80, [(2433, 2), (1231, 8), (400, 3)]), (128, 128, [(5000, 2), (3001, 4), (2999, 3)]),
                                           (77, 80, [(5000, 3), (3001, 4), (2999, 2)]), (400, 64, [(2433, 4), (1663, 3)])])
def test_qlinear_wide_few_row_tiles_in_launches_of_several_matrices(fq, torch, M, rows, runs):
    """Sampled columns of every matrix against the oracle, with the bound of the test above; guard bytes, and no element left out."""
    K, total = 4224, sum(N for N, _ in runs)
    assert fq.fq_qlinear_route(M, [N for N, _ in runs], [b for _, b in runs], K) == ("few_rows", rows, 64)
    rng = np.random.default_rng(21)
    segs, sampled, cols_all, col0 = [], [], [], 0
    for i, (N, bits) in enumerate(runs):
        codes = fq_synth.codes(91 + i, N, K, bits)
        s = (np.abs(fq_synth.activations(94 + i, N, K // 128).astype(np.float32)) * 0.01 + 1e-3).astype(np.float16)
        z = (fq_synth.codes(97 + i, N, K // 128, bits).astype(np.float32) + 0.25 * (i == 1)).astype(np.float16)
        segs.append(fq.PackedMatrix.from_host(codes, s, z, bits))
        cols = sampled_columns(rng, N, 50)
        sampled.append(oracle.dequant(codes[cols], s[cols], z[cols]))
        cols_all.append(col0 + cols)
        col0 += N
    X = fq_synth.activations(90, M, K)
    out = Guarded(torch, M * total * 2)
    out.half(M, total).fill_(float("nan"))
    fq.fq_qlinear_mixed(dev(torch, X), segs, out=out.half(M, total))
    assert out.intact()
    y = host16(out.half(M, total)).astype(np.float64)
    assert np.all(np.isfinite(y))
    W = np.concatenate(sampled, axis=0)
    r, size = oracle.qlinear(X, W), oracle.qlinear(np.abs(X), np.abs(W))
    err = np.abs(y[:, np.concatenate(cols_all)] - r)
    assert np.all(err <= 2.0 ** -11 * np.abs(r) + 1e-6 * size + 2.0 ** -24)


@pytest.mark.parametrize("zeros", ["fractions", "odd_large", "largest", "negative"])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", [(1, 300, 1024), (2, 300, 1024), (3, 300, 8320), (4, 70, 128), (4, 300, 2048), (16, 5200, 1152),
                                  (16, 11008, 1280)], ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_of_a_few_rows_takes_any_zero_exactly(fq, torch, bits, case, zeros):
    """Up to sixteen rows no weight is rounded, whatever its zero: beside the output's rounding (2^-11 |r|) there are only
    those of fp32 sums, a few 2^-24 of sum |x| scale (code + |zero|), and up to three rows of the bias of 1024 that
    the streamed codes carry.  A code - zero rounded to fp16 would be 2^-12 of it off per weight.  Some of the groups
    keep integer zeros, and zeros in steps that are exact beside every code."""
    M, N, K = case
    G = K // 128
    rng = np.random.default_rng(1000 * bits + N + K)
    codes = fq_synth.codes(64, N, K, bits)
    s = (np.abs(fq_synth.activations(65, N, G).astype(np.float32)) * 1e-4 + 1e-4).astype(np.float16)
    X = fq_synth.activations(66, M, K)
    z = {"fractions": rng.uniform(0, 2 ** bits, (N, G)), "odd_large": 2 * rng.integers(512, 1024, (N, G)) + 1,
         "largest": rng.choice([65504.0, 64512.0, 40000.0, 2049.0, 1e-6], (N, G)),
         "negative": -rng.uniform(0, 300, (N, G))}[zeros].astype(np.float16)
    z[:, 1::3] = fq_synth.codes(67, N, G, bits)[:, 1::3]
    z[:, 2::6] += np.float16(2.0 ** (bits - 11)) * (np.abs(z[:, 2::6]) < 2 ** bits)
    w = fq.PackedMatrix.from_host(codes, s, z, bits)
    out = Guarded(torch, M * N * 2)
    fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N))
    assert out.intact()
    r = oracle.qlinear(X, oracle.dequant(codes, s, z))
    per_code = codes.astype(np.float32) + np.repeat(np.abs(z.astype(np.float32)), 128, axis=1) + (1024.0 if M <= 3 else 0.0)
    size = oracle.qlinear(np.abs(X), per_code * np.repeat(s.astype(np.float32), 128, axis=1))
    err = np.abs(host16(out.half(M, N)).astype(np.float64) - r)
    bound = 2.0 ** -11 * np.abs(r) + 1e-6 * size + 2.0 ** -25
    assert np.count_nonzero(err > bound) == 0


@pytest.mark.parametrize("zeros", ["fractions", "odd_large", "largest", "negative"])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", [(210, 290, 256), (433, 421, 256), (429, 196, 1024), (825, 135, 1536), (33, 4096, 1152), (60, 4096, 2176),
                                  (1036, 98, 128), (71, 8207, 640), (80, 8250, 1024)],
                         ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_few_row_tiles_take_any_zero_exactly(fq, torch, bits, case, zeros):
    """Nor do the taller tiles of sixteen columns and of 32 by 32 round any weight, which serve sizes that tiles of sixteen rows would
    serve otherwise: the bound of the test above, on sampled columns; and for sizes that tiles of 64 columns and 80 rows would
    serve faster.  A third of the groups keep integer zeros."""
    M, N, K = case
    G = K // 128
    rng = np.random.default_rng(1000 * bits + N + K)
    codes = fq_synth.codes(84, N, K, bits)
    s = (np.abs(fq_synth.activations(85, N, G).astype(np.float32)) * 1e-4 + 1e-4).astype(np.float16)
    X = fq_synth.activations(86, M, K)
    z = {"fractions": rng.uniform(0, 2 ** bits, (N, G)), "odd_large": 2 * rng.integers(512, 1024, (N, G)) + 1,
         "largest": rng.choice([65504.0, 64512.0, 40000.0, 2049.0, 1e-6], (N, G)),
         "negative": -rng.uniform(0, 300, (N, G))}[zeros].astype(np.float16)
    z[:, 1::3] = fq_synth.codes(87, N, G, bits)[:, 1::3]
    name, rows, columns = fq.fq_qlinear_route(M, N, bits, K)
    assert name == "few_rows" and (rows == 16 or columns == 16 or (rows, columns) == (32, 32))
    out = Guarded(torch, M * N * 2)
    fq.fq_qlinear(dev(torch, X), fq.PackedMatrix.from_host(codes, s, z, bits), out=out.half(M, N))
    assert out.intact()
    cols = sampled_columns(rng, N, 90)
    codes, s, z = codes[cols], s[cols], z[cols]
    r = oracle.qlinear(X, oracle.dequant(codes, s, z))
    per_code = codes.astype(np.float32) + np.repeat(np.abs(z.astype(np.float32)), 128, axis=1)
    size = oracle.qlinear(np.abs(X), per_code * np.repeat(s.astype(np.float32), 128, axis=1))
    err = np.abs(host16(out.half(M, N))[:, cols].astype(np.float64) - r)
    assert np.count_nonzero(err > 2.0 ** -11 * np.abs(r) + 1e-6 * size + 2.0 ** -25) == 0


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("M", [1, 5])
def test_qlinear_of_very_long_rows_against_oracle(fq, torch, bits, M):
    """Rows that neither the decode kernel's LDS nor the few-row kernel's offsets hold: the generic kernel.  Its wavefronts sum
    8200 groups each in fp32, roundings of 2^-24 of the sum so far that add up to less than 1e-4 of the row's rms."""
    N, K = 5, (1 << 22) + 128
    assert fq.fq_qlinear_route(M, N, bits, K)[0] == "generic"
    w, codes, s, z = make_matrix(fq, 90, N, K, bits)
    X = fq_synth.activations(91, M, K)
    out = Guarded(torch, M * N * 2)
    fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N))
    assert out.intact()
    assert qerr(host16(out.half(M, N)), oracle.qlinear(X, oracle.dequant(codes, s, z))) <= TOL


def test_qlinear_tile_rejects_other_tile_heights(fq, torch):
    w, *_ = make_matrix(fq, 1, 64, 128, 4)
    with pytest.raises(fq.FqError) as e:
        fq.fq_qlinear(dev(torch, fq_synth.activations(1, 32, 128)), w, tile_rows=64)
    assert e.value.code == -2


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("M", [1, 16, 48])
def test_qlinear_exact_on_integer_case(fq, torch, bits, M):
    """Power-of-two scales and small-integer activations: every partial sum is exact."""
    N, K = 96, 512
    codes = fq_synth.codes(1, N, K, bits)
    s = np.full((N, K // 128), 0.25, dtype=np.float16)
    z = np.full((N, K // 128), float(1 << (bits - 1)), dtype=np.float16)
    X = (fq_synth.codes(2, M, K, 3).astype(np.float32) - 4).astype(np.float16)
    w = fq.PackedMatrix.from_host(codes, s, z, bits)
    r = oracle.qlinear(X, oracle.dequant(codes, s, z))
    assert np.array_equal(r * 4, np.rint(r * 4)) and np.max(np.abs(r)) * 4 < 2 ** 22  # exact in fp32 partial sums
    y = host16(fq.fq_qlinear(dev(torch, X), w)).astype(np.float64)
    assert np.array_equal(y, oracle.round_f16(r).astype(np.float64))


@pytest.mark.parametrize("bits", (2, 3, 4))
@pytest.mark.parametrize("M", [1, 40])
@pytest.mark.parametrize("midpoint", [False, True])
def test_qlinear_on_truncated_codes(fq, torch, bits, M, midpoint):
    """Section "Elastic Serving": the b-bit layer obtained by dropping bits of the 8-bit one."""
    N, K = 256, 512
    W = fq_synth.weights(77, N, K)
    q8, s8, z8 = oracle.quantize_rtn(W, 8)
    q, s, z = oracle.truncate(q8, s8, z8, 8 - bits, midpoint=midpoint)
    w = fq.PackedMatrix.from_host(q, s, z, bits)
    W32 = oracle.dequant(q, s, z)
    assert np.array_equal(fq.fq_dequant(w).cpu().numpy().view(np.uint32), W32.view(np.uint32))
    X = fq_synth.activations(78, M, K)
    y = host16(fq.fq_qlinear(dev(torch, X), w))
    assert qerr(y, oracle.qlinear(X, W32)) <= TOL


@pytest.mark.parametrize("bits", BITS)
def test_qlinear_full_size_sampled(fq, torch, bits):
    """Llama-2-7B matrix shapes at M=1 and M=2048; the oracle computes sampled rows and columns."""
    rng = np.random.default_rng(bits)
    for (N, K) in [(4096, 4096), (11008, 4096), (4096, 11008)]:
        w, codes, s, z = make_matrix(fq, 200 + bits, N, K, bits)
        cols = np.unique(np.concatenate([rng.integers(0, N, size=192), [0, N - 1]]))
        W32 = oracle.dequant(codes[cols], s[cols], z[cols])
        for M in (1, 2048):
            X = fq_synth.activations(10, M, K)
            y = host16(fq.fq_qlinear(dev(torch, X), w))
            rows = np.arange(M) if M == 1 else np.unique(np.concatenate([rng.integers(0, M, size=48), [0, M - 1]]))
            r = oracle.qlinear(X[rows], W32)
            ysub = y[np.ix_(rows, cols)].astype(np.float64)
            # rms over the sampled columns stands in for the row rms
            assert qerr(ysub, r) <= TOL, (N, K, M)
            assert np.all(np.isfinite(y.astype(np.float32)))


def test_qlinear_is_deterministic(fq, torch):
    w, *_ = make_matrix(fq, 5, 4096, 4096, 3)
    for M in (1, 512):
        X = dev(torch, fq_synth.activations(6, M, 4096))
        a = fq.fq_qlinear(X, w)
        b = fq.fq_qlinear(X, w)
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_more_bits_track_the_unquantized_layer_better_on_gpu(fq, torch):
    N, K, M = 512, 1024, 64
    W = fq_synth.weights(31, N, K)
    X = fq_synth.activations(32, M, K)
    Y = oracle.qlinear(X, W)
    errs = []
    for bits in BITS:
        codes, s, z = oracle.quantize_rtn(W, bits)
        y = host16(fq.fq_qlinear(dev(torch, X), fq.PackedMatrix.from_host(codes, s, z, bits))).astype(np.float64)
        errs.append(np.sqrt(np.mean((y - Y) ** 2) / np.mean(Y ** 2)))
    assert errs[0] > errs[1] > errs[2] > errs[3] and errs[3] < 1e-2


# --------------------------------------------------------------- dense head
@pytest.mark.parametrize("tile", [0, 128, 256])
@pytest.mark.parametrize("case", [(40, 512, 256), (300, 1000, 384), (257, 1026, 128), (2048, 32000, 512)], ids=str)
def test_dense_head_against_oracle(fq, torch, case, tile):
    """Both kernels behind fq_dense_f16 (128- and 256-row tiles), pinned through fq_dense_f16_tile, and the
    library's own choice; ragged sizes cover rows and columns past the last full tile."""
    M, N, K = case
    X = fq_synth.activations(13, M, K)
    W = fq_synth.weights(14, N, K).astype(np.float16)
    y = host16(fq.fq_dense_f16(dev(torch, X), dev(torch, W), tile_rows=tile))
    if M * N > 1 << 20:
        rng = np.random.default_rng(0)
        rows = np.unique(np.concatenate([rng.integers(0, M, 40), [0, M - 1]]))
        cols = np.unique(np.concatenate([rng.integers(0, N, 300), [0, N - 1]]))
        r = oracle.dense_f16(X[rows], W[cols])
        assert qerr(y[np.ix_(rows, cols)], r) <= TOL
    else:
        assert qerr(y, oracle.dense_f16(X, W)) <= TOL


# Few rows: the tiles of 16, 32, 64 and 128 rows, rows that end inside a block and in a second row tile, columns that end
# inside a block, a wavefront's columns and a 64-column group, K of fewer stages than the ring holds and of more.
ROWS_CASES = [(1, 1000, 128), (16, 70, 384), (17, 1030, 1024), (32, 1, 256), (33, 257, 640), (64, 1001, 1024),
              (65, 130, 384), (128, 2000, 512), (129, 1003, 256), (300, 66, 1152)]


@pytest.mark.parametrize("case", ROWS_CASES, ids=str)
def test_head_few_rows_against_oracle(fq, torch, case):
    """Logits at the tolerance of the head, written nowhere else; and the loss of the same call chain, whose logits
    are the same sums, so that the two calls differ by the order of the fp32 merges only."""
    M, V, K = case
    X, W = fq_synth.activations(70, M, K), fq_synth.weights(71, V, K, 0.05).astype(np.float16)
    out = Guarded(torch, M * V * 2)
    fq.fq_dense_f16(dev(torch, X), dev(torch, W), out=out.half(M, V))
    assert out.intact()
    logits = oracle.dense_f16(X, W)
    err = np.abs(host16(out.half(M, V)).astype(np.float64) - logits)
    # one rounding to fp16, and fp32 sums of K products
    assert np.all(err <= 2.0 ** -11 * np.abs(logits) + 1e-6 * oracle.dense_f16(np.abs(X), np.abs(W)))
    lab = fq_synth.labels(72, M, V)
    lab[0] = V - 1
    lab[M // 2:M // 2 + 1] = -1
    ws, nll = Guarded(torch, fq.fq_head_nll_workspace_bytes(M, V)), Guarded(torch, M * 4)
    got = fq.fq_head_nll(dev(torch, X), dev(torch, W), dev(torch, lab), out=nll.f32(M), workspace=ws.bytes())
    assert ws.intact() and nll.intact()
    two = fq.fq_token_nll(out.half(M, V).clone(), dev(torch, lab))
    assert float((got - two).abs().max()) <= 2e-5
    assert np.max(np.abs(got.cpu().numpy().astype(np.float64) - oracle.token_nll(oracle.round_f16(logits), lab))) <= 2e-3


# (M, V, K), the kernel and tile of the logits, the rows of the loss's tile: every tile of the kernel whose wavefronts share K,
# with rows and columns that end inside a block or tile, one group, fewer groups than wavefronts, one turn and several; and the
# streaming one of 96 rows.
SHARED_K_CASES = [((1, 20, 640), ("shared_k", 16, 16), 16), ((33, 20, 256), ("shared_k", 16, 16), 16),
                  ((1, 4117, 1024), ("shared_k", 16, 32), 16), ((16, 6272, 4096), ("shared_k", 16, 64), 16),
                  ((17, 2093, 1024), ("shared_k", 32, 16), 16), ((101, 1377, 384), ("shared_k", 32, 32), 16),
                  ((819, 259, 1024), ("shared_k", 32, 32), 32), ((72, 4129, 640), ("shared_k", 32, 64), 32),
                  ((33, 2874, 1152), ("shared_k", 48, 16), 16), ((104, 2308, 384), ("shared_k", 48, 32), 32),
                  ((102, 4104, 640), ("shared_k", 48, 64), 48), ((101, 2727, 512), ("shared_k", 64, 32), 32),
                  ((100, 6249, 768), ("shared_k", 64, 64), 64), ((67, 5559, 640), ("shared_k", 80, 32), 48),
                  ((67, 8403, 1024), ("shared_k", 80, 64), 80), ((82, 8409, 1792), ("shared_k", 96, 64), 96),
                  ((105, 8227, 1664), ("shared_k", 112, 64), 112), ((116, 8725, 1792), ("shared_k", 128, 64), 128),
                  ((82, 8264, 1152), ("stream", 96, 128), 96), ((180, 1300, 128), ("stream", 96, 128), 96)]


@pytest.mark.parametrize("case, route, loss_rows", SHARED_K_CASES, ids=lambda c: "-".join(map(str, c)) if isinstance(c, tuple) else "")
def test_head_of_few_rows_and_columns_against_oracle(fq, torch, case, route, loss_rows):
    """Logits to one rounding and fp32 sums, written nowhere else; the loss of the same sums, to the order of its merges."""
    M, V, K = case
    assert fq.fq_dense_route(M, V, K) == route
    assert fq.fq_dense_route(M, V, K, loss=True)[:2] == (route[0], loss_rows)
    X, W = fq_synth.activations(80, M, K), fq_synth.weights(81, V, K, 0.05).astype(np.float16)
    lab = fq_synth.labels(82, M, V)
    lab[0] = V - 1
    lab[M // 2:M // 2 + 1] = -1
    out = Guarded(torch, M * V * 2)
    ws, nll = Guarded(torch, fq.fq_head_nll_workspace_bytes(M, V)), Guarded(torch, M * 4)
    fq.fq_dense_f16(dev(torch, X), dev(torch, W), out=out.half(M, V))
    got = fq.fq_head_nll(dev(torch, X), dev(torch, W), dev(torch, lab), out=nll.f32(M), workspace=ws.bytes())
    assert out.intact() and ws.intact() and nll.intact()
    assert float((got - fq.fq_token_nll(out.half(M, V).clone(), dev(torch, lab))).abs().max()) <= 2e-5
    rows = np.unique(np.concatenate([np.arange(min(M, 6)), np.arange(max(0, M - 20), M)]))
    logits = oracle.dense_f16(X[rows], W)
    err = np.abs(host16(out.half(M, V))[rows].astype(np.float64) - logits)
    assert np.all(err <= 2.0 ** -11 * np.abs(logits) + 1e-6 * oracle.dense_f16(np.abs(X[rows]), np.abs(W)))


def test_head_nll_of_shared_k_carries_nan_and_infinity(fq, torch):
    """As below, in the kernel whose wavefronts share K: a NaN in four columns reaches the loss, 64 columns of -inf add nothing."""
    M, V, K = 20, 200, 1024
    assert fq.fq_dense_route(M, V, K, loss=True)[0] == "shared_k"
    X, W = np.zeros((M, K), dtype=np.float16), np.zeros((V, K), dtype=np.float16)
    X[:, 0] = 1.0
    lab = dev(torch, np.full(M, 150, dtype=np.int32))
    W[100:104, 0] = np.nan
    assert np.isnan(fq.fq_head_nll(dev(torch, X), dev(torch, W), lab).cpu().numpy()).all()
    W[100:104, 0], W[0:64, 0] = 0.0, -np.inf
    assert np.allclose(fq.fq_head_nll(dev(torch, X), dev(torch, W), lab).cpu().numpy(), math.log(V - 64), atol=1e-4)


def test_head_nll_few_rows_carries_nan_and_infinity(fq, torch):
    """A NaN in four columns only (one lane's share) reaches the loss; a 64-column group of -inf adds nothing to it."""
    M, V, K = 20, 200, 128
    X, W = np.zeros((M, K), dtype=np.float16), np.zeros((V, K), dtype=np.float16)
    X[:, 0] = 1.0
    lab = dev(torch, np.full(M, 150, dtype=np.int32))
    W[100:104, 0] = np.nan
    assert np.isnan(fq.fq_head_nll(dev(torch, X), dev(torch, W), lab).cpu().numpy()).all()
    W[100:104, 0], W[0:64, 0] = 0.0, -np.inf
    assert np.allclose(fq.fq_head_nll(dev(torch, X), dev(torch, W), lab).cpu().numpy(), math.log(V - 64), atol=1e-4)


# ----------------------------------------------------------------------- NLL
def test_token_nll_closed_forms(fq, torch):
    V = 32000
    x = np.zeros((6, V), dtype=np.float16)
    x[1] += np.float16(65504.0)
    x[2] -= np.float16(65504.0)
    x[3, 17] = 60.0
    x[4, 17] = 60.0
    lab = np.array([0, 31999, 5, 17, 18, -1], dtype=np.int32)
    got = fq.fq_token_nll(dev(torch, x), dev(torch, lab)).cpu().numpy().astype(np.float64)
    want = [math.log(V)] * 3 + [0.0, 60.0, 0.0]
    assert np.allclose(got, want, rtol=0, atol=1e-4)
    assert np.allclose(got, oracle.token_nll(x, lab), rtol=0, atol=1e-4)


@pytest.mark.parametrize("shape", [(2048, 32000), (130, 1001), (7, 8)])
def test_token_nll_against_oracle(fq, torch, shape):
    M, V = shape
    L = fq_synth.logits(21, M, V)
    lab = fq_synth.labels(22, M, V)
    lab[0], lab[-1] = 0, V - 1
    got = fq.fq_token_nll(dev(torch, L), dev(torch, lab)).cpu().numpy().astype(np.float64)
    want = oracle.token_nll(L, lab)
    assert np.max(np.abs(got - want)) <= 2e-3
    assert abs(got.mean() - want.mean()) <= 1e-3  # per-sequence mean NLL
    assert abs(math.exp(got.mean()) / oracle.perplexity(want) - 1) <= 1e-3


@pytest.mark.parametrize("case", [(2048, 32000, 512), (2048, 32000, 4096), (300, 1001, 256), (5, 70, 128)], ids=str)
def test_head_nll_fused_against_oracle(fq, torch, case):
    """Head GEMM with the loss in its epilogue against the oracle's chain dense -> fp16 logits -> NLL (on a
    sample of rows where the full product is too slow for the oracle), and against the library's own two
    calls, which it must reproduce up to the order of the fp32 merges."""
    M, V, K = case
    X = fq_synth.activations(51, M, K)
    W = fq_synth.weights(52, V, K, 0.02 if K > 1024 else 0.05, 99).astype(np.float16)
    lab = fq_synth.labels(53, M, V)
    lab[0], lab[-1] = 0, V - 1
    if M > 4:
        lab[2] = -1          # ignored position
        lab[3] = V           # out of range counts as ignored too
    dX, dW, dl = dev(torch, X), dev(torch, W), dev(torch, lab)
    got = fq.fq_head_nll(dX, dW, dl).cpu().numpy().astype(np.float64)
    two = fq.fq_token_nll(fq.fq_dense_f16(dX, dW), dl).cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - two)) <= 2e-5
    rows = np.arange(M)
    if M * V * K > 1 << 30:
        rng = np.random.default_rng(1)
        rows = np.unique(np.concatenate([rng.integers(0, M, 24 if K <= 512 else 6), [0, 2, 3, 255, 256, M - 1]]))
    want = oracle.token_nll(oracle.round_f16(oracle.dense_f16(X[rows], W)), lab[rows])
    assert np.max(np.abs(got[rows] - want)) <= 2e-3
    assert abs(got[rows].mean() - want.mean()) <= 1e-3
    if M > 4:
        assert got[2] == 0.0 and got[3] == 0.0


# ---------------------------------------------------------------------- glue
@pytest.mark.parametrize("shape", [(2048, 32000), (130, 1001), (7, 8), (3, 32768)])
def test_logit_l2_against_oracle(fq, torch, shape):
    """fp32 accumulation of up to 32768 squares in four partial sums per thread: relative error of the
    sum below 2e-6, of its root below 1e-6; the bound asked is 1e-5 (plus exact zero for equal rows)."""
    M, V = shape
    a = fq_synth.logits(400, M, V)
    b = fq_synth.logits(401, M, V)
    b[0] = a[0]                      # distance exactly 0
    b[M - 1] = a[M - 1]
    b[M - 1, V - 1] = np.float16(float(a[M - 1, V - 1]) + 2.0)  # a single differing entry, in the ragged tail
    got = fq.fq_logit_l2(dev(torch, a), dev(torch, b)).cpu().numpy().astype(np.float64)
    want = oracle.logit_l2(a, b)
    assert got[0] == 0.0
    assert got[M - 1] == want[M - 1]
    assert np.max(np.abs(got - want) / np.maximum(want, 1e-30)) <= 1e-5 or np.allclose(got, want, rtol=1e-5, atol=0)
    # large magnitudes: differences up to 2 * 65504 still square and sum in range of fp32
    big = np.full((2, V), 65504.0, dtype=np.float16)
    neg = -big
    got = fq.fq_logit_l2(dev(torch, big), dev(torch, neg)).cpu().numpy().astype(np.float64)
    assert np.allclose(got, oracle.logit_l2(big, neg), rtol=1e-5)


@pytest.mark.parametrize("V", [1, 7, 9, 15, 17, 255, 257, 511, 513, 1003, 8191, 8197, 16387, 31001])
@pytest.mark.parametrize("M", [5, 260])
def test_row_kernels_on_unaligned_rows(fq, torch, M, V):
    """Rows that start anywhere between 16-byte boundaries: elements before the first whole chunk, behind the last, and
    rows without any; both workgroup sizes.  A logit of its own size in every position of the ends makes a missed
    or doubled one show.  Bounds: those of the aligned rows."""
    a, b = fq_synth.logits(410, M, V), fq_synth.logits(411, M, V)
    a[:, :8] += np.arange(1, 1 + min(8, V), dtype=np.float16)[None, :]
    a[:, -8:] -= np.arange(1, 1 + min(8, V), dtype=np.float16)[None, :]
    lab = fq_synth.labels(412, M, V)
    lab[0], lab[-1] = V - 1, 0
    got = fq.fq_token_nll(dev(torch, a), dev(torch, lab)).cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - oracle.token_nll(a, lab))) <= 2e-3
    got = fq.fq_logit_l2(dev(torch, a), dev(torch, b)).cpu().numpy().astype(np.float64)
    assert np.allclose(got, oracle.logit_l2(a, b), rtol=1e-5, atol=0)


@pytest.mark.parametrize("V", [31, 100, 2040, 8000, 8001, 32000, 32001])
@pytest.mark.parametrize("M", [5, 260])
def test_token_nll_of_masked_rows(fq, torch, M, V):
    """Logits of -inf add nothing wherever they stand: whole chunks of them behind, before and between a thread's other
    ones, all but the label, and next to one NaN, which reaches the loss; both workgroup sizes, rows aligned and not.
    Bounds: those of finite rows."""
    x = fq_synth.logits(416, M, V)
    lab = (fq_synth.labels(417, M, V) % (V // 4) + V // 2).astype(np.int32)
    x[0, V - V // 4:] = -np.inf
    x[1, :V // 2] = -np.inf
    x[2, np.arange(V) // 16 % 2 == 1] = -np.inf
    x[3] = -np.inf
    x[np.arange(M), lab] = np.float16(1.5)
    got = fq.fq_token_nll(dev(torch, x), dev(torch, lab)).cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - oracle.token_nll(x, lab))) <= 2e-3
    assert got[3] == 0.0
    for at, width in ((0, 1), (V // 2 - 1, 1), (V // 2 - 1, 15), (V - 1, 1), (V - 1, 9)):  # labels lie between V / 2 and 3 V / 4
        y = x.copy()
        y[:, max(0, at - 24):at + 24] = -np.inf
        y[:, max(0, at - width + 1):at + 1] = np.nan
        y[np.arange(M), lab] = np.float16(1.5)
        assert np.isnan(fq.fq_token_nll(dev(torch, y), dev(torch, lab)).cpu().numpy()).all(), (at, width)


@pytest.mark.parametrize("V", [2040, 2048, 2056, 4096, 4104, 8184, 8192, 8200, 16384, 16392, 32768, 32776])
@pytest.mark.parametrize("M", [5, 260])
def test_row_kernels_around_whole_trips(fq, torch, M, V):
    """Rows of one chunk a thread, one more, and around whole trips of four chunks a thread, for both workgroup sizes.
    The last chunk stands out, so that one dropped, or added again by a thread past the row's end, shows.  Bounds:
    those of the other sizes."""
    a, b = fq_synth.logits(413, M, V), fq_synth.logits(414, M, V)
    a[:, -8:] += np.float16(6)
    lab = fq_synth.labels(415, M, V)
    got = fq.fq_token_nll(dev(torch, a), dev(torch, lab)).cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - oracle.token_nll(a, lab))) <= 2e-3
    got = fq.fq_logit_l2(dev(torch, a), dev(torch, b)).cpu().numpy().astype(np.float64)
    assert np.allclose(got, oracle.logit_l2(a, b), rtol=1e-5, atol=0)


@pytest.mark.parametrize("H", [256, 4096, 11008, 13824])
def test_glue_steps_against_oracle(fq, torch, H):
    M = 9
    a, b, c = (fq_synth.activations(40 + i, M, H) for i in range(3))
    f = lambda t: t.astype(np.float64)
    want = {
        0: oracle.rms_rows(f(a)),
        1: oracle.rms_rows(f(a) + f(b) + f(c)),
        2: oracle.round_f16(f(a) + f(b)),
        3: oracle.rms_rows(oracle.silu_mul(a, b)),
        4: oracle.rms_rows(f(a) + f(b)),
    }
    da, db, dc = dev(torch, a), dev(torch, b), dev(torch, c)
    for op, w in want.items():
        got = host16(fq.fq_glue(op, da, db if op else None, dc if op == 1 else None))
        # fp32 on the GPU against fp64 in the oracle: agree to one fp16 ulp, and almost always exactly
        diff = np.abs(got.astype(np.float64) - w.astype(np.float64))
        ulp = np.maximum(np.abs(w.astype(np.float64)), 2.0 ** -14) * 2.0 ** -10
        assert np.all(diff <= ulp), op
        assert np.mean(diff > 0) < 2e-3, op


# --------------------------------------------------------------------- stack
def build_stack(fq, shapes_key, seed, bit_choices=BITS):
    sh = fq_synth.MODEL_SHAPES[shapes_key]
    layers, host = [], []
    for l in range(sh["layers"]):
        mats, hmats = [], []
        for j, (N, K) in enumerate(fq_synth.block_matrix_shapes(sh["hidden"], sh["ffn"])):
            W = fq_synth.weights(seed, N, K, 0.02, l, j)
            by_bits, hby = {}, {}
            for b in bit_choices:
                codes, s, z = oracle.quantize_rtn(W, b)
                by_bits[b] = fq.PackedMatrix.from_host(codes, s, z, b)
                hby[b] = (codes, s, z)
            mats.append(by_bits)
            hmats.append(hby)
        layers.append(mats)
        host.append(hmats)
    return fq.Stack(layers), host, sh


@pytest.mark.parametrize("M", [1, 4, 40])
def test_stack_forward_against_oracle(fq, torch, M):
    stack, host, sh = build_stack(fq, "tiny", 300)
    bitvec = fq_synth.bit_vector(M, 7 * sh["layers"], probs=(0.25, 0.25, 0.25, 0.25))
    x = fq_synth.activations(301, M, sh["hidden"])
    got = host16(fq.fq_stack_forward(stack, bitvec, dev(torch, x)))
    # end to end: fp16 re-rounding between steps lets single ulps flip, so the bound is looser
    mats = [[oracle.dequant(*host[l][j][int(bitvec[7 * l + j])]) for j in range(7)] for l in range(sh["layers"])]
    want = oracle.stack_forward(x, mats)
    assert np.max(np.abs(got.astype(np.float64) - want.astype(np.float64))) <= 2e-2
    assert np.mean(np.abs(got.astype(np.float64) - want.astype(np.float64))) <= 2e-3
    # teacher-forced: one block at a time from the GPU's own layer input
    xin = x
    for l in range(sh["layers"]):
        sub = fq.Stack([stack.layers[l]])
        gout = host16(fq.fq_stack_forward(sub, bitvec[7 * l:7 * l + 7], dev(torch, xin)))
        t = oracle.block_forward(xin, mats[l])
        assert np.max(np.abs(gout.astype(np.float64) - t["x_next"].astype(np.float64))) <= 1e-2, l
        xin = gout
    assert np.array_equal(xin.view(np.uint16), got.view(np.uint16))


@pytest.mark.parametrize("M", [1, 40])
def test_stack_forward_replays_from_a_captured_graph(fq, torch, M):
    """The launches of a stack forward can be captured once and replayed: every replay, with eager work
    and synchronisations in between, gives the eager result bit for bit."""
    stack, host, sh = build_stack(fq, "tiny", 320)
    bitvec = fq_synth.bit_vector(7, 7 * sh["layers"], probs=(0.25, 0.25, 0.25, 0.25))
    x = dev(torch, fq_synth.activations(321, M, sh["hidden"]))
    ws = torch.empty(fq.fq_stack_workspace_bytes(M, sh["hidden"], sh["ffn"]), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(x)
    fq.fq_stack_forward(stack, bitvec, x, out=out, workspace=ws)  # eager; also the warm-up before capture
    torch.cuda.synchronize()
    want = out.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fq.fq_stack_forward(stack, bitvec, x, out=out, workspace=ws)
    for r in range(4):
        out.fill_(float("nan"))
        ws.random_(0, 255)  # eager work between the replays; the workspace holds no state
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), r


def test_block_steps_teacher_forced(fq, torch):
    """Each of the seven linears and five glue steps of a block, fed the oracle's inputs."""
    stack, host, sh = build_stack(fq, "tiny", 310)
    bitvec = np.array([2, 3, 4, 8, 3, 2, 4], dtype=np.uint8)
    M = 24
    x = fq_synth.activations(311, M, sh["hidden"])
    mats = [oracle.dequant(*host[0][j][int(bitvec[j])]) for j in range(7)]
    t = oracle.block_forward(x, mats)
    inputs = ["u", "u", "u", "a", "u2", "u2", "m"]
    outputs = ["q", "k", "v", "o", "g", "p", "d"]
    for j in range(7):
        w = stack.layers[0][j][int(bitvec[j])]
        y = host16(fq.fq_qlinear(dev(torch, t[inputs[j]]), w))
        assert qerr(y, oracle.qlinear(t[inputs[j]], mats[j])) <= TOL, outputs[j]


# ------------------------------------------------- full-size stacks (sampled)
def build_selected_stack(fq, hidden, ffn, layers, bitvec, seed):
    """Only the packing the bit vector selects is built for each matrix."""
    dev_layers, host = [], []
    for l in range(layers):
        mats, hmats = [], []
        for j, (N, K) in enumerate(fq_synth.block_matrix_shapes(hidden, ffn)):
            b = int(bitvec[7 * l + j])
            W = fq_synth.weights(seed, N, K, 0.02, l, j)
            codes, s, z = oracle.quantize_rtn(W, b)
            mats.append({b: fq.PackedMatrix.from_host(codes, s, z, b)})
            hmats.append((codes, s, z))
        dev_layers.append(mats)
        host.append(hmats)
    return fq.Stack(dev_layers), host


@pytest.mark.parametrize("model,M,probs", [("7b", 2048, (0.3, 0.3, 0.3, 0.1)), ("13b", 4096, (0.6, 0.3, 0.1, 0.0)),
                                           ("7b", 1, (0.3, 0.3, 0.3, 0.1)), ("13b", 1, (0.6, 0.3, 0.1, 0.0)),
                                           ("7b", 16, (0.3, 0.3, 0.3, 0.1))],
                         ids=["7b_M2048", "13b_M4096", "7b_M1", "13b_M1", "7b_M16"])
def test_llama_shaped_stack_sampled_rows(fq, torch, model, M, probs):
    """Two blocks at Llama-2 7B / 13B shapes in the launch configuration the benchmark times; rows of the
    stack are independent, so the oracle runs a sample of them through both blocks.  Sixteen rows take the
    row-wise steps as launches of their own and all linears through the few-row kernel."""
    sh = fq_synth.MODEL_SHAPES[model]
    L = 2
    bitvec = fq_synth.bit_vector(11, 7 * L, probs=probs)
    stack, host = build_selected_stack(fq, sh["hidden"], sh["ffn"], L, bitvec, 500)
    x = fq_synth.activations(501, M, sh["hidden"])
    got = host16(fq.fq_stack_forward(stack, bitvec, dev(torch, x)))
    assert np.all(np.isfinite(got.astype(np.float32)))
    rows = np.arange(M) if M <= 16 else np.array([0, 1, M // 2 - 1, M // 2, M - 129, M - 1])
    mats = [[oracle.dequant(*host[l][j]) for j in range(7)] for l in range(L)]
    want = oracle.stack_forward(x[rows], mats)
    diff = np.abs(got[rows].astype(np.float64) - want.astype(np.float64))
    assert diff.max() <= 2e-2 and diff.mean() <= 2e-3
    # first block teacher-forced at the qlinear tolerance: the GPU's own u against the oracle's linear
    u = oracle.rms_rows(x[rows].astype(np.float64))
    w0 = stack.layers[0][0][int(bitvec[0])]
    y = host16(fq.fq_qlinear(dev(torch, np.ascontiguousarray(u)), w0))
    assert qerr(y, oracle.qlinear(u, mats[0][0])) <= TOL


def test_ensemble_sweep_scores_candidates_like_the_oracle(fq, torch):
    """Several configuration vectors over one stack, each scored by per-sequence mean NLL through the
    fp16 head (the candidate loop of Algorithm 1 on a small stand-in model)."""
    stack, host, sh = build_stack(fq, "tiny", 700)
    V, T = 1000, 96
    head = fq_synth.weights(701, V, sh["hidden"], 0.3).astype(np.float16)
    x = fq_synth.activations(702, T, sh["hidden"])
    labels = fq_synth.labels(703, T, V)
    dhead, dx, dl = dev(torch, head), dev(torch, x), dev(torch, labels)
    scores = []
    for cand in range(4):
        bitvec = fq_synth.bit_vector(cand, 7 * sh["layers"], probs=(0.25, 0.25, 0.25, 0.25))
        h = fq.fq_stack_forward(stack, bitvec, dx)
        logits = fq.fq_dense_f16(h, dhead)
        nll = fq.fq_token_nll(logits, dl).cpu().numpy().astype(np.float64)
        # the loss kernel against the oracle on the very logits it read: the 1e-3 per-sequence bar
        ref_same_logits = oracle.token_nll(host16(logits), labels)
        assert abs(nll.mean() - ref_same_logits.mean()) <= 1e-3
        # whole chain against the oracle's own forward: fp16 re-rounding lets it drift a little
        mats = [[oracle.dequant(*host[l][j][int(bitvec[7 * l + j])]) for j in range(7)] for l in range(sh["layers"])]
        hx = oracle.stack_forward(x, mats)
        ref = oracle.token_nll(oracle.round_f16(oracle.dense_f16(hx, head)), labels)
        assert abs(nll.mean() - ref.mean()) <= 2e-2
        scores.append((nll.mean(), ref.mean()))
    # the ranking the search would use is the oracle's
    assert np.array_equal(np.argsort([s[0] for s in scores]), np.argsort([s[1] for s in scores]))


def test_sensitivity_table_ranks_like_the_oracle(fq, torch):
    """Sensitivity analysis: QM(n_up) = all 8-bit, one matrix lowered at a time.  The distance is a norm of
    differences of fp16 logits, so its own rounding floor is about ulp(logit)/sqrt(6) per entry; values are
    compared with 3 % + that floor, and the filter's pick must agree wherever the oracle's values are apart
    by more than that."""
    from paper_2501_07139_amd import sweep

    stack, host, sh = build_stack(fq, "tiny", 500)
    L, M, V = sh["layers"], 32, 1000
    up = np.full(7 * L, 8, dtype=np.uint8)
    x = fq_synth.activations(501, M, sh["hidden"])
    head = fq_synth.weights(502, V, sh["hidden"], 0.05).astype(np.float16)
    entries = [0, 3, 6, 7 + 4, 7 * (L - 1) + 1, 7 * L - 1]
    got = sweep.sensitivity_table(stack, dev(torch, head), up, dev(torch, x), entries=entries)
    assert sorted(got) == sorted((e, b) for e in entries for b in (2, 3, 4))

    def logits_for(bitvec):
        mats = [[oracle.dequant(*host[l][j][int(bitvec[7 * l + j])]) for j in range(7)] for l in range(L)]
        return oracle.round_f16(oracle.dense_f16(oracle.stack_forward(x, mats), head))  # the stored fp16 logits

    ref = logits_for(up)
    floor = float(np.sqrt(M * V / 6.0) * 2.0 ** -11 * np.sqrt(np.mean(ref.astype(np.float64) ** 2)))
    want = {}
    for (e, b) in got:
        cand = up.copy()
        cand[e] = b
        want[(e, b)] = float(np.sqrt(np.sum(oracle.logit_l2(logits_for(cand), ref) ** 2)))
        assert abs(got[(e, b)] - want[(e, b)]) <= 0.03 * want[(e, b)] + 2 * floor, (e, b, got[(e, b)], want[(e, b)])
    # lowering to fewer bits moves the logits further
    for e in entries:
        assert got[(e, 2)] > got[(e, 3)] > got[(e, 4)]
    # the filter keeps the same candidates as the oracle's table where those are clearly apart
    keys = sorted(got)
    pick_gpu = sweep.analysis_filter(got, keys, 6)
    pick_cpu = sweep.analysis_filter(want, keys, 6)
    cut = sorted(want.values())[5]
    clear = [k for k in keys if abs(want[k] - cut) > 0.03 * cut + 2 * floor]
    assert {k for k in pick_gpu if k in clear} == {k for k in pick_cpu if k in clear}


def test_tree_search_on_the_gpu_makes_choices_the_oracle_agrees_with(fq, torch):
    """Algorithm 1 driven by the GPU evaluator on a small stack.  Every scored candidate's perplexity must
    match the oracle's within 2e-3 relative (per-sequence NLL bound 1e-3, a little slack for exp), and every
    iteration must keep a set of models that is a correct top-#stem under the oracle's values up to such
    near-ties; the path itself must obey the one-way, one-matrix-per-step rule and end at QM(n_low)."""
    from paper_2501_07139_amd import search, sweep

    levels = (2, 4, 8)
    stack, host, sh = build_stack(fq, "tiny", 600, bit_choices=levels)
    L, M, V = sh["layers"], 64, 1000
    shapes = fq_synth.block_matrix_shapes(sh["hidden"], sh["ffn"]) * L
    x = fq_synth.activations(601, M, sh["hidden"])
    head = fq_synth.weights(602, V, sh["hidden"], 0.05).astype(np.float16)
    labels = fq_synth.labels(603, M, V)
    up = np.full(7 * L, 8, dtype=np.uint8)
    xd, hd, ld = dev(torch, x), dev(torch, head), torch.from_numpy(labels).cuda()
    table = sweep.sensitivity_table(stack, hd, up, xd)
    assert len(table) == 7 * L * 2
    ev = search.CalibrationEval(stack, hd, xd, ld)
    trace = []
    stems, branches = 2, 3
    paths = search.tree_search(up, levels, table, ev, shapes, stems, branches, trace=trace)
    assert 7 * L <= len(trace) <= 7 * L * 2             # every matrix goes down in one or two steps
    assert ev.blocks_run < ev.evaluations * L           # successors restart at the block they change
    for path in paths:
        assert path[-1].bitvec == (2,) * (7 * L)
        for a, b in zip(path, path[1:]):
            assert sum(p != q for p, q in zip(a.bitvec, b.bitvec)) == 1 and all(q <= p for p, q in zip(a.bitvec, b.bitvec))

    deq = {}

    def oracle_ppl(bits):
        mats = []
        for l in range(L):
            row = []
            for j in range(7):
                key = (l, j, bits[7 * l + j])
                if key not in deq:
                    deq[key] = oracle.dequant(*host[l][j][bits[7 * l + j]])
                row.append(deq[key])
            mats.append(row)
        logits = oracle.round_f16(oracle.dense_f16(oracle.stack_forward(x, mats), head))
        return oracle.perplexity(oracle.token_nll(logits, labels))

    for it in trace[::6] + trace[-2:]:                  # a sample of the iterations, incl. the last ones
        want = {b: oracle_ppl(b) for b, _ in it}
        for b, p in it:
            assert abs(p - want[b]) <= 2e-3 * want[b], (b, p, want[b])
        kept = [b for b, _ in it[:stems]]
        cut = sorted(want.values())[min(stems, len(it)) - 1]
        for b in kept:                                  # nothing kept is clearly worse than the oracle's cut
            assert want[b] <= cut * (1 + 4e-3)



# ------------------------------------- the hot path's own unpack, bit for bit
def _random_packing(fq, seed, N, K, bits, fractional):
    """Random codes, positive fp16 scales, and zeros that are integers (what the quantizer stores) or
    integers over a power of two (what truncating code bits leaves: Section "Elastic Serving")."""
    codes = fq_synth.codes(seed, N, K, bits)
    G = K // 128
    s = (np.abs(fq_synth.activations(seed + 1, N, G).astype(np.float32)) * 0.01 + 2e-3).astype(np.float16)
    zi = fq_synth.codes(seed + 2, N, G, bits).astype(np.float32)
    z = (zi / (1 << (8 - bits)) if fractional and bits < 8 else (zi / 4 if fractional else zi)).astype(np.float16)
    return fq.PackedMatrix.from_host(codes, s, z, bits), oracle.dequant(codes, s, z)


@pytest.mark.parametrize("fractional", [False, True], ids=["int_zero", "frac_zero"])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("shape", [(4096, 512), (11008, 1536), (200, 640)], ids=lambda s: "N%d_K%d" % s)
def test_gemm_unpack_is_bit_exact_through_an_identity(fq, torch, bits, shape, fractional):
    """X = I_K, M = K: the matrix-core kernel must return its own dequantized weights, rounded once to
    fp16, transposed: out[m, n] = fp16(scale * (code - zero))[n, m], every other term being an exact zero.
    N = 4096 runs the 128-wide tiles, N = 11008 with M = 1536 the 256-wide ones (2 and 4 bits); N = 200 ends
    in a ragged tile."""
    N, K = shape
    w, W32 = _random_packing(fq, 900 + bits, N, K, bits, fractional)
    X = np.eye(K, dtype=np.float16)
    want = np.ascontiguousarray(oracle.round_f16(W32.astype(np.float64)).T)
    for tile_rows in (128, 256, 0):   # either tile kernel, and the library's own choice
        y = host16(fq.fq_qlinear(dev(torch, X), w, tile_rows=tile_rows))
        assert y.shape == want.shape
        assert np.array_equal(y.view(np.uint16), want.view(np.uint16)), tile_rows


@pytest.mark.parametrize("fractional", [False, True], ids=["int_zero", "frac_zero"])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("M,shape", [(M, s) for M in (1, 16) for s in ((4096, 4096), (11008, 4096), (96, 512), (4096, 11008))] +
                         [(M, s) for M in (2, 3) for s in ((4096, 512), (5120, 512), (11008, 512), (96, 8064))] + [(2, (96, 8320))],
                         ids=lambda v: "N%d_K%d" % v if isinstance(v, tuple) else "M%d" % v)
def test_gemv_unpack_is_bit_exact_on_one_hot_rows(fq, torch, bits, M, shape, fractional):
    """One-hot activations: up to three rows the decode kernel, at sixteen the few-row kernel must return single
    dequantized weights rounded once to fp16 (bias, group exponent and zero all leave exactly).  4096 rows of weights at
    2 and 3 bits run the smallest work units of the decode kernel, 5120 at 3 bits halves, 11008 whole supertile rows, each
    with its body for one activation row and for several; long rows of 4 bits have a body of their own.  The positions
    walk through all 128 places of a group and through different groups."""
    N, K = shape
    assert fq.fq_qlinear_route(M, N, bits, K)[0] == ("stream" if M <= 3 else "few_rows")
    w, W32 = _random_packing(fq, 950 + bits, N, K, bits, fractional)
    want16 = oracle.round_f16(W32.astype(np.float64))
    G = K // 128
    for t in range(0, 128, 16 if M == 16 else 37):
        ks = [((5 * t + 7 * m) % G) * 128 + (t + m) % 128 for m in range(M)]
        X = np.zeros((M, K), dtype=np.float16)
        X[np.arange(M), ks] = 1.0
        y = host16(fq.fq_qlinear(dev(torch, X), w))
        want = np.ascontiguousarray(want16[:, ks].T)
        assert np.array_equal(y.view(np.uint16), want.view(np.uint16)), (t, ks[:3])


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("M", [1, 2, 3, 16])
@pytest.mark.parametrize("scale", [1e-2, 1e-3, 1e-4, 30.0])
def test_gemv_keeps_its_accuracy_for_small_and_large_activations(fq, torch, bits, M, scale):
    """The decode kernel (up to three rows) stages x times a power of two per bit field; a per-group exponent keeps the
    staged values normal fp16 numbers, so the 2e-3 bar holds whatever the scale of the activations (fq_qlinear
    takes any fp16 x), as it does for the few-row kernel, which takes x as it is, at M = 16 and 17."""
    N, K = 512, 4096
    w, codes, s, z = make_matrix(fq, 120 + bits, N, K, bits)
    W32 = oracle.dequant(codes, s, z)
    for rows in (M, 17):
        X = (fq_synth.activations(19, rows, K).astype(np.float32) * scale).astype(np.float16)
        X[0, 5] = np.float16(scale * 50.0)          # an outlier inside one group
        y = host16(fq.fq_qlinear(dev(torch, X), w))
        assert qerr(y, oracle.qlinear(X, W32)) <= TOL, rows


@pytest.mark.parametrize("bits", BITS)
def test_quantize_pack_qlinear_from_the_librarys_own_quantizer(fq, torch, bits):
    """Row a1 end to end: fp32 weights -> fq_quantize_rtn -> fq_pack_groups -> fq_qlinear, against the oracle's
    own quantizer, dequantizer and product from the same weights."""
    N, K = 300, 1024
    W = fq_synth.weights(140 + bits, N, K)
    codes, s, z = fq.fq_quantize_rtn(W, bits)
    oc, os_, oz = oracle.quantize_rtn(W, bits)
    assert np.array_equal(codes, oc) and np.array_equal(s.view(np.uint16), os_.view(np.uint16))
    assert np.array_equal(z.view(np.uint16), oz.view(np.uint16))
    w = fq.PackedMatrix.from_host(codes, s, z, bits)
    W32 = oracle.dequant(oc, os_, oz)
    assert np.array_equal(fq.fq_dequant(w).cpu().numpy().view(np.uint32), W32.view(np.uint32))
    for M in (1, 7, 48):
        X = fq_synth.activations(141, M, K)
        assert qerr(host16(fq.fq_qlinear(dev(torch, X), w)), oracle.qlinear(X, W32)) <= TOL, M


# ---------------------------------------------- guard bytes around every buffer
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("case", [(1, 70, 256), (5, 200, 384), (16, 96, 11008), (33, 70, 256), (300, 200, 384),
                                  (129, 1030, 512)], ids=lambda c: "M%d_N%d_K%d" % c)
def test_qlinear_writes_only_its_output(fq, torch, bits, case):
    """Ragged M and N: nothing outside out[M, N] is written, and what is written matches the oracle."""
    M, N, K = case
    w, codes, s, z = make_matrix(fq, 160 + bits, N, K, bits)
    X = fq_synth.activations(161, M, K)
    out = Guarded(torch, M * N * 2)
    fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N))
    torch.cuda.synchronize()
    assert out.intact()
    assert qerr(host16(out.half(M, N)), oracle.qlinear(X, oracle.dequant(codes, s, z))) <= TOL


@pytest.mark.parametrize("M", [1, 3, 40])
def test_stack_forward_stays_inside_output_and_workspace(fq, torch, M):
    """The workspace bound fq_stack_workspace_bytes is exact: one byte less is refused, and with exactly that
    many bytes nothing beyond the workspace or the output is touched."""
    stack, host, sh = build_stack(fq, "tiny", 330)
    bitvec = fq_synth.bit_vector(3, 7 * sh["layers"], probs=(0.25, 0.25, 0.25, 0.25))
    x = dev(torch, fq_synth.activations(331, M, sh["hidden"]))
    need = fq.fq_stack_workspace_bytes(M, sh["hidden"], sh["ffn"])
    ws, out = Guarded(torch, need), Guarded(torch, M * sh["hidden"] * 2)
    got = fq.fq_stack_forward(stack, bitvec, x, out=out.half(M, sh["hidden"]), workspace=ws.bytes())
    torch.cuda.synchronize()
    assert ws.intact() and out.intact()
    want = fq.fq_stack_forward(stack, bitvec, x)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    with pytest.raises(fq.FqError) as e:
        fq.fq_stack_forward(stack, bitvec, x, workspace=ws.bytes()[:need - 1])
    assert e.value.code == -6


@pytest.mark.parametrize("case", [(300, 1001, 256), (5, 70, 128), (257, 513, 384)], ids=str)
def test_head_nll_stays_inside_output_and_workspace(fq, torch, case):
    M, V, K = case
    X = dev(torch, fq_synth.activations(171, M, K))
    W = dev(torch, fq_synth.weights(172, V, K, 0.05, 99).astype(np.float16))
    lab = dev(torch, fq_synth.labels(173, M, V))
    need = fq.fq_head_nll_workspace_bytes(M, V)
    ws, out = Guarded(torch, need), Guarded(torch, M * 4)
    got = fq.fq_head_nll(X, W, lab, out=out.f32(M), workspace=ws.bytes())
    torch.cuda.synchronize()
    assert ws.intact() and out.intact()
    assert torch.equal(got, fq.fq_head_nll(X, W, lab))
    with pytest.raises(fq.FqError) as e:
        fq.fq_head_nll(X, W, lab, workspace=ws.bytes()[:need - 16])
    assert e.value.code == -6


def test_stream_read_reads_every_word_once(fq, torch):
    """The read-only measurement kernel: the XOR of its checksum words is the XOR of all 32-bit words of the
    buffer, whatever the split over workgroups (a size with a ragged tail of 16-byte units)."""
    n = (3 << 20) + 16 * 37
    rng = np.random.default_rng(5)
    host = rng.integers(0, 2 ** 32, size=n // 4, dtype=np.uint32)
    buf = torch.from_numpy(host.view(np.int32)).cuda()
    sink = fq.fq_stream_read(buf)
    torch.cuda.synchronize()
    got = np.bitwise_xor.reduce(sink.cpu().numpy().view(np.uint32))
    assert got == np.bitwise_xor.reduce(host)
    with pytest.raises(fq.FqError):
        fq.fq_stream_read(buf[:3])


# ------------------------------------------------- mixed widths within a matrix
MIXED_CASES = [
    (384, [(70, 8), (200, 2), (130, 4)]),                              # one launch of three runs, ragged everywhere
    (256, [(64, 3)]),                                                  # a single run: plain fq_qlinear
    (1024, [(16, 2), (48, 3), (100, 4), (33, 8), (64, 2)]),            # two launches; odd column offsets (no 8-byte rows)
    (512, [(128, 4), (128, 2), (256, 8), (128, 3), (64, 4), (64, 2), (32, 8), (224, 3)]),   # the most runs allowed
]


@pytest.mark.parametrize("M", [1, 5, 16, 40, 300])
@pytest.mark.parametrize("case", MIXED_CASES, ids=lambda c: "K%d_%druns" % (c[0], len(c[1])))
def test_qlinear_mixed_widths_within_a_matrix(fq, torch, M, case):
    """A matrix stored as runs of output rows at different bit-widths (Section "Large Language Model
    Quantization": widths vary within a module too): against the oracle's product with the runs' dequantized
    rows stacked, at the fq_qlinear tolerance; nothing outside out[M, sum N] written; and column range by
    column range what fq_qlinear gives for that run alone."""
    K, runs = case
    segs, rows = [], []
    for i, (N, bits) in enumerate(runs):
        w, codes, s, z = make_matrix(fq, 300 + 7 * i + bits, N, K, bits)
        segs.append(w)
        rows.append(oracle.dequant(codes, s, z))
    X = fq_synth.activations(31, M, K)
    want = oracle.qlinear(X, np.concatenate(rows, axis=0))
    total = sum(N for N, _ in runs)
    out = Guarded(torch, M * total * 2)
    fq.fq_qlinear_mixed(dev(torch, X), segs, out=out.half(M, total))
    torch.cuda.synchronize()
    assert out.intact()
    y = host16(out.half(M, total))
    assert qerr(y, want) <= TOL
    col = 0
    for w in segs:
        alone = host16(fq.fq_qlinear(dev(torch, X), w)).astype(np.float64)
        part = y[:, col:col + w.N].astype(np.float64)
        assert np.max(np.abs(part - alone)) <= 1e-3 * max(1.0, np.sqrt(np.mean(alone ** 2)))
        col += w.N


def test_qlinear_mixed_full_size_sampled(fq, torch):
    """The benchmark's mixed matrix (4096 rows as 60/30/10 % at 2/3/4 bits, K = 4096) at 1536 rows, where its one launch
    takes the 256-row tiles, with a row pitch wider than the runs' own N (odd run widths included).  Sampled rows and
    columns against the oracle; guard bytes."""
    K, M = 4096, 1536
    runs = [(2433, 2), (1231, 3), (432, 4)]
    assert fq.fq_qlinear_route(M, [N for N, _ in runs], [b for _, b in runs], K)[0] == "tiles_256"
    rng = np.random.default_rng(17)
    segs, sampled, cols_all, col0 = [], [], [], 0
    for i, (N, bits) in enumerate(runs):
        w, codes, s, z = make_matrix(fq, 900 + i, N, K, bits)
        segs.append(w)
        cols = np.unique(np.concatenate([rng.integers(0, N, size=64), [0, N - 1]]))
        sampled.append(oracle.dequant(codes[cols], s[cols], z[cols]))
        cols_all.append(col0 + cols)
        col0 += N
    X = fq_synth.activations(32, M, K)
    out = Guarded(torch, M * col0 * 2)
    fq.fq_qlinear_mixed(dev(torch, X), segs, out=out.half(M, col0))
    torch.cuda.synchronize()
    assert out.intact()
    y = host16(out.half(M, col0))
    assert np.all(np.isfinite(y.astype(np.float32)))
    rows = np.unique(np.concatenate([rng.integers(0, M, size=48), [0, 255, 256, M - 1]]))
    want = oracle.qlinear(X[rows], np.concatenate(sampled, axis=0))
    got = y[np.ix_(rows, np.concatenate(cols_all))].astype(np.float64)
    assert qerr(got, want) <= TOL


def test_qlinear_mixed_rejects_bad_arguments(fq, torch):
    w, *_ = make_matrix(fq, 1, 64, 128, 4)
    x = dev(torch, fq_synth.activations(1, 2, 128))
    with pytest.raises(fq.FqError):
        fq.fq_qlinear_mixed(x, [w] * 9)
    with pytest.raises(fq.FqError):
        fq.fq_qlinear_mixed(x, [])
    w2, *_ = make_matrix(fq, 2, 64, 256, 4)
    with pytest.raises(fq.FqError):
        fq.fq_qlinear_mixed(x, [w, w2])


def _random_cases(seed, count):
    rng = np.random.default_rng(seed)
    cases = []
    for _ in range(count):
        M = int(rng.choice([1, 2, 3, 7, 15, 16, 17, 31, 64, 100, 129, 257, 300]))
        N = int(rng.integers(1, 700))
        K = 128 * int(rng.integers(1, 13))
        bits = int(rng.choice(BITS))
        cases.append((M, N, K, bits))
    return cases


@pytest.mark.parametrize("case", _random_cases(2024, 48), ids=lambda c: "M%d_N%d_K%d_b%d" % c)
def test_qlinear_on_seeded_random_shapes(fq, torch, case):
    """Shapes nobody picked by hand: any M around the decode / matrix-core switch and the tile heights, any N
    (ragged against every supertile height), K from one group to twelve; either kernel family, both tile
    heights above 16 rows; guard bytes around the output."""
    M, N, K, bits = case
    w, codes, s, z = make_matrix(fq, 500 + N + bits, N, K, bits)
    X = fq_synth.activations(M + K, M, K)
    want = oracle.qlinear(X, oracle.dequant(codes, s, z))
    for tile_rows in ((0,) if M <= 16 else (128, 256)):
        out = Guarded(torch, M * N * 2)
        fq.fq_qlinear(dev(torch, X), w, out=out.half(M, N), tile_rows=tile_rows)
        torch.cuda.synchronize()
        assert out.intact(), tile_rows
        assert qerr(host16(out.half(M, N)), want) <= TOL, tile_rows


def test_qlinear_mixed_holds_its_segments(fq, torch):
    """A segment whose attributes are computed may change the list that it came in: the call goes on with the ones it was given."""
    x = dev(torch, fq_synth.activations(95, 5, 256))
    made = [fq.PackedMatrix.from_host(*oracle.quantize_rtn(fq_synth.weights(96 + n, n, 256), 4), 4) for n in (70, 64, 96)]
    want = fq.fq_qlinear_mixed(x, made)

    class Leaves:
        def __init__(self, w, segments):
            self.w, self.segments = w, segments

        def __getattr__(self, name):
            self.segments.clear()
            return getattr(self.w, name)

    segments = []
    segments += [Leaves(w, segments) for w in made]
    out = torch.zeros_like(want)
    assert fq.fq_qlinear_mixed(x, segments, out=out) is out and segments == []
    assert torch.equal(out, want)


def test_calls_with_an_output_agree_with_those_that_allocate(fq, torch):
    """With every buffer given a call goes through the extension module: the same results bit for bit, on the current stream, on one
    given by object or by handle, and the same refusals."""
    M, N, K, V = 5, 96, 256, 300
    x, W = dev(torch, fq_synth.activations(90, M, K)), dev(torch, fq_synth.weights(91, V, K, 0.05).astype(np.float16))
    lab = dev(torch, fq_synth.labels(92, M, V))
    w = fq.PackedMatrix.from_host(*oracle.quantize_rtn(fq_synth.weights(93, N, K), 4), 4)
    w3 = fq.PackedMatrix.from_host(*oracle.quantize_rtn(fq_synth.weights(94, 70, K), 3), 3)
    h, f = dict(dtype=torch.float16, device="cuda"), dict(dtype=torch.float32, device="cuda")
    logits = fq.fq_dense_f16(x, W)
    ws = torch.empty(fq.fq_head_nll_workspace_bytes(M, V), dtype=torch.uint8, device="cuda")
    calls = [(lambda **k: fq.fq_qlinear(x, w, **k), lambda: torch.empty(M, N, **h)),
             (lambda **k: fq.fq_qlinear(x.repeat(8, 1), w, tile_rows=128, **k), lambda: torch.empty(8 * M, N, **h)),
             (lambda **k: fq.fq_qlinear_mixed(x, [w, w3], **k), lambda: torch.empty(M, N + 70, **h)),
             (lambda **k: fq.fq_dense_f16(x, W, **k), lambda: torch.empty(M, V, **h)),
             (lambda **k: fq.fq_head_nll(x, W, lab, **(dict(k, workspace=ws) if k else k)), lambda: torch.empty(M, **f)),
             (lambda **k: fq.fq_token_nll(logits, lab, **k), lambda: torch.empty(M, **f)),
             (lambda **k: fq.fq_logit_l2(logits, logits.flip(0), **k), lambda: torch.empty(M, **f))]
    side = torch.cuda.Stream()
    for call, buffer in calls:
        want = call()
        torch.cuda.synchronize()
        for stream in (None, side, side.cuda_stream):
            out = buffer().fill_(7)
            torch.cuda.synchronize()
            assert call(out=out, **({} if stream is None else {"stream": stream})) is out
            torch.cuda.synchronize()
            assert torch.equal(out, want)
        with torch.cuda.stream(side):
            out = call(out=buffer().fill_(7))
        side.synchronize()
        assert torch.equal(out, want)
    with pytest.raises(fq.FqError):
        fq.fq_qlinear(x[:, :128].contiguous(), w, out=calls[0][1]())
    with pytest.raises(TypeError):
        fq.fq_qlinear(x.t(), w, out=calls[0][1]())
    with pytest.raises(TypeError):
        fq.fq_qlinear(x, w, out=calls[0][1]().float())
    with pytest.raises(fq.FqError):
        fq.fq_qlinear(x, w, out=calls[0][1](), group=64)
    with pytest.raises(fq.FqError):
        fq.fq_qlinear(x, w, out=calls[0][1](), tile_rows=64)
