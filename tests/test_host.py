"""Host logic of libfq against the oracle, and the shape of the C-ABI (no GPU needed)."""
import ctypes
import os
import re

import numpy as np
import pytest

import fq_synth
import oracle
import paper_2501_07139_amd as fq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BITS = (2, 3, 4, 8)


def test_library_exports_every_declared_symbol():
    text = open(os.path.join(ROOT, "include", "fq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(fq_[a-z0-9_]+)\s*\(", text))
    assert declared == set(fq.EXPORTS)
    lib = ctypes.CDLL(fq.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    assert "gfx950" in fq.fq_version()


@pytest.mark.parametrize("bits", BITS)
def test_quantizer_matches_oracle_bit_for_bit(bits):
    W = fq_synth.weights(40 + bits, 130, 640)
    W[3, :128] = 0.0
    W[4, 128:256] = np.abs(W[4, 128:256])
    W[5, :] *= 1e-7  # scales below the fp16 normal range
    W[6, :] *= 3e3   # large values
    got = fq.fq_quantize_rtn(W, bits)
    want = oracle.quantize_rtn(W, bits)
    for g, w in zip(got, want):
        assert np.array_equal(np.asarray(g).view(np.uint8), np.asarray(w).view(np.uint8))


@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("shape", [(1, 128), (70, 256), (64, 1024), (200, 384)])
def test_packer_against_oracle_unpack(bits, shape):
    N, K = shape
    G = K // 128
    for kind in range(4):
        if kind == 0:
            codes = fq_synth.codes(bits, N, K, bits, kind)
        elif kind == 1:
            codes = np.tile((np.arange(K) % (1 << bits)).astype(np.uint8), (N, 1))
        elif kind == 2:
            codes = np.tile((np.arange(N) % (1 << bits)).astype(np.uint8)[:, None], (1, K))
        else:
            codes = np.full((N, K), (1 << bits) - 1, dtype=np.uint8)
        s = fq_synth.activations(1, N, G).astype(np.float16)
        z = fq_synth.activations(2, N, G).astype(np.float16)
        packed, st, zt = fq.fq_pack_groups(codes, s, z, bits)
        assert packed.size == fq.fq_packed_bytes(N, K, bits) == oracle.packed_bytes(N, K, bits)
        assert packed.size == (N + 63) // 64 * 64 * K * bits // 8
        assert st.size == zt.size == fq.fq_meta_count(N, K) == (N + 63) // 64 * 64 * G
        assert np.array_equal(oracle.unpack(packed, N, K, bits), codes)
        assert np.array_equal(oracle.untile_meta(st, N, G).view(np.uint16), s.view(np.uint16))
        assert np.array_equal(oracle.untile_meta(zt, N, G).view(np.uint16), z.view(np.uint16))
    # pad rows are zero codes with zero scale
    Np = (N + 63) // 64 * 64
    if Np > N:
        full = oracle.unpack(packed, Np, K, bits)
        assert not full[N:].any()
        assert not oracle.untile_meta(st, Np, G)[N:].any()


def test_walking_one_code():
    N, K, bits = 64, 128, 3
    s = np.ones((N, 1), dtype=np.float16)
    z = np.zeros((N, 1), dtype=np.float16)
    for n, k in [(0, 0), (63, 127), (17, 102), (33, 103), (5, 19)]:
        codes = np.zeros((N, K), dtype=np.uint8)
        codes[n, k] = 5
        packed, _, _ = fq.fq_pack_groups(codes, s, z, bits)
        assert int(np.unpackbits(packed).sum()) == 2
        assert np.array_equal(oracle.unpack(packed, N, K, bits), codes)


def test_error_codes_without_launching_anything():
    W = np.zeros((4, 128), dtype=np.float32)
    with pytest.raises(fq.FqError) as e:
        fq.fq_quantize_rtn(W, 5)
    assert e.value.code == -3
    with pytest.raises(fq.FqError) as e:
        fq.fq_quantize_rtn(W, 4, group=64)
    assert e.value.code == -4
    with pytest.raises(fq.FqError) as e:
        fq.fq_quantize_rtn(np.zeros((4, 100), dtype=np.float32), 4)
    assert e.value.code == -2
    codes = np.full((4, 128), 9, dtype=np.uint8)
    with pytest.raises(fq.FqError) as e:
        fq.fq_pack_groups(codes, np.ones((4, 1), np.float16), np.zeros((4, 1), np.float16), 3)
    assert e.value.code == -3 and "fit" in str(e.value)
    assert fq.fq_packed_bytes(4, 100, 4) == 0 and fq.fq_packed_bytes(4, 128, 5) == 0
    lib = fq._lib
    assert lib.fq_qlinear(None, 1, None, None, None, 1, 128, 4, 128, None, None) == -1
    assert "NULL" in fq.fq_last_error()
    assert lib.fq_qlinear(16, 1, 16, 16, 16, 1, 128, 7, 128, 16, None) == -3
    assert lib.fq_qlinear(16, 1, 16, 16, 16, 1, 128, 4, 64, 16, None) == -4
    assert lib.fq_qlinear(16, 1, 16, 16, 16, 1, 100, 4, 128, 16, None) == -2
    assert lib.fq_qlinear(16, 1, 24, 16, 16, 1, 128, 4, 128, 16, None) == -5
    assert lib.fq_qlinear(16, 0, 16, 16, 16, 1, 128, 4, 128, 16, None) == -2
    assert lib.fq_token_nll(None, None, 1, 1, None, None) == -1
    assert lib.fq_logit_l2(None, 16, 1, 1, 16, None) == -1
    assert lib.fq_logit_l2(16, 16, 0, 8, 16, None) == -2
    assert lib.fq_logit_l2(16, 24, 1, 8, 16, None) == -5
    assert lib.fq_head_nll(None, 1, 16, 8, 128, 16, 16, 16, 1 << 20, None) == -1
    assert lib.fq_head_nll(16, 1, 16, 8, 100, 16, 16, 16, 1 << 20, None) == -2
    assert lib.fq_head_nll(16, 4, 16, 70, 128, 16, 16, 16, 8, None) == -6 and "need" in fq.fq_last_error()
    assert lib.fq_head_nll(16, 4, 16, 70, 128, 16, 16, None, 1 << 20, None) == -6
    assert lib.fq_head_nll(16, 4, 24, 70, 128, 16, 16, 16, 1 << 20, None) == -5
    assert fq.fq_head_nll_workspace_bytes(4, 70) == 4 * 2 * 8 + 4 * 4 and fq.fq_head_nll_workspace_bytes(0, 70) == 0
    assert fq.fq_head_nll_workspace_bytes(3, 64) % 16 == 0
    assert lib.fq_attn_decode(None, 16, 16, 16, 16, 0, 8, 2, 16, 16, 16, 1 << 20, None) == -1
    assert lib.fq_attn_decode(16, 16, 16, 16, 16, 8, 8, 2, 16, 16, 16, 1 << 20, None) == -2     # pos == Tmax
    assert lib.fq_attn_decode(16, 16, 16, 16, 16, 0, 8, 2, 16, 16, 16, 8, None) == -6
    assert lib.fq_attn_decode(16, 16, 24, 16, 16, 0, 8, 2, 16, 16, 16, 1 << 20, None) == -5
    assert fq.fq_attn_workspace_bytes(128, 2) >= 2 * 1 * 130 * 4 and fq.fq_attn_workspace_bytes(129, 2) >= 2 * 2 * 130 * 4
    assert fq.fq_decode_workspace_bytes(256, 640, 128) >= 8 * 512 + 2 * 1280 + fq.fq_attn_workspace_bytes(128, 2)
    assert fq.fq_decode_workspace_bytes(200, 640, 128) == 0
    assert lib.fq_attn_prefill(None, 16, 16, 4, 16, 16, 8, 2, 16, 16, 16, 1 << 24, None) == -1
    assert lib.fq_attn_prefill(16, 16, 16, 9, 16, 16, 8, 2, 16, 16, 16, 1 << 24, None) == -2     # T > Tmax
    assert lib.fq_attn_prefill(16, 16, 16, 4, 16, 16, 8, 2, 16, 16, 16, 8, None) == -6
    assert fq.fq_attn_prefill_workspace_bytes(65, 2) >= 65 * 256 * 2 + 256 * 128 * 2
    assert fq.fq_prefill_workspace_bytes(0, 256, 640) == 0 and fq.fq_prefill_workspace_bytes(4, 200, 640) == 0
    assert lib.fq_glue(9, 16, 16, 16, 1, 128, 16, None) == -2
    assert lib.fq_dense_f16(16, 1, 16, 1, 100, 16, None) == -2
    # the matrix-core kernels address their arrays through 32-bit offsets: 4 GiB of activations is refused
    assert lib.fq_qlinear(16, 1 << 20, 16, 16, 16, 128, 4096, 4, 128, 16, None) == -2
    assert "4 GiB" in fq.fq_last_error()
    assert lib.fq_dense_f16(16, 1 << 20, 16, 128, 4096, 16, None) == -2
    assert fq.fq_stack_workspace_bytes(0, 128, 128) == 0


def test_stack_forward_rejects_a_missing_packing_before_launching():
    layer = fq.fq_layer()
    for j in range(7):
        layer.m[j].N = 256 if j in (4, 5) else 128
        layer.m[j].K = 256 if j == 6 else 128
        for i in range(4):
            layer.m[j].packed[i] = 4096
            layer.m[j].scales[i] = 4096
            layer.m[j].zeros[i] = 4096
    layer.m[3].packed[1] = None  # no 3-bit packing for matrix o
    table = (fq.fq_layer * 1)(layer)
    bitvec = np.array([4, 4, 4, 3, 4, 4, 4], dtype=np.uint8)
    rc = fq._lib.fq_stack_forward(table, 1, bitvec.ctypes.data_as(ctypes.c_void_p), 4096, 4, 4096, 4096, 1 << 30, None)
    assert rc == -1 and "3-bit" in fq.fq_last_error()
    bitvec[3] = 5
    rc = fq._lib.fq_stack_forward(table, 1, bitvec.ctypes.data_as(ctypes.c_void_p), 4096, 4, 4096, 4096, 1 << 30, None)
    assert rc == -3
    bitvec[3] = 4
    rc = fq._lib.fq_stack_forward(table, 1, bitvec.ctypes.data_as(ctypes.c_void_p), 4096, 4, 4096, 4096, 16, None)
    assert rc == -6


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU only: asked for more it says so and exits without touching a device."""
    import subprocess
    import sys

    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "one GPU" in (r.stdout + r.stderr)


def test_rope_table_against_the_closed_form():
    """fq_rope_table: (cos, sin) of pos * base^(-2i/d), fp64 rounded once to fp32."""
    Tmax, d = 300, 128
    table = np.empty((Tmax, d // 2, 2), dtype=np.float32)
    rc = fq._lib.fq_rope_table(Tmax, d, 10000.0, table.ctypes.data_as(ctypes.c_void_p))
    assert rc == 0
    ang = np.arange(Tmax, dtype=np.float64)[:, None] * 10000.0 ** (-2.0 * np.arange(d // 2, dtype=np.float64) / d)
    # pow and ** may differ in the last place of the fp64 angle: one fp32 ulp of slack, exact almost everywhere
    assert np.max(np.abs(table[..., 0] - np.cos(ang))) <= 2.0 ** -23
    assert np.max(np.abs(table[..., 1] - np.sin(ang))) <= 2.0 ** -23
    assert np.array_equal(table[0, :, 0], np.ones(d // 2, dtype=np.float32)) and not table[0, :, 1].any()
    assert np.allclose(table[..., 0].astype(np.float64) ** 2 + table[..., 1].astype(np.float64) ** 2, 1.0, atol=3e-7)
    assert fq._lib.fq_rope_table(0, d, 10000.0, table.ctypes.data_as(ctypes.c_void_p)) == -2
    assert fq._lib.fq_rope_table(4, 7, 10000.0, table.ctypes.data_as(ctypes.c_void_p)) == -2
    assert fq._lib.fq_rope_table(4, d, 10000.0, None) == -1


def test_dense_tile_argument_is_validated_on_the_host():
    one = ctypes.c_void_p(16)
    assert fq._lib.fq_dense_f16_tile(one, 4, one, 4, 128, one, 64, None) == -2
    assert "tile_rows" in fq.fq_last_error()


def test_new_entry_points_validate_their_arguments_on_the_host():
    """fq_qlinear_tile, fq_qlinear_mixed and fq_stream_read refuse bad arguments before anything is launched."""
    import ctypes

    lib = fq._lib
    assert lib.fq_qlinear_tile(16, 32, 16, 16, 16, 64, 128, 4, 128, 16, 64, None) == -2 and "tile_rows" in fq.fq_last_error()
    assert lib.fq_qlinear_tile(None, 32, 16, 16, 16, 64, 128, 4, 128, 16, 256, None) == -1
    seg = (fq._Segment * 2)(fq._Segment(16, 16, 16, 64, 4), fq._Segment(16, 16, 16, 64, 5))
    p = ctypes.cast(seg, ctypes.c_void_p)
    assert lib.fq_qlinear_mixed(16, 1, p, 0, 128, 128, 16, None) == -2
    assert lib.fq_qlinear_mixed(16, 1, p, fq.MAX_SEGMENTS + 1, 128, 128, 16, None) == -2
    assert lib.fq_qlinear_mixed(16, 1, None, 1, 128, 128, 16, None) == -1
    assert lib.fq_qlinear_mixed(16, 1, p, 2, 128, 128, 16, None) == -3          # the second run's width
    assert lib.fq_qlinear_mixed(16, 1, p, 1, 100, 128, 16, None) == -2          # K
    assert lib.fq_qlinear_mixed(24, 1, p, 1, 128, 128, 16, None) == -5          # alignment of x
    assert lib.fq_qlinear_mixed(16, 0, p, 1, 128, 128, 16, None) == -2
    assert lib.fq_stream_read(None, 64, 16, None) == -1
    assert lib.fq_stream_read(16, 40, 16, None) == -2 and lib.fq_stream_read(16, 0, 16, None) == -2
    assert lib.fq_stream_read(24, 64, 16, None) == -5
    assert fq.fq_set_decode_mode(0) in (0, 1)


# ------------------------------------------------------------ dispatch by time
def route(M, N, bits, K):
    return fq.fq_qlinear_route(M, N, bits, K)[0]


@pytest.mark.parametrize("bits", BITS)
def test_few_row_kernel_leaves_the_sizes_that_others_run_faster(bits):
    """Sizes at which the few-row kernel was measured slower than the kernel of the general path: many rows whose
    activations no L2 holds (2048 x 1024 x 2816: 37 against 30 us in 128-row tiles, 24 to 29 in tall tiles of 128 rows), three and four rows of wide matrices (four of
    19741 x 1792: 11.0 against 9.2); and neighbours at which it is the faster one."""
    for M, N, K in ((2048, 1024, 2816), (1890, 1420, 6400), (2480, 1066, 15616)):
        assert fq.fq_qlinear_route(M, N, bits, K) == ("tiles_256", 128, 128)
    for M, N, K in ((1024, 1024, 2816), (512, 4096, 4096), (77, 4096, 11008), (300, 70, 256)):
        assert route(M, N, bits, K) == "few_rows"
    for M, N, K in ((3, 21160, 8192), (4, 19741, 1792), (4, 18581, 1024), (3, 4096, 4096), (2, 4096, 4096), (1, 11008, 4096)):
        assert route(M, N, bits, K) == "stream"
    for M, N, K in ((3, 4096, 11008), (4, 4096, 4096), (4, 16384, 4096), (4, 20000, 512), (4, 20000, 11008), (5, 20000, 2048), (16, 512, 512)):
        assert route(M, N, bits, K) == "few_rows"
    # 64 columns a tile just beyond one round of tiles over the chip pay for a second one (20739 x 1664: 11.3 against 9.8 us)
    assert fq.fq_qlinear_route(5, 20739, bits, 1664)[1:] == (16, 64 if bits == 3 else 32)
    assert fq.fq_qlinear_route(5, 16384, bits, 1664)[1:] == (16, 64)


def test_short_rows_stay_with_the_few_row_kernel():
    """Rows of up to 1280 for which the estimates of the large tiles are too low: measured 7.6 against 11.6 us at the first of
    these, 7.1 / 8.05, 7.5 / 11.6, 7.4 / 11.2, 6.2 / 8.9; and, of up to 32 columns, sizes whose scales the large tiles would round to fp16."""
    for M, N, bits, K in ((300, 2539, 3, 256), (55, 15513, 2, 256), (2126, 402, 3, 256), (1188, 650, 4, 256), (247, 2848, 3, 256)):
        assert route(M, N, bits, K) == "few_rows"
    for M, N, bits, K in ((52, 23114, 4, 768), (3470, [10, 240], [8, 8], 512), (2134, [4, 4, 322], [8, 8, 8], 512), (41, [1765, 16941], [2, 4], 640),
                          (2116, 454, 4, 512), (5706, [4, 40, 32], [8, 3, 8], 384), (1930, [124, 67, 260], [2, 4, 8], 1152)):
        name, _, columns = fq.fq_qlinear_route(M, N, bits, K)
        assert name == "few_rows" and columns < 64


def test_tiles_of_few_columns_by_their_measured_times():
    """Sizes whose tile an earlier fit of the estimates had missed: these tiles take 3.7, 3.8, 4.3, 4.5, 17.7 and 17.7 us, the ones taken
    then 4.4, 4.4, 5.2, 5.0, 20.3 and 19.2."""
    for M, N, bits, K, tile in ((71, 116, 3, 128, (16, 16)), (21, 68, 3, 256, (16, 16)), (797, 47, 2, 896, (16, 16)), (358, 131, 8, 896, (16, 16)),
                                (1153, 433, 4, 4480, (48, 64)), (784, 443, 8, 6016, (48, 32))):
        assert fq.fq_qlinear_route(M, N, bits, K) == ("few_rows", *tile)


def test_short_rows_of_five_blocks_keep_their_zeros_exact():
    """65 to 80 rows of up to 1024: not the tiles of 64 columns and several row blocks, which round code - zero to fp16, where three
    rounds of sixteen rows take little more time."""
    for M, N, bits, K in ((71, 8207, 2, 640), (80, 8250, 4, 1024), (73, 9473, 2, 1024), (69, 9624, 8, 640), (65, [1, 9368], [2, 4], 640),
                          (79, [3227, 12, 5099], [3, 8, 2], 896), (68, [48, 3, 9480], [3, 8, 4], 1024), (65, [9423, 80], [8, 3], 768), (35, [5241, 16], [8, 3], 5120)):
        name, rows, columns = fq.fq_qlinear_route(M, N, bits, K)
        assert name == "few_rows" and (rows == 16 or columns == 16 or (rows, columns) == (32, 32))


def test_tall_tiles_leave_short_rows_to_the_others():
    """A round of 256-row tiles has a fixed part that the 128-row ones lack: measured 11.9 against 9.0 us at the first of
    these, 13.0 / 10.0, 15.8 / 13.9, 13.4 / 11.9 (and 110 / 64 for two rounds, the second one almost empty); and sizes at which the tall ones are faster."""
    for M, N, bits, K in ((638, 17743, 3, 12544), (1152, 7079, 3, 8832)):  # and many rounds, to the 128-row ones: 328 against 341, 164 / 184 in few-row tiles
        assert route(M, N, bits, K) == "tiles_128"
    for M, N, bits, K in ((229, 20424, 4, 128), (1842, 3280, 3, 128), (1932, 3144, 4, 384), (675, 5636, 8, 256), (640, 11008, 4, 4096)):
        assert route(M, N, bits, K) == "tiles_128"
    for M, N, bits, K in ((2048, 11008, 2, 4096), (2048, 4096, 8, 11008), (2048, 11008, 3, 1024)):
        assert route(M, N, bits, K) == "tiles_256"


def test_route_takes_every_size_that_the_linear_takes():
    for M in (1, 2, 3, 4, 16, 17, 128, 129, 2048, 4096, 70000):
        for N in (1, 64, 70, 4096, 30000):
            for K in (128, 1152, 4096, 16384):
                name, rows, cols = fq.fq_qlinear_route(M, [N, N], [3, 8], K)
                assert name in fq.ROUTES and (rows > 0) == (cols > 0) == (name not in ("stream", "generic"))
                assert name in (("stream", "few_rows") if M <= 16 else ("few_rows", "tiles_128", "tiles_256"))
    assert route(3, 64, 4, (1 << 22) + 128) == "generic" and route(16, 64, 4, 1 << 22) == "few_rows"
    out = np.zeros(3, dtype=np.int32)
    one = np.array([4], dtype=np.int32)
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (one, one, out)]
    assert fq._lib.fq_qlinear_route(1, None, p[1], 1, 128, p[2]) == -1
    for M, count, K in ((0, 1, 128), (1, 0, 128), (1, 4, 128), (1, 1, 100), (1, 1, 0)):
        assert fq._lib.fq_qlinear_route(M, p[0], p[1], count, K, p[2]) == -2
    with pytest.raises(fq.FqError):
        fq.fq_qlinear_route(1, 64, 5, 128)


def test_large_tiles_by_their_measured_times():
    """Calls from K = 2048 on that an earlier estimate of the 128-row tiles had given to the slower kernel.  us in tall tiles and in the others:
    51.7 / 58.6, 64.4 / 74.9, 36.3 / 41.3, 65.5 / 74.0, 365 / 478, 298 / 367; then 183 / 150, 169 / 152, 148 / 133, 39.4 / 37.1,
    79.0 / 60.5, 155 / 122."""
    for M, N, bits, K in ((229, 22016, 8, 4096), (250, 22016, 8, 5120), (234, 17177, 2, 2304), (499, 11008, 8, 5120), (2174, [11008, 11008], [8, 2], 4096),
                          (1223, [13824, 13824], [4, 3], 4096)):
        assert route(M, N, bits, K) == "tiles_256"
    for M, N, bits, K in ((552, 12288, 2, 11008), (1811, 4164, 4, 10112), (1032, 7134, 2, 8960), (5473, 374, 3, 2816), (314, [15852, 850], [2, 3], 3968),
                          (538, [231, 1204, 10772], [4, 3, 2], 7424)):
        assert route(M, N, bits, K) == "tiles_128"


def test_route_names_the_kernel_and_the_height_of_its_tiles():
    """The 256-row kernel is named as itself however low its tiles are, with the height of the highest."""
    heights = set()
    for M, N, bits, K in ((1890, 1420, 2, 6400), (800, 22016, 4, 4096), (2048, 11008, 2, 4096), (1500, 11008, 2, 4096), (1536, [4096, 4096, 4096], [4, 3, 2], 4096)):
        name, rows, columns = fq.fq_qlinear_route(M, N, bits, K)
        assert (name, columns) == ("tiles_256", 128) and rows == fq.fq_qlinear_tall_tile(M, N, bits, K)[3]
        heights.add(rows)
    assert len(heights) > 3 and min(heights) == 128 and max(heights) == 256
    assert fq.fq_qlinear_route(640, 11008, 4, 4096) == ("tiles_128", 128, 128)


def test_tall_tiles_cover_every_row_once():
    """The kernel's own cut of the rows, up to the most whose activations stay below 4 GiB: tiles of one to sixteen blocks that follow one another
    from the first row to the last."""
    N, bits = np.array([64, 2000, 11008], dtype=np.int32), np.array([2, 8, 4], dtype=np.int32)
    out = np.zeros(4, dtype=np.int32)
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (N, bits, out)]
    cut = lambda M, count, K, tile: fq._lib.fq_qlinear_tall_tile(M, p[0], p[1], count, K, tile, p[2])
    for M, K in ((17, 128), (256, 128), (257, 384), (2048, 4096), (5003, 1024), (2965900, 640), (3355443, 640), ((1 << 24) - 1, 128)):
        assert cut(M, 1, K, 0) == 0
        row = 0
        for tile in range(out[0]):
            assert cut(M, 1, K, tile) == 0
            _, first, rows, worked = out.tolist()
            assert first == row and 1 <= rows <= worked and worked in (128, 160, 192, 208, 224, 240, 256), (M, K, tile, out)
            row += rows
        assert row == M and cut(M, 1, K, out[0]) == -2
    for M in (300, 611, 1536, 4000):  # as many tiles for the matrices of a launch together
        assert cut(M, 3, 4096, 0) == 0 and sum(fq.fq_qlinear_tall_tile(M, N, bits, 4096, t)[2] for t in range(out[0])) == M
    assert fq._lib.fq_qlinear_tall_tile(300, p[0], None, 1, 128, 0, p[2]) == -1
    for M, count, K, tile in ((0, 1, 128, 0), (300, 0, 128, 0), (300, 4, 128, 0), (300, 1, 100, 0), (300, 1, 128, -1), (1 << 24, 1, 128, 0)):
        assert cut(M, count, K, tile) == -2


@pytest.mark.parametrize("bits", BITS)
def test_parity_cases_reach_every_tile_of_the_few_row_kernel(bits):
    """The tile shapes that the rule chooses over 20000 sizes against those of the GPU tests' lists of cases, and their number: up
    to 64 rows eleven, and of 64 columns 80 rows, with less than 8 bits 96, 112 and 128 too."""
    from test_gpu_parity import SKINNY_CASES, WIDE_CASES

    rng = np.random.default_rng(7)
    size = lambda lo, hi: int(np.exp(rng.uniform(np.log(lo), np.log(hi))))
    draws = [(size(3, 3000), size(1, 30000), 128 * size(1, 130)) for _ in range(20000)]
    reached = {fq.fq_qlinear_route(M, N, bits, K) for M, N, K in draws}
    cases = SKINNY_CASES + [c for c, blocks in WIDE_CASES if bits < 8 or blocks <= 5]
    assert {r for r in reached if r[0] == "few_rows"} == {fq.fq_qlinear_route(M, N, bits, K) for M, N, K in cases}
    assert len({r for r in reached if r[0] == "few_rows"}) == (12 if bits == 8 else 15)


def test_logits_and_loss_share_k_together():
    """Sharing K changes the order of a logit's sum, so the head and the loss have to agree on it; and every size has a tile."""
    rng = np.random.default_rng(11)
    size = lambda lo, hi: int(np.exp(rng.uniform(np.log(lo), np.log(hi))))
    for _ in range(5000):
        M, V, K = size(1, 5000), size(1, 200000), 128 * size(1, 200)
        logits, loss = fq.fq_dense_route(M, V, K), fq.fq_dense_route(M, V, K, loss=True)
        assert (logits[0] == "shared_k") == (loss[0] == "shared_k") and logits[0] in fq.DENSE_ROUTES
        assert loss[0] != "shared_k" or loss[2] == 64
    out = np.zeros(3, dtype=np.int32)
    assert fq._lib.fq_dense_route(1, 1, 128, 0, None) == -1
    for M, V, K in ((0, 1, 128), (1, 0, 128), (1, 1, 100), (1, 1, 0)):
        assert fq._lib.fq_dense_route(M, V, K, 0, out.ctypes.data_as(ctypes.c_void_p)) == -2


def test_extension_module_leaves_what_it_does_not_take():
    """Anything but plain contiguous device tensors of the right type goes the long way, which raises."""
    import torch

    x, w = torch.zeros(2, 128, dtype=torch.float16), fq.PackedMatrix(*[torch.zeros(64)] * 3, 64, 128, 4)
    for call in (lambda: fq._bind.qlinear(x, w, x, None, 128, 0), lambda: fq._bind.qlinear(None, None, None, None, 128, 0),
                 lambda: fq._bind.qlinear(x, w, x), lambda: fq._bind.mixed(x, [w], x, None, 128), lambda: fq._bind.mixed(x, 5, x, None, 128),
                 lambda: fq._bind.dense_f16(x, x, x, None), lambda: fq._bind.head_nll(x, x, x, x, x, None),
                 lambda: fq._bind.token_nll(x, x, x, None), lambda: fq._bind.logit_l2(x, x, x, None)):
        assert call() is None
    for call in (lambda: fq.fq_qlinear(x, w, out=x), lambda: fq.fq_dense_f16(x, x, out=x), lambda: fq.fq_logit_l2(x, x, out=x),
                 lambda: fq.fq_token_nll(x, x, out=x), lambda: fq.fq_qlinear_mixed(x, [w], out=x), lambda: fq.fq_head_nll(x, x, x, out=x, workspace=x)):
        with pytest.raises(TypeError, match="device tensor"):
            call()


def test_no_kernel_uses_scratch_memory():
    """Registers that do not fit are kept in memory, and a kernel whose loops wait for their copies by count waits for all of them at
    every reload.  Read from the metadata that the compiler leaves in the library beside each kernel."""
    msgpack = pytest.importorskip("msgpack")
    import struct

    with open(os.path.join(os.path.dirname(fq.__file__), "libfq.so"), "rb") as f:
        raw = f.read()
    kernels, at = [], raw.find(b"AMDGPU\0")
    while at >= 0:
        name, size, kind = struct.unpack("<III", raw[at - 12:at])
        if (name, kind) == (7, 32):
            kernels += msgpack.unpackb(raw[at + 8:at + 8 + size])["amdhsa.kernels"]
        at = raw.find(b"AMDGPU\0", at + 7)
    assert len([k for k in kernels if "skinny_kernel" in k[".name"]]) == 15
    assert [k[".name"] for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]] == []


@pytest.mark.parametrize("lost", ["missing", "other torch"])
def test_package_works_without_the_extension_module(lost):
    """On a host whose Python or torch the extension module was not built for, the package imports and its calls go through ctypes."""
    import subprocess
    import sys

    code = """
import sys, warnings, torch
if sys.argv[1] == "missing":
    sys.modules["paper_2501_07139_amd._bind"] = None
else:
    torch.__version__ = "0.0"
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import paper_2501_07139_amd as fq
assert fq._bind is None and any("_bind" in str(w.message) for w in seen)
assert fq.fq_qlinear_route(77, 4096, 3, 11008)[0] == "few_rows"
x, w = torch.zeros(2, 128, dtype=torch.float16), fq.PackedMatrix(*[torch.zeros(64)] * 3, 64, 128, 4)
for call in (lambda: fq.fq_qlinear(x, w, out=x), lambda: fq.fq_dense_f16(x, x, out=x), lambda: fq.fq_logit_l2(x, x, out=x),
             lambda: fq.fq_token_nll(x, x, out=x), lambda: fq.fq_qlinear_mixed(x, [w], out=x), lambda: fq.fq_head_nll(x, x, x, out=x, workspace=x)):
    try:
        call()
    except TypeError as e:
        assert "device tensor" in str(e)
    else:
        raise AssertionError("accepted a host tensor")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code, lost], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
