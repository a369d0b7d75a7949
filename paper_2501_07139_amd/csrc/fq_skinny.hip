// Dequant-GEMM for few rows: prompts, batched decoding, the remainder of a sequence (FlexQuant, arXiv 2501.07139,
// Section "Introduction": the hosted model is served on prompts of any length).
//
// What bounds it.  At tens of rows the packed weights are read once and the matrix cores have little to do; a tile
// of 128 x 128 would leave most CUs idle (4096 columns are 32 such tiles) and walk all of K one group after another.
// Here a workgroup owns 16*MB rows x 16*S columns of the output and its eight wavefronts share K: wavefront w takes
// groups w, w + 8, ...  The wavefronts have nothing to exchange before their partial sums meet in LDS at the end, so
// there is no barrier in the loop.  Weights come as packed chunks (a lane's 32 weights of a group are its operands of
// four k-steps) straight from global memory into registers, requested when the group before them has been unpacked;
// activations through a ring of half groups in LDS that is the wavefront's own, filled by direct copies (as operands straight
// from global memory, consecutive lanes in different rows, they took twice as long).
//
// Arithmetic: code - zero in fp16, fp32 sums per group, and the group's scale applied to the sum in fp32; tiles too large
// for a second set of accumulators scale the weights in fp16 instead, like the large tiles of the calibration
// forward.  Tiles of sixteen rows, which decoding uses, multiply the codes and take the zero from the group's sum in fp32
// (see ZERO_APART).  Sums over the wavefronts in a fixed order.
#include "fq_device.h"
#include "fq_internal.h"

namespace {

constexpr int SNW = 8; // wavefronts per workgroup, each a slice of K

struct SkinnyJob {
    const uint32_t *packed;
    const _Float16 *scales, *zeros;
    _Float16 *out;
    int N, bits, tile0, ld; // tile0: index of the matrix's first tile in the launch's list
};
struct SkinnyJobs {
    SkinnyJob j[3];
    int count, total;
};

// The packed dwords of S consecutive sixteen-row sub-blocks of group g.  S divides 4 and the rows of a matrix are padded
// to 64, so every sub-block exists.  packed: descriptor of the supertile rows from the one that holds the first sub-block;
// part: the first sub-block's place in it.
template <int BITS, int S>
__device__ __forceinline__ void skinny_load(fq_rsrc packed, int part, int G, int g, int lane, uint32_t (&C)[S][BITS])
{
    constexpr int SUB = Fmt<BITS>::SUB, TILE = tile_dwords<BITS>() * 4;
    constexpr int PER = S < SUB ? S : SUB; // sub-blocks taken from one supertile
#pragma unroll
    for (int t = 0; t < S / PER; ++t) {
        const uint32_t off = (uint32_t)(t * G + g) * (uint32_t)TILE;
        if constexpr (SUB == 1) {
            buf_load_chunk<BITS>(packed, off, 0, lane, C[t]);
        } else if constexpr (PER == SUB) { // whole planes: the sub-blocks' dwords are consecutive in a lane's run over them
            u4v pl[Fmt<BITS>::PLANES];
#pragma unroll
            for (int p = 0; p < Fmt<BITS>::PLANES; ++p)
                pl[p] = buf_load_b128(packed, (uint32_t)lane * 16u + 1024u * p, off);
#pragma unroll
            for (int j = 0; j < SUB * BITS; ++j) {
                const u4v v = pl[j >> 2];
                C[t * PER + j / BITS][j % BITS] = (j & 3) == 0 ? v.x : ((j & 3) == 1 ? v.y : ((j & 3) == 2 ? v.z : v.w));
            }
        } else {
#pragma unroll
            for (int u = 0; u < PER; ++u)
                buf_load_chunk<BITS>(packed, off, part + u, lane, C[u]);
        }
    }
}

// The four k-steps' operands of a chunk: code - zero in fp16, times the scale if SCALED (see unpack_khalf).
template <int BITS, bool INTZ, bool SCALED>
__device__ __forceinline__ void skinny_unpack(const uint32_t (&C)[BITS], h2 zero2, h2 scale2, h8 (&a)[4])
{
    UnpackConsts<BITS> uc; // afresh: what the two forms share would be taken out of them, ahead of the branch
    uc.init();
    h8 lo[2], hi[2];
    unpack_khalf<BITS, INTZ, SCALED, 0>(C, zero2, scale2, uc, lo);
    unpack_khalf<BITS, INTZ, SCALED, 1>(C, zero2, scale2, uc, hi);
    a[0] = lo[0];
    a[1] = lo[1];
    a[2] = hi[0];
    a[3] = hi[1];
}

// The four halves that lane FROM of each run of sixteen lanes holds, in all of its lanes.
template <int FROM>
__device__ __forceinline__ h4 row16_bcast(u2v v)
{
    constexpr int CTRL = 0x150 + FROM; // row_newbcast
    const u2v all = {(uint32_t)__builtin_amdgcn_update_dpp(0, (int)v.x, CTRL, 0xf, 0xf, true),
                     (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v.y, CTRL, 0xf, 0xf, true)};
    return __builtin_bit_cast(h4, all);
}

// Activation stages of half a group (two k-steps, 128 bytes a row) that a wavefront keeps in LDS.
template <int MB>
struct SkinnyRing { static constexpr int H = MB <= 2 ? 4 : 2, STAGE = 16 * MB * 8; }; // STAGE: 16-byte slots

// LDS in 16-byte slots: the wavefronts' rings, and later the partial sums.
template <int MB, int S>
constexpr int skinny_slots()
{
    constexpr int ring = SNW * SkinnyRing<MB>::H * SkinnyRing<MB>::STAGE, red = SNW * MB * S * 64;
    return ring > red ? ring : red;
}

// One tile of 16*MB rows x 16*S columns.
template <int BITS, int MB, int S>
__device__ __forceinline__ void skinny_tile(h8 *smem, const _Float16 *__restrict__ x, int M, int K, const SkinnyJob job,
                                            int tile, int row_tiles)
{
    constexpr bool F32 = S < 4 || MB == 1; // scale applied to the group's sums in fp32
    // Zeros leave through the group's sums, sum code x - zero sum x, so that any fp16 zero is exact, as in the decode kernel
    // (2048 x 2048, 16 rows at 2 bits, error over the rms of the result: 2.06e-4, the output's own rounding; with code - zero
    // in fp16 2.3e-4 for fractional zeros and 4.0e-4 for odd ones beyond 1024).  sum x is one more matrix product, of rows
    // of ones: level in time, and there is no branch on the zeros.
    constexpr bool ZERO_APART = MB == 1;
    constexpr int H = SkinnyRing<MB>::H, STAGE = SkinnyRing<MB>::STAGE, COPIES = 2 * MB;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, c = lane >> 4;
    const int G = K >> 7;
    const int m0 = (tile % row_tiles) * (16 * MB), sb0 = (tile / row_tiles) * S;
    // descriptors of what the tile reads of the matrix: S sub-blocks of every group
    constexpr int SUB = Fmt<BITS>::SUB, TILE = tile_dwords<BITS>();
    const fq_rsrc packed = make_rsrc(job.packed + (size_t)(sb0 / SUB) * G * TILE, (uint32_t)((S + SUB - 1) / SUB * G) * (TILE * 4u));
    const fq_rsrc scales = make_rsrc(job.scales + (size_t)sb0 * G * 16, (uint32_t)(S * G) * 32u);
    const fq_rsrc zeros = make_rsrc(job.zeros + (size_t)sb0 * G * 16, (uint32_t)(S * G) * 32u);

    f4 acc[S][MB];
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j)
            acc[u][j] = f4{0.f, 0.f, 0.f, 0.f};

    if (wave < G) { // uniform over the wavefront
        // Activation copies, global memory straight into this wavefront's ring: copy i of a stage fills rows 8i ..
        // 8i + 7, slot (row, pos) with chunk pos ^ (row / 2) % 8 of the row's eight, so that the operand reads below
        // touch every bank once.  Rows past M re-read the last row: their results are not stored.
        h8 *const ring = smem + wave * (H * STAGE);
        const fq_rsrc xr = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2u);
        uint32_t xoff[COPIES];
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int row = 8 * i + (lane >> 3);
            xoff[i] = ((uint32_t)min(m0 + row, M - 1) * (uint32_t)K + 8u * (uint32_t)((lane & 7) ^ ((row >> 1) & 7))) * 2u;
        }
        const int turns = (G - wave + SNW - 1) / SNW, stages = 2 * turns; // groups and half groups of this wavefront
        auto copy = [&](int h) { // past the end: the last half group again, into a slot that is not read any more
            const int hc = min(h, stages - 1);
            const uint32_t off = (uint32_t)(wave + SNW * (hc >> 1)) * 256u + (uint32_t)(hc & 1) * 128u;
            h8 *dst = ring + (h & (H - 1)) * STAGE;
#pragma unroll
            for (int i = 0; i < COPIES; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, dst + 64 * i, 16, xoff[i], off, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        uint32_t w[S][BITS];
        h4 sc[S];              // F32: scales of the rows 4c..4c+3, whose sums the lane holds
        uint32_t ss[S], zr[S]; // scale (not F32) and zero of the row r, whose weights the lane unpacks
        // ZERO_APART: scales and zeros of the rows 4c..4c+3 of two sub-blocks in one load: all lanes of one c need the same
        // eight bytes of each, so lanes r / 4 = 0, 1, 2, 3 take scales and zeros of the first, then of the second, and
        // the others get them by broadcasts within the sixteen lanes (21085 x 1024 at 2 bits, 6 rows: 9.3 us with a load for
        // each, 8.1 with this one).
        constexpr int NM = (S + 1) / 2;
        const char *meta_lane[NM];
        u2v meta[NM];
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            const _Float16 *from = (r & 4) ? job.zeros : job.scales;
            meta_lane[q] = reinterpret_cast<const char *>(from + ((size_t)(sb0 + min(2 * q + (r >> 3), S - 1)) * G * 16 + 4 * c));
        }
        auto load_w = [&](int t) { // past the end: the last group again (nobody uses it)
            const int g = min(wave + SNW * t, G - 1);
            skinny_load<BITS, S>(packed, sb0 % SUB, G, g, lane, w);
            if constexpr (ZERO_APART) {
#pragma unroll
                for (int q = 0; q < NM; ++q)
                    meta[q] = *reinterpret_cast<const u2v *>(meta_lane[q] + (size_t)g * 32);
                return;
            }
#pragma unroll
            for (int u = 0; u < S; ++u) {
                const uint32_t at = (uint32_t)(u * G + g) * 32u;
                zr[u] = buf_load_u16(zeros, 2u * (uint32_t)r, at);
                if constexpr (F32)
                    sc[u] = __builtin_bit_cast(h4, buf_load_b64(scales, 8u * (uint32_t)c, at));
                else
                    ss[u] = buf_load_u16(scales, 2u * (uint32_t)r, at);
            }
        };
        load_w(0);
#pragma unroll
        for (int h = 0; h < H; ++h)
            copy(h);
        int rd[2]; // slot of operand (row r, k-step s of the half group); block j is 128 slots further
#pragma unroll
        for (int s = 0; s < 2; ++s)
            rd[s] = r * 8 + ((4 * s + c) ^ (r >> 1));
        for (int t = 0; t < turns; ++t) {
            h8 a[S][4];
            float scf[S][4], zf[S][4];
            static_for<S>([&](auto u_tag) {
                constexpr int u = decltype(u_tag)::value;
                if constexpr (ZERO_APART) {
                    skinny_unpack<BITS, true, !F32>(w[u], h2{0, 0}, h2{}, a[u]); // the codes themselves
                    const h4 s4 = row16_bcast<8 * (u & 1)>(meta[u / 2]), z4 = row16_bcast<8 * (u & 1) + 4>(meta[u / 2]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        scf[u][v] = (float)s4[v];
                        zf[u][v] = (float)z4[v];
                    }
                } else {
                    const h2 z2 = as_h2(zr[u] * 0x10001u), s2 = F32 ? h2{} : as_h2(ss[u] * 0x10001u);
                    const _Float16 z = z2[0];
                    // integer zeros (what the quantizer produces): bias and zero leave in one addition
                    if (__builtin_amdgcn_ballot_w64(z != __builtin_truncf16(z)) == 0)
                        skinny_unpack<BITS, true, !F32>(w[u], z2, s2, a[u]);
                    else
                        skinny_unpack<BITS, false, !F32>(w[u], z2, s2, a[u]);
                    if constexpr (F32) {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            scf[u][v] = (float)sc[u][v];
                    }
                }
            });
            load_w(t + 1);
            f4 p[S][MB], xs = {0.f, 0.f, 0.f, 0.f}; // xs: sum over the group of the lane's activation row
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                // The stage's copies are older than the COPIES * (H - 1) copies of the stages behind it.  The loads of
                // load_w lie between them too but are not counted, so the wait reaches into the next group's weights,
                // asked for half a turn ago or less.
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(vmcnt_at_most(COPIES * (H - 1)));
                __builtin_amdgcn_sched_barrier(0);
                const h8 *stage = ring + ((2 * t + half) & (H - 1)) * STAGE;
                h8 xf[2][MB];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int j = 0; j < MB; ++j)
                        xf[s][j] = stage[rd[s] + 128 * j];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int u = 0; u < S; ++u)
#pragma unroll
                        for (int j = 0; j < MB; ++j) {
                            if constexpr (F32)
                                p[u][j] = mfma16x16x32(a[u][2 * half + s], xf[s][j], (half | s) == 0 ? f4{0.f, 0.f, 0.f, 0.f} : p[u][j]);
                            else
                                acc[u][j] = mfma16x16x32(a[u][2 * half + s], xf[s][j], acc[u][j]);
                        }
                if constexpr (ZERO_APART) {
                    const _Float16 one = 1;
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        xs = mfma16x16x32(h8{one, one, one, one, one, one, one, one}, xf[s][0], xs);
                }
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(FQ_WAIT_LGKMCNT0); // the operands have left the slot
                copy(2 * t + half + H);
            }
            if constexpr (F32) {
#pragma unroll
                for (int u = 0; u < S; ++u)
#pragma unroll
                    for (int j = 0; j < MB; ++j)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            acc[u][j][v] = fmaf(scf[u][v], ZERO_APART ? fmaf(-zf[u][v], xs[v], p[u][j][v]) : p[u][j][v], acc[u][j][v]);
            }
        }
    }

    // The partial sums take the rings' memory: every wavefront's copies have to land first.
    __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0);
    __syncthreads();
    f4 *red = reinterpret_cast<f4 *>(smem);
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j)
            red[((wave * S + u) * MB + j) * 64 + lane] = acc[u][j];
    __syncthreads();
    // block (u, j): lane holds m = 16j + lane%16 and n = 16u + 4*(lane/16) + v; four values at once where every row of
    // the output (a column range of a wider array when ld > N) starts 8-byte aligned
    const bool vec_ok = (job.ld & 3) == 0 && (reinterpret_cast<uintptr_t>(job.out) & 7) == 0;
    const int waves = min(SNW, G);
    for (int b = wave; b < S * MB; b += SNW) {
        f4 sum = red[b * 64 + lane];
        for (int w = 1; w < waves; ++w)
            sum += red[(w * S * MB + b) * 64 + lane];
        const int m = m0 + 16 * (b % MB) + r, n = 16 * (sb0 + b / MB) + 4 * c;
        if (m >= M)
            continue;
        _Float16 *o = job.out + (size_t)m * job.ld + n;
        if (n + 3 < job.N && vec_ok) {
            *reinterpret_cast<h4 *>(o) = h4{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (n + v < job.N)
                    o[v] = (_Float16)sum[v];
        }
    }
}

template <int MB, int S>
__global__ __launch_bounds__(64 * SNW, (MB == 1 && S <= 2) ? 4 : 2) void skinny_kernel(const _Float16 *__restrict__ x, int M, int K,
                                                                                 int row_tiles, SkinnyJobs jobs)
{
    __shared__ h8 smem[skinny_slots<MB, S>()]; // the kernel's only LDS object: see the waits in skinny_tile
    // the workgroups of an XCD take a contiguous run of tiles (row-tile fastest): tiles that share weights share an L2
    const int per_xcd = (jobs.total + 7) >> 3;
    int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= jobs.total)
        return; // uniform over the workgroup, before any barrier
    SkinnyJob job = jobs.j[0];
    if (jobs.count > 1 && tile >= jobs.j[1].tile0)
        job = jobs.j[1];
    if (jobs.count > 2 && tile >= jobs.j[2].tile0)
        job = jobs.j[2];
    tile -= job.tile0;
    switch (job.bits) {
    case 2: skinny_tile<2, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    case 3: skinny_tile<3, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    case 4: skinny_tile<4, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    default: skinny_tile<8, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    }
}

typedef void (*SkinnyKernel)(const _Float16 *, int, int, int, SkinnyJobs);

constexpr int SKINNY_CUS = 256;

struct SkinnyPlan {
    int mb, s_log2, row_tiles;
    double us;
};

// Tile shape for a launch of more than sixteen rows.  The time of a shape, as fitted to measurements at 4096 x 4096, 11008
// x 4096 and 4096 x 11008, all widths, 1 to 512 rows: a launch costs 2 us, a round of tiles over the chip 1.6 us (3.2
// us for the largest sums to add up) beside its turns of eight groups, and a turn 0.1 + 0.29 S + 0.34 MB us -- unpacking S
// sub-blocks and moving MB row blocks of activations add up, the matrix instructions hide behind them.  8-bit chunks
// are twice the bytes, 3-bit ones that are less than a supertile come in single dwords (0.39 and 0.45 S us).  The
// smallest shapes leave room for a second workgroup on a CU, so their rounds are not whole ones.  4 x 1 is never ahead
// of 2 x 2.  The turns take no less than the activations need to reach an XCD's L2 at 0.8 TB/s: with thirty and more row
// tiles the tiles that an XCD works on share hardly any (2048 rows of 1024 x 2816: 37 us where the turns alone would be 24).
// Over 2300 sizes of 17 to 3000 rows half the launches are within 9 % of this, a twentieth more than 25 % off.
//
// Up to sixteen rows every shape has one row block and the number of sub-blocks is all there is to choose (it does not change
// a sum).  Fitted to 2500 sizes of 64 to 24000 columns with each S: 3.4 us and a turn of 0.13 + 0.28 S us (8 bits 0.37 S;
// 3-bit S < 4: 0.2 + 0.5 S) while every CU has one tile; a second one on some CUs costs nearly a second turn, and from two a
// CU on the time grows with the tiles.  64 columns a tile just beyond one round (20739 x 1664, 4 bits) 11.3 us, 32 columns 9.8.
SkinnyPlan skinny_plan(int M, const fq_packed_ref *w, int count)
{
    SkinnyPlan best = {1, 0, 1, 1e30};
    const int blocks = (M + 15) / 16, turns = ((w[0].K >> 7) + SNW - 1) / SNW;
    for (int sl = 0; sl < 3; ++sl) {
        const int S = 1 << sl;
        long col_tiles = 0;
        double sub = 0.0, one_block = 0.0; // us of a turn: a sub-block's; all of a tile of one row block
        for (int i = 0; i < count; ++i) {
            col_tiles += (w[i].N + 16 * S - 1) / (16 * S);
            const bool dwords = w[i].bits == 3 && S < 4;
            const double u = w[i].bits == 8 ? 0.39 : (dwords ? 0.45 : 0.29);
            sub = sub > u ? sub : u;
            const double t = dwords ? 0.2 + 0.5 * S : 0.13 + (w[i].bits == 8 ? 0.37 : 0.28) * S;
            one_block = one_block > t ? one_block : t;
        }
        if (blocks == 1) {
            const double waves = (double)col_tiles / SKINNY_CUS;
            double fixed = 3.4, factor = 1.0;
            if (waves > 1.0 && S == 4) {
                factor = (double)(long)(waves + 0.999);
                fixed = 2.4 + factor;
            } else if (waves > 1.0) {
                factor = S == 1 ? (waves <= 2.0 ? 2.2 : 1.5 * waves) : (waves <= 2.0 ? 1.9 : 1.25 * waves);
                fixed = 3.1 + 0.3 * waves;
            }
            const double us = fixed + factor * turns * one_block;
            if (us < best.us)
                best = {1, sl, 1, us};
            continue;
        }
        for (int mb = 1; mb <= (S == 1 ? 3 : 4); ++mb) {
            const int row_tiles = (blocks + mb - 1) / mb;
            if ((blocks + row_tiles - 1) / row_tiles != mb)
                continue; // as many row tiles of fewer blocks do
            const double tiles = (double)row_tiles * (double)col_tiles, waves = tiles / SKINNY_CUS;
            const double rounds = waves <= 1.0 ? 1.0 : ((mb == 1 && S <= 2) ? 1.15 * waves : (double)(long)(waves + 0.999));
            const double in_xcd = tiles > 8.0 ? tiles / 8.0 : 1.0; // 32 of them at a time, row-tile fastest
            const double rows = 16.0 * mb * (row_tiles < 32 ? (row_tiles < in_xcd ? row_tiles : in_xcd) : (in_xcd < 32.0 ? in_xcd : 32.0));
            const double l2 = (in_xcd > 32.0 ? in_xcd / 32.0 : 1.0) * rows * w[0].K * 2.0 / 0.8e6; // us
            const double work = rounds * turns * (0.1 + sub * S + 0.34 * mb);
            const double us = 2.0 + rounds * (S == 4 && mb > 1 ? 3.2 : 1.6) + (work > l2 ? work : l2);
            if (us < best.us)
                best = {mb, sl, row_tiles, us};
        }
    }
    return best;
}

// Time of the 128-row tile kernel on the same launch: 5.4 us and 1.31 us a group of 128 k up to one tile a CU, from 1.5
// us (3 bits: 1.8) a group on with two on some.  Over 2300 sizes the time is 0.8 to 1.15 of this from K = 1024 on, where at
// most one tile a CU is there, and 1 to 1.5 below; with more tiles 0.86 to 1.1 from K = 4096 on and up to twice this on short
// rows, which go to the few-row kernel.
double tile_kernel_us(int M, const fq_packed_ref *w, int count)
{
    long tiles = 0;
    double three = 0.0;
    for (int i = 0; i < count; ++i) {
        tiles += (long)((w[i].N + 127) / 128) * ((M + 127) / 128);
        three = w[i].bits == 3 ? 0.3 : three;
    }
    if (tiles > 2 * SKINNY_CUS)
        return 0.0; // several rounds of tiles fill the chip: the large tiles are the better ones
    const double group = tiles <= SKINNY_CUS ? 1.31 : 1.5 + three + 0.7 * (tiles - SKINNY_CUS) / SKINNY_CUS;
    return 5.4 + (w[0].K >> 7) * group;
}

} // namespace

// Whether the kernel's 32-bit byte offsets reach all of a launch's activations and of a tile's weights.
bool fq_skinny_can(int M, int K) { return K <= (1 << 22) && (size_t)M * K * 2 < ((size_t)1 << 32); }

// Whether a launch goes to the skinny kernel.  Few rows (M <= 16): from four rows on, three of long rows, where the
// streaming kernel stages one row after another (4096 x 4096, 4 bits: 7.5 against 5.8 us at 4 rows, 17 against 6.0 at 16; at
// one row 4.2 against 6.1; 4096 x 11008 at 3 rows 11.3 against 10), and where that kernel has no room for the rows.  Four
// rows of more columns than one round of the widest tiles covers stay with the streaming kernel unless they are
// short or long ones (19741 x 1792 at 2 bits 9.2 against 11.0 us, and level on average from 1024 to 8192; below, 0.75 of
// its time, above 0.9), three also if they are long (21160 x 8192 at 3 bits 22.6 against 25.2).  More rows: where the models above put it ahead of the tile kernel (4096 x 11008, 3 bits: 23 against
// 109 us at 77 rows, 34 against 116 at 256, 64 against 117 at 512; 1024 x 2816, 2 bits, at 2048 rows 37 against 30).
bool fq_skinny_pays(int M, const fq_packed_ref *w, int count)
{
    if (!fq_skinny_can(M, w[0].K))
        return false;
    if (M > 16)
        return skinny_plan(M, w, count).us < tile_kernel_us(M, w, count);
    const int K = w[0].K;
    long columns = 0;
    for (int i = 0; i < count; ++i)
        columns += w[i].N;
    const bool wide = columns > 64 * SKINNY_CUS;
    bool stream = M < 3 || (M == 3 && (K < 8192 || wide)) || (M == 4 && K >= 1024 && K < 8192 && wide);
    for (int i = 0; i < count; ++i)
        stream = stream && fq_gemv_can_stream(M, K, w[i].bits, 0);
    return !stream;
}

void fq_skinny_tile(int M, const fq_packed_ref *w, int count, int *rows, int *columns)
{
    const SkinnyPlan plan = skinny_plan(M, w, count);
    *rows = 16 * plan.mb;
    *columns = 16 << plan.s_log2;
}

// Up to three matrices that share the input (same K), in one launch.
int fq_launch_skinny(const void *x, int M, const fq_packed_ref *w, void *const *outs, int count, fq_stream st)
{
    static const SkinnyKernel table[4][3] = {
        {skinny_kernel<1, 1>, skinny_kernel<1, 2>, skinny_kernel<1, 4>},
        {skinny_kernel<2, 1>, skinny_kernel<2, 2>, skinny_kernel<2, 4>},
        {skinny_kernel<3, 1>, skinny_kernel<3, 2>, skinny_kernel<3, 4>},
        {nullptr, skinny_kernel<4, 2>, skinny_kernel<4, 4>},
    };
    const SkinnyPlan plan = skinny_plan(M, w, count);
    SkinnyJobs jobs;
    jobs.count = count;
    int total = 0;
    for (int i = 0; i < count; ++i) {
        jobs.j[i] = SkinnyJob{static_cast<const uint32_t *>(w[i].packed), static_cast<const _Float16 *>(w[i].scales),
                              static_cast<const _Float16 *>(w[i].zeros), static_cast<_Float16 *>(outs[i]), w[i].N, w[i].bits,
                              total, w[i].ld ? w[i].ld : w[i].N};
        total += plan.row_tiles * ((w[i].N + (16 << plan.s_log2) - 1) >> (4 + plan.s_log2));
    }
    for (int i = count; i < 3; ++i)
        jobs.j[i] = jobs.j[0];
    jobs.total = total;
    hipLaunchKernelGGL(table[plan.mb - 1][plan.s_log2], dim3(8 * ((total + 7) / 8)), dim3(64 * SNW), 0, st,
                       static_cast<const _Float16 *>(x), M, w[0].K, plan.row_tiles, jobs);
    return (int)hipGetLastError();
}
