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
// Two bodies: tiles of 16 or 32 columns, or of sixteen rows (skinny_tile), and tiles of 64 columns and two to eight blocks of sixteen rows
// (skinny_wide_tile), which unpack a weight once for all of them.
//
// Arithmetic: code - zero in fp16, fp32 sums per group, and the group's scale applied to the sum in fp32.  Tiles of sixteen rows,
// which decoding uses, of sixteen columns and of 32 by 32 multiply the codes and take the zero from the group's sum in fp32
// (see ZERO_APART).  Sums over the wavefronts in a fixed order.
#include "fq_device.h"
#include "fq_internal.h"

#include <climits>

namespace {

constexpr int SNW = 8; // wavefronts per workgroup, each a slice of K

struct SkinnyJob {
    const uint32_t *packed;
    const _Float16 *scales, *zeros;
    _Float16 *out;
    int N, bits, ld, pad;
};
struct SkinnyJobs {
    SkinnyJob j[3];
};
constexpr int SKINNY_JOBS_AT = 32; // bytes of the kernel's arguments ahead of the jobs: a pointer and six numbers

// The packed dwords of S consecutive sixteen-row sub-blocks of group g, in the order that skinny_chunk expects.  S divides 4
// and the rows of a matrix are padded to 64, so every sub-block exists.  packed: descriptor of the supertile rows from the
// one that holds the first sub-block; part: the first sub-block's place in it.
template <int BITS, int S>
__device__ __forceinline__ void skinny_load(fq_rsrc packed, int part, int G, int g, int lane, uint32_t (&w)[S * BITS])
{
    constexpr int SUB = Fmt<BITS>::SUB, TILE = tile_dwords<BITS>() * 4, PLANES = Fmt<BITS>::PLANES;
    const uint32_t lo = (uint32_t)lane * 16u;
    if constexpr (S >= SUB) { // whole planes: a lane's dwords of a supertile are consecutive over them
#pragma unroll
        for (int t = 0; t < S / SUB; ++t)
#pragma unroll
            for (int p = 0; p < PLANES; ++p) {
                const u4v v = buf_load_b128(packed, lo + 1024u * p, (uint32_t)(t * G + g) * (uint32_t)TILE);
                w[4 * (PLANES * t + p)] = v.x;
                w[4 * (PLANES * t + p) + 1] = v.y;
                w[4 * (PLANES * t + p) + 2] = v.z;
                w[4 * (PLANES * t + p) + 3] = v.w;
            }
    } else if constexpr (BITS == 3 && S == 2) { // dwords 0..5 or 6..11: a whole plane and half of the middle one
        const u4v v = buf_load_b128(packed, lo + (part == 0 ? 0u : 2048u), (uint32_t)g * (uint32_t)TILE);
        const u2v q = buf_load_b64(packed, lo + (part == 0 ? 1024u : 1032u), (uint32_t)g * (uint32_t)TILE);
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
        w[4] = q.x;
        w[5] = q.y;
    } else {
        buf_load_chunk<BITS>(packed, (uint32_t)g * (uint32_t)TILE, part, lane, w);
    }
}

// Sub-block u's dwords.
template <int BITS, int S>
__device__ __forceinline__ void skinny_chunk(const uint32_t (&w)[S * BITS], int part, int u, uint32_t (&C)[BITS])
{
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
        const int at = u * BITS + i;
        if constexpr (BITS == 3 && S == 2)
            C[i] = part == 0 ? w[at] : w[(at + 4) % 6];
        else
            C[i] = w[at];
    }
}

// The four k-steps' operands of a chunk: code - zero in fp16 (see unpack_khalf).
template <int BITS, bool INTZ>
__device__ __forceinline__ void skinny_unpack(const uint32_t (&C)[BITS], h2 zero2, const UnpackConsts<BITS> &uc, h8 (&a)[4])
{
    h8 lo[2], hi[2];
    unpack_khalf<BITS, INTZ, false, 0>(C, zero2, h2{}, uc, lo);
    unpack_khalf<BITS, INTZ, false, 1>(C, zero2, h2{}, uc, hi);
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

// Partial sums of so many blocks of 16 x 16 at a time go through LDS: two for each of the eight wavefronts to add up.
template <int MB, int S>
struct SkinnyRed { static constexpr int N = MB * S < 16 ? MB * S : 16; };

// The sums of the wavefronts, in a fixed order, and the store.
template <int MB, int S>
__device__ __forceinline__ void skinny_store(h8 *smem, const f4 (&acc)[S][MB], int M, int G, const SkinnyJob &job, int m0, int sb0)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, c = lane >> 4;
    // The partial sums take the rings' memory: every wavefront's copies have to land first.
    __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0);
    // block (u, j): lane holds m = 16j + lane%16 and n = 16u + 4*(lane/16) + v; four values at once where every row of
    // the output (a column range of a wider array when ld > N) starts 8-byte aligned
    const bool vec_ok = (job.ld & 3) == 0 && (reinterpret_cast<uintptr_t>(job.out) & 7) == 0;
    const int waves = min(SNW, G);
    constexpr int RED = SkinnyRed<MB, S>::N;
    f4 *red = reinterpret_cast<f4 *>(smem);
    static_for<(MB * S + RED - 1) / RED>([&](auto pass_tag) {
        constexpr int first = decltype(pass_tag)::value * RED, N = MB * S - first < RED ? MB * S - first : RED; // block b = u * MB + j
        __syncthreads();
        static_for<N>([&](auto b_tag) {
            constexpr int b = decltype(b_tag)::value, u = (first + b) / MB, j = (first + b) % MB;
            red[(wave * RED + b) * 64 + lane] = acc[u][j];
        });
        __syncthreads();
        auto store = [&](int b, f4 sum) {
            const int m = m0 + 16 * ((first + b) % MB) + r, n = 16 * (sb0 + (first + b) / MB) + 4 * c;
            if (m >= M)
                return;
            _Float16 *o = job.out + (size_t)m * job.ld + n;
            if (n + 3 < job.N && vec_ok) {
                *reinterpret_cast<h4 *>(o) = h4{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < job.N)
                        o[v] = (_Float16)sum[v];
            }
        };
        auto at_once = [&](int b) { // read one behind the other they took eight times an LDS access
            f4 of[SNW];
#pragma unroll
            for (int v = 0; v < SNW; ++v)
                of[v] = red[(v * RED + b) * 64 + lane];
            f4 sum = of[0];
#pragma unroll
            for (int v = 1; v < SNW; ++v)
                sum += of[v];
            return sum;
        };
        auto in_turn = [&](int b) {
            f4 sum = red[b * 64 + lane];
            for (int v = 1; v < waves; ++v)
                sum += red[(v * RED + b) * 64 + lane];
            return sum;
        };
        // two loops: with the choice inside of one, rows of up to 896 took 1 % longer
        if (waves == SNW) {
            for (int b = wave; b < N; b += SNW)
                store(b, at_once(b));
        } else {
            for (int b = wave; b < N; b += SNW)
                store(b, in_turn(b));
        }
    });
}

// Activation stages of half a group (two k-steps, 128 bytes a row) that a wavefront keeps in LDS.
template <int MB>
struct SkinnyRing { static constexpr int H = MB <= 2 ? 4 : 2, STAGE = 16 * MB * 8; }; // STAGE: 16-byte slots

// A tile of 16*MB rows x 16*S columns: S <= 2, or sixteen rows.
template <int BITS, int MB, int S>
__device__ __forceinline__ void skinny_tile(h8 *smem, const _Float16 *__restrict__ x, int M, int K, const SkinnyJob job,
                                            int tile, int row_tiles)
{
    // Zeros leave through the group's sums, sum code x - zero sum x, so that any fp16 zero is exact, as in the decode kernel
    // (2048 x 2048, 16 rows at 2 bits, error over the rms of the result: 2.06e-4, the output's own rounding; with code - zero
    // in fp16 2.3e-4 for fractional zeros and 4.0e-4 for odd ones beyond 1024).  sum x is one more matrix product, of rows
    // of ones, and there is no branch on the zeros.  Sixteen rows: level in time; 32 x 32 and 32 x 16, which serve what sixteen rows
    // otherwise would: 0.5 and 0.9 % more over 230 sizes; 48 x 16 2.5 %, and so would the others be.
    constexpr bool ZERO_APART = S == 1 || MB <= 2;
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
        uint32_t w[S * BITS];
        h4 sc[S];       // scales of the rows 4c..4c+3, whose sums the lane holds
        uint32_t zr[S]; // zero of the row r, whose weights the lane unpacks
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
                sc[u] = __builtin_bit_cast(h4, buf_load_b64(scales, 8u * (uint32_t)c, at));
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
                uint32_t C[BITS];
                skinny_chunk<BITS, S>(w, sb0 % SUB, u, C);
                UnpackConsts<BITS> uc; // afresh: what the two forms share would be taken out of them, ahead of the branch
                uc.init();
                if constexpr (ZERO_APART) {
                    skinny_unpack<BITS, true>(C, h2{0, 0}, uc, a[u]); // the codes themselves
                    const h4 s4 = row16_bcast<8 * (u & 1)>(meta[u / 2]), z4 = row16_bcast<8 * (u & 1) + 4>(meta[u / 2]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        scf[u][v] = (float)s4[v];
                        zf[u][v] = (float)z4[v];
                    }
                } else {
                    const h2 z2 = as_h2(zr[u] * 0x10001u);
                    const _Float16 z = z2[0];
                    // integer zeros (what the quantizer produces): bias and zero leave in one addition
                    if (__builtin_amdgcn_ballot_w64(z != __builtin_truncf16(z)) == 0)
                        skinny_unpack<BITS, true>(C, z2, uc, a[u]);
                    else
                        skinny_unpack<BITS, false>(C, z2, uc, a[u]);
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        scf[u][v] = (float)sc[u][v];
                }
            });
            load_w(t + 1);
            f4 p[S][MB], xs[MB] = {}; // xs: sums over the group of the lane's activation rows
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
                        for (int j = 0; j < MB; ++j)
                            p[u][j] = mfma16x16x32(a[u][2 * half + s], xf[s][j], (half | s) == 0 ? f4{0.f, 0.f, 0.f, 0.f} : p[u][j]);
                if constexpr (ZERO_APART) {
                    const _Float16 one = 1;
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int j = 0; j < MB; ++j)
                            xs[j] = mfma16x16x32(h8{one, one, one, one, one, one, one, one}, xf[s][j], xs[j]);
                }
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(FQ_WAIT_LGKMCNT0); // the operands have left the slot
                copy(2 * t + half + H);
            }
#pragma unroll
            for (int u = 0; u < S; ++u)
#pragma unroll
                for (int j = 0; j < MB; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[u][j][v] = fmaf(scf[u][v], ZERO_APART ? fmaf(-zf[u][v], xs[j][v], p[u][j][v]) : p[u][j][v], acc[u][j][v]);
        }
    }

    skinny_store<MB, S>(smem, acc, M, G, job, m0, sb0);
}

// A tile of 16*MB rows x 64 columns, MB = 2 .. 8.  An unpacked operand feeds MB products and an activation four, and the largest
// tiles make one round over the chip of what takes two or three of the smaller ones (4096 columns: up to 512 rows; 11008: up
// to 128).  Bound by what the wavefronts issue: 300 x 4096 x 11008 at 2 bits 37 us in tiles of 80 rows, 21 of them without the
// copies, the weight loads, the unpack and the scales (48 rows: 51).  A stage of the ring is sixteen rows of one group, so that it takes the same memory for
// every MB, and the scale is applied to the group's sums in fp32, block by block.
constexpr int WIDE_H = 4, WIDE_STAGE = 256, WIDE_COPIES = 4; // stages, 16-byte slots of one, copies that fill one
constexpr int META_TURNS = 4, META_SLOTS = 16;               // scales and zeros of a turn: 256 bytes

template <int BITS, int MB>
__device__ __forceinline__ void skinny_wide_tile(h8 *smem, const _Float16 *__restrict__ x, int M, int K, const SkinnyJob job,
                                            int tile, int row_tiles)
{
    constexpr int S = 4, H = WIDE_H, STAGE = WIDE_STAGE, COPIES = WIDE_COPIES;
    // Bodies that have registers for the sums and operands but for little else: what follows from the lane is formed where it is used.  Kept
    // over the turns it would spill, and a reload waits for every copy in flight (3 bits, 128 rows: 9 % more time); bodies with room take 3 to 5 %
    // more time this way.
    constexpr bool TIGHT = (BITS == 3 && MB == 8) || (BITS == 4 && MB >= 7);

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, c = lane >> 4;
    const int G = K >> 7;
    const int m0 = (tile % row_tiles) * (16 * MB), sb0 = (tile / row_tiles) * S;
    // descriptors of what the tile reads of the matrix: S sub-blocks of every group
    constexpr int SUB = Fmt<BITS>::SUB, TILE = tile_dwords<BITS>();
    const fq_rsrc packed = make_rsrc(job.packed + (size_t)(sb0 / SUB) * G * TILE, (uint32_t)((S + SUB - 1) / SUB * G) * (TILE * 4u));

    f4 acc[S][MB];
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j)
            acc[u][j] = f4{0.f, 0.f, 0.f, 0.f};

    if (wave < G) { // uniform over the wavefront
        // Copies, global memory straight into the ring: copy i of a stage fills rows 4i .. 4i + 3, slot (row, pos) with
        // chunk pos ^ row of the row's sixteen, so that the operand reads below touch every bank once.  The row is
        // part of the lane offset, which the descriptor's range check covers: rows past M read as zero and are not stored.
        h8 *const ring = smem + wave * (H * STAGE);
        // From the first row of a block: copy i's is 4 i rows further, and 64 i (bits that K * 2, a multiple of 256, leaves clear)
        // exchanged in it.
        uint32_t xoff[TIGHT ? 1 : COPIES];
#pragma unroll
        for (int i = 0; i < (TIGHT ? 1 : COPIES); ++i)
            xoff[i] = ((uint32_t)(4 * i + c) * (uint32_t)K + 8u * (uint32_t)(r ^ c ^ (4 * i))) * 2u;
        const int turns = (G - wave + SNW - 1) / SNW; // groups of this wavefront
        int nt = 0, nj = 0, ns = 0;                   // group, row block and slot of the next copy
        auto copy = [&]() { // past the end: the last group's rows again, into a stage that is not read any more
            const uint32_t off = (uint32_t)(wave + SNW * min(nt, turns - 1)) * 256u;
            // The descriptor starts at the block's first row and ends with the last row of all: scalar work, where block and row in
            // the lane offset were two vector instructions a copy, a tenth of a turn's (300 x 4096 x 11008 at 3 bits 40.0 -> 38.9 us, at 4096 x
            // 4096 17.9 -> 17.7; over 52 sizes 0 to 4 % less, 1.7 on average).
            const int row = m0 + 16 * nj;
            const fq_rsrc xr = make_rsrc(x + (size_t)row * K, row < M ? (uint32_t)(M - row) * (uint32_t)K * 2u : 0u);
            if constexpr (TIGHT)
                asm volatile("" : "+v"(xoff[0]));
            h8 *dst = ring + ns * STAGE;
#pragma unroll
            for (int i = 0; i < COPIES; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, dst + 64 * i, 16, TIGHT ? (xoff[0] ^ (64u * i)) + 8u * i * (uint32_t)K : xoff[TIGHT ? 0 : i],
                                                         off, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            ns = (ns + 1) & (H - 1);
            if (++nj == MB) {
                nj = 0;
                ++nt;
            }
        };
        auto lane_here = [&]() {
            int l = lane;
            if constexpr (TIGHT)
                asm volatile("" : "+v"(l));
            return l;
        };
        uint32_t w[S * BITS];
        // Scales and zeros of the S sub-blocks, one copy of a dword a lane: sub-block u's sixteen scales and sixteen zeros
        // at bytes 64u and 64u + 32 of the turn's slots.
        char *const metas = reinterpret_cast<char *>(smem + SNW * H * STAGE + wave * (META_TURNS * META_SLOTS));
        auto load_w = [&](int t) { // past the end: the last group again (nobody uses it)
            const int g = min(wave + SNW * t, G - 1);
            const int l = lane_here();
            skinny_load<BITS, S>(packed, sb0 % SUB, G, g, l, w);
            const char *const meta_lane = reinterpret_cast<const char *>((l & 8) ? job.zeros : job.scales) +
                                          ((size_t)(sb0 + (l >> 4)) * G * 32 + 4 * (l & 7));
            __builtin_amdgcn_global_load_lds(meta_lane + (size_t)g * 32, metas + (t % META_TURNS) * (META_SLOTS * 16), 4, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        load_w(0);
#pragma unroll
        for (int h = 0; h < H; ++h)
            copy();
        int slot = 0; // of the stage whose operands are read next
        constexpr bool ROOM = MB <= 5; // registers for operands one stage ahead and for the scales
        h8 xf[ROOM ? 2 : 1][4];
        auto read = [&](h8 (&to)[4]) {
            // Loads complete in the order they were issued, and the copies of H - 1 stages are younger than this one's.  The
            // loads of load_w may be among them but are not counted (how many they are is the compiler's affair): the
            // wait then reaches a little further than it has to.
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(vmcnt_at_most(COPIES * (H - 1)));
            __builtin_amdgcn_sched_barrier(0);
            const h8 *stage = ring + slot * STAGE;
            const int l = lane_here(), rd = (l & 15) * 16 + ((l >> 4) ^ (l & 15)); // slot of operand (row r, k-step 0)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                to[s] = stage[rd ^ (4 * s)];
            slot = (slot + 1) & (H - 1);
        };
        for (int t = 0; t < turns; ++t) {
            read(xf[0]);
            // the turn's scales and zeros, issued a turn ago: a turn's copies are younger (at the start, H stages')
            __builtin_amdgcn_s_waitcnt(vmcnt_at_most(COPIES * (MB < H ? MB : H)));
            __builtin_amdgcn_sched_barrier(0);
            const char *const meta = metas + (t % META_TURNS) * (META_SLOTS * 16);
            const int row = lane_here() & 15; // whose weights the lane unpacks
            h8 a[S][4];
            h4 scales[S]; // of the rows 4c..4c+3, whose sums the lane holds
            uint32_t C[S][BITS];
            h2 z2[S];
            bool frac = false;
#pragma unroll
            for (int u = 0; u < S; ++u) {
                skinny_chunk<BITS, S>(w, sb0 % SUB, u, C[u]);
                if constexpr (ROOM)
                    scales[u] = *reinterpret_cast<const h4 *>(meta + 64 * u + 8 * c);
                const _Float16 z = *reinterpret_cast<const _Float16 *>(meta + 64 * u + 32 + 2 * row);
                z2[u] = h2{z, z};
                frac |= z != __builtin_truncf16(z);
            }
            // integer zeros (what the quantizer produces): bias and zero leave in one addition
            if (__builtin_amdgcn_ballot_w64(frac) == 0) {
                UnpackConsts<BITS> uc; // afresh: what the two forms share would be taken out of them, ahead of the branch
                uc.init();
#pragma unroll
                for (int u = 0; u < S; ++u)
                    skinny_unpack<BITS, true>(C[u], z2[u], uc, a[u]);
            } else {
                UnpackConsts<BITS> uc;
                uc.init();
#pragma unroll
                for (int u = 0; u < S; ++u)
                    skinny_unpack<BITS, false>(C[u], z2[u], uc, a[u]);
            }
            load_w(t + 1);
            static_for<MB>([&](auto j_tag) {
                constexpr int j = decltype(j_tag)::value;
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(FQ_WAIT_LGKMCNT0); // the operands have left their stage
                copy();
                if constexpr (ROOM && j + 1 < MB)
                    read(xf[(j + 1) & 1]); // on their way during the products below
                if constexpr (!ROOM) {
                    const int off = 8 * (lane_here() >> 4); // read again: kept over the blocks they would spill
#pragma unroll
                    for (int u = 0; u < S; ++u)
                        scales[u] = *reinterpret_cast<const h4 *>(meta + 64 * u + off);
                }
                f4 p[S];
                __builtin_amdgcn_s_setprio(1); // products ahead of the other wavefront's unpacking
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int u = 0; u < S; ++u)
                        p[u] = mfma16x16x32(a[u][s], xf[ROOM ? j & 1 : 0][s], s == 0 ? f4{0.f, 0.f, 0.f, 0.f} : p[u]);
#pragma unroll
                for (int u = 0; u < S; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[u][j][v] = fmaf((float)scales[u][v], p[u][v], acc[u][j][v]);
                __builtin_amdgcn_s_setprio(0);
                if constexpr (!ROOM && j + 1 < MB)
                    read(xf[0]);
            });
        }
    }

    skinny_store<MB, S>(smem, acc, M, G, job, m0, sb0);
}

// LDS in 16-byte slots: the wavefronts' rings, and later the partial sums.
template <int MB, int S>
constexpr int skinny_slots()
{
    constexpr int ring = SNW * (MB > 1 && S == 4 ? WIDE_H * WIDE_STAGE + META_TURNS * META_SLOTS : SkinnyRing<MB>::H * SkinnyRing<MB>::STAGE);
    constexpr int red = SNW * SkinnyRed<MB, S>::N * 64;
    return ring > red ? ring : red;
}

template <int BITS, int MB, int S>
__device__ __forceinline__ void skinny_any(h8 *smem, const _Float16 *__restrict__ x, int M, int K, const SkinnyJob &job, int tile,
                                           int row_tiles)
{
    if constexpr (MB > 1 && S == 4)
        skinny_wide_tile<BITS, MB>(smem, x, M, K, job, tile, row_tiles);
    else
        skinny_tile<BITS, MB, S>(smem, x, M, K, job, tile, row_tiles);
}

// 8-bit chunks and more than five row blocks are more registers than there are; fq_plan_skinny does not put them together.
constexpr int WIDEST_8BIT = 5;

// The scalars come first: the build has them preloaded into registers at wavefront start, so that which tile, of which matrix, is known
// without a round trip to the argument buffer and one round fetches that matrix's fields.  (Selected by value from all three, with
// nothing preloaded, they took four rounds one after another: 4096 x 4096 at 4 rows and 2 bits 6.0 us against 5.4.)  first1, first2: first tile of the second and
// third matrix, beyond the last tile where there is none.
template <int MB, int S>
__global__ __launch_bounds__(64 * SNW, (MB == 1 && S <= 2) ? 4 : 2) void skinny_kernel(const _Float16 *__restrict__ x, int M, int K, int row_tiles,
                                                                                 int total, int first1, int first2, SkinnyJobs jobs)
{
    __shared__ h8 smem[skinny_slots<MB, S>()]; // the kernel's only LDS object: see the waits in skinny_tile
    // the workgroups of an XCD take a contiguous run of tiles (row-tile fastest): tiles that share weights share an L2
    const int per_xcd = (total + 7) >> 3;
    int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= total)
        return; // uniform over the workgroup, before any barrier
    const int index = (tile >= first1) + (tile >= first2);
    const SkinnyJob job = kernel_argument<SkinnyJobs>(SKINNY_JOBS_AT)->j[index];
    tile -= index == 0 ? 0 : (index == 1 ? first1 : first2);
    switch (job.bits) {
    case 2: skinny_any<2, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    case 3: skinny_any<3, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    case 4: skinny_any<4, MB, S>(smem, x, M, K, job, tile, row_tiles); break;
    default:
        if constexpr (MB <= WIDEST_8BIT)
            skinny_any<8, MB, S>(smem, x, M, K, job, tile, row_tiles);
        break;
    }
}

typedef void (*SkinnyKernel)(const _Float16 *, int, int, int, int, int, int, SkinnyJobs);
static_assert(last_argument_at(SkinnyKernel{}) == SKINNY_JOBS_AT);

constexpr int SKINNY_CUS = 256;

} // namespace

// Tile shape for a launch, by estimated time.  More than sixteen rows, fitted to 900 sizes of 17 to 1400 rows, 200 to 27648
// columns and K = 256 to 13824, every shape that can serve each, and for 16 and 32 columns, sixteen rows and the L2 to 1800 more that go
// down to 40 columns and K = 128: of these the kernel and tile chosen take 1.2 % longer than the best one on average, 40 are more than 3 %
// slower than the tile that the estimate ahead of these took and 9 more than 10 %, most of them calls of 4 to 8 us:
//  - 64 columns, 32 rows and more: 2.2 us, 1.9 + 0.48 MB us a round over the chip (larger sums to add up), 0.6 + 0.4 MB us a
//    turn of eight groups -- unpacking, then the products and the copies of MB blocks (8 bits 0.36 more, 3 bits 0.08).
//  - 16 and 32 columns: 2.3 and 2.7 us, 1.8 us a round, 0.03 + 0.11 S + 0.29 MB + 0.03 S MB us a turn (8 bits 0.21 S, single dwords
//    of 3 bits 0.32 S): moving the activations is what a turn takes.
//  - sixteen rows: as below, 4.2 us (64 columns 4.6) and 0.92 of the turns, 3 bits S = 1 0.6 in the first; the smallest leave room for a second
//    workgroup on a CU.
// (Taken when the partial sums of a block were still read one after another: a round is 0.2 to 0.5 us less now, in every shape.)
// The turns take no less than the activations need to reach an XCD's L2 at 0.9 TB/s: with thirty and more row tiles the tiles
// that an XCD works on share hardly any.  80 rows and more a tile are the choice wherever a round of them takes what would be two of smaller
// ones: 300 x 4096 x 4096 at 4 bits 23.5 -> 17.5 us, 300 x 4096 x 11008 at 2 bits 48 -> 35, 77 x 11008 x 4096 23.6 -> 17.2, 512
// x 4096 x 11008 at 2 bits 60 -> 53; up to 1280 rows, where the sizes end that their times were fitted to: beyond, they are up to a half longer
// (1500 x 4096 x 11008 at 2 bits 184 us, against 155 in the large tiles).  Of 400 sizes of 700 to 4000 rows 9 would be more than 10 % slower
// without that line, and all together 3 % faster: it is a matter for a fit of its own.
//
// Five blocks of short rows (65 to 80 rows, K up to 1024, from 8193 columns on) stay in tiles of sixteen rows, which take any zero
// exactly, where those are expected to be close (18 %): one round of all five blocks is faster (78 x 9284 x 1024 at 2 bits 8.9
// against 10.7 us) but rounds code - zero.  So do launches of 3- and 8-bit matrices within 2 %.
//
// Up to sixteen rows every shape has one row block and the number of sub-blocks is all there is to choose (it does not change
// a sum).  Fitted to 2500 sizes of 64 to 24000 columns with each S: 3.4 us and a turn of 0.13 + 0.28 S us (8 bits 0.37 S;
// 3 bits S = 1 0.7, S = 2 1.2) while every CU has one tile; a second one on some CUs costs nearly a second turn, and from two a
// CU on the time grows with the tiles.  64 columns a tile just beyond one round (20739 x 1664, 4 bits) 11.3 us, 32 columns 9.8.
fq_skinny_plan fq_plan_skinny(int M, const fq_packed_ref *w, int count)
{
    fq_skinny_plan best = {1, 0, 1, 1e30}, sixteen = best; // sixteen: of the tiles of sixteen rows
    const int blocks = (M + 15) / 16, turns = ((w[0].K >> 7) + SNW - 1) / SNW;
    bool eight = false, three = false;
    for (int i = 0; i < count; ++i) {
        eight = eight || w[i].bits == 8;
        three = three || w[i].bits == 3;
    }
    for (int sl = 0; sl < 3; ++sl) {
        const int S = 1 << sl;
        long col_tiles = 0;
        double one_block = 0.0; // us of a turn of a tile of one row block
        for (int i = 0; i < count; ++i) {
            col_tiles += (w[i].N + 16 * S - 1) / (16 * S);
            const double dwords = blocks > 1 && turns == 1 ? 0.6 : 0.2 + 0.5 * S; // 3 bits, where sub-blocks come in single dwords
            const double t = w[i].bits == 3 && (S == 1 || (S == 2 && blocks == 1)) ? dwords : 0.13 + (w[i].bits == 8 ? 0.37 : 0.28) * S;
            one_block = one_block > t ? one_block : t;
        }
        const int largest = S == 1 ? 3 : (S == 2 ? 4 : (M > 1280 ? 4 : (eight ? WIDEST_8BIT : 8)));
        for (int mb = 1; mb <= largest; ++mb) {
            const int row_tiles = (blocks + mb - 1) / mb;
            if ((blocks + row_tiles - 1) / row_tiles != mb)
                continue; // as many row tiles of fewer blocks do
            const double tiles = (double)row_tiles * (double)col_tiles, waves = tiles / SKINNY_CUS;
            const double whole = waves <= 1.0 ? 1.0 : (double)(long)(waves + 0.999);
            double fixed, work;
            if (mb == 1) {
                double factor = 1.0;
                fixed = blocks == 1 ? 3.4 : (S == 4 ? 4.6 : 4.2);
                if (waves > 1.0 && S == 4) {
                    factor = whole;
                    fixed += factor - 1.0;
                } else if (waves > 1.0) {
                    factor = S == 1 ? (waves <= 2.0 ? 2.2 : 1.5 * waves) : (waves <= 2.0 ? 1.9 : (blocks == 1 ? 1.25 : 1.4) * waves);
                    fixed += 0.3 * waves - 0.3;
                }
                work = factor * turns * one_block * (blocks == 1 ? 1.0 : 0.92);
            } else {
                double mean = 0.0, most = 0.0; // us of a turn, over the tiles of the launch
                for (int i = 0; i < count; ++i) {
                    const int bits = w[i].bits;
                    const double t = S == 4 ? 0.6 + 0.4 * mb + (bits == 8 ? 0.36 : (bits == 3 ? 0.08 : 0.0))
                                            : 0.03 + (bits == 8 ? 0.21 : (bits == 3 && S == 1 ? 0.32 : 0.11)) * S + 0.29 * mb + 0.03 * S * mb;
                    mean += t * ((w[i].N + 16 * S - 1) / (16 * S)) / (double)col_tiles;
                    most = most > t ? most : t;
                }
                fixed = S == 4 ? 2.2 + whole * (1.9 + 0.48 * mb) : (S == 1 ? 2.3 : 2.7) + 1.8 * whole;
                work = whole * turns * (whole == 1.0 ? most : mean);
            }
            if (blocks > 1) {
                const double in_xcd = tiles > 8.0 ? tiles / 8.0 : 1.0; // 32 of them at a time, row-tile fastest
                const double rows = 16.0 * mb * (row_tiles < 32 ? (row_tiles < in_xcd ? row_tiles : in_xcd) : (in_xcd < 32.0 ? in_xcd : 32.0));
                const double l2 = (in_xcd > 32.0 ? in_xcd / 32.0 : 1.0) * rows * w[0].K * 2.0 / 0.9e6; // us
                work = work > l2 ? work : l2;
            }
            if (fixed + work < best.us)
                best = {mb, sl, row_tiles, fixed + work};
            if (mb == 1 && fixed + work < sixteen.us)
                sixteen = {mb, sl, row_tiles, fixed + work};
        }
    }
    const bool rounds = best.s_log2 != 0 && best.mb > (best.s_log2 == 1 ? 2 : 1); // code - zero, to fp16
    const double margin = best.mb == 5 && blocks == 5 && turns == 1 ? 1.18 : (eight && three ? 1.02 : 1.0);
    if (rounds && sixteen.us < best.us * margin)
        return sixteen;
    return best;
}

// Whether the kernel's 32-bit byte offsets reach all of a launch's activations and of a tile's weights.
bool fq_skinny_can(int M, int K) { return K <= (1 << 22) && (size_t)M * K * 2 < ((size_t)1 << 32); }

// Whether a launch of up to sixteen rows goes to the skinny kernel (more rows: see fq_plan_gemm): from four rows on,
// three of long rows, where the
// streaming kernel stages one row after another (4096 x 4096, 4 bits: 7.5 against 5.8 us at 4 rows, 17 against 6.0 at 16; at
// one row 4.2 against 6.1; 4096 x 11008 at 3 rows 11.3 against 10), and where that kernel has no room for the rows.  Four
// rows of more columns than one round of the widest tiles covers stay with the streaming kernel unless they are
// short or long ones (19741 x 1792 at 2 bits 9.2 against 11.0 us, and level on average from 1024 to 8192; below, 0.75 of
// its time, above 0.9), three also if they are long (21160 x 8192 at 3 bits 22.6 against 25.2).
bool fq_skinny_pays(int M, const fq_packed_ref *w, int count)
{
    if (!fq_skinny_can(M, w[0].K))
        return false;
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

// Up to three matrices that share the input (same K), in one launch; plan: fq_plan_skinny's for it.
int fq_launch_skinny(const void *x, int M, const fq_packed_ref *w, void *const *outs, int count, const fq_skinny_plan &plan, fq_stream st)
{
    static const SkinnyKernel table[8][3] = {
        {skinny_kernel<1, 1>, skinny_kernel<1, 2>, skinny_kernel<1, 4>},
        {skinny_kernel<2, 1>, skinny_kernel<2, 2>, skinny_kernel<2, 4>},
        {skinny_kernel<3, 1>, skinny_kernel<3, 2>, skinny_kernel<3, 4>},
        {nullptr, skinny_kernel<4, 2>, skinny_kernel<4, 4>},
        {nullptr, nullptr, skinny_kernel<5, 4>},
        {nullptr, nullptr, skinny_kernel<6, 4>},
        {nullptr, nullptr, skinny_kernel<7, 4>},
        {nullptr, nullptr, skinny_kernel<8, 4>},
    };
    SkinnyJobs jobs = {};
    int first[4] = {0, INT_MAX, INT_MAX, INT_MAX}, total = 0;
    for (int i = 0; i < count; ++i) {
        jobs.j[i] = SkinnyJob{static_cast<const uint32_t *>(w[i].packed), static_cast<const _Float16 *>(w[i].scales),
                              static_cast<const _Float16 *>(w[i].zeros), static_cast<_Float16 *>(outs[i]), w[i].N, w[i].bits,
                              w[i].ld ? w[i].ld : w[i].N, 0};
        first[i] = total;
        total += plan.row_tiles * ((w[i].N + (16 << plan.s_log2) - 1) >> (4 + plan.s_log2));
    }
    hipLaunchKernelGGL(table[plan.mb - 1][plan.s_log2], dim3(8 * ((total + 7) / 8)), dim3(64 * SNW), 0, st,
                       static_cast<const _Float16 *>(x), M, w[0].K, plan.row_tiles, total, first[1], first[2], jobs);
    return (int)hipGetLastError();
}
