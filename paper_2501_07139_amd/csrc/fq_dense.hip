// Unquantized fp16 GEMM for many rows: out[M,N] = x[M,K] . W[N,K]^T, the vocabulary head of the
// calibration forward (FlexQuant, arXiv 2501.07139, Algorithm 1, calibrationEval: the logits whose
// token losses give a candidate's perplexity).
//
// Neither operand needs unpacking, so both go through LDS and every workgroup owns a large output tile:
// 256 activation rows x 256 weight rows, 64 k per iteration, 512 threads = 8 wavefronts in a 2 (rows) x
// 4 (weights) grid, each 128 x 64 = 8 x 4 blocks of 16x16x32 fp16 MFMA with fp32 accumulators.  Per 32
// MFMAs a wavefront reads 12 operands from LDS, and a CU fetches 64 KiB per 8.4 MFLOP.  Both tiles are
// copied from global memory straight into a double-buffered LDS tile (128 KiB, one workgroup per CU),
// row-major with the eight 16-byte chunks of a row XOR-swizzled by (row / 2) % 8: the copy writes whole
// rows and the operand reads of sixteen rows by one chunk touch every bank once.  The copy of iteration
// kt+1 is issued before the MFMAs of iteration kt; one barrier per iteration.
//
// Fused loss (the same calibrationEval, logits never stored): instead of writing its 128 x 64 logits a
// wavefront rounds them to fp16, as the stored logits would be, and reduces every row to the pair
// (maximum, sum of exp(logit - maximum)) over its 64 columns; a second small kernel merges a row's pairs
// over the vocabulary and subtracts the label's logit, which the one lane that holds it has set aside.
#include "fq_device.h"
#include "fq_internal.h"
#include "fq_lse.h"

namespace {

constexpr int DT = 256;        // tile rows of either operand
constexpr int DK = 64;         // k per iteration: 8 chunks of 16 bytes per row
constexpr int DSLOTS = DT * 8; // 16-byte slots of one operand tile

__device__ __forceinline__ int dense_slot(int row, int ch) { return row * 8 + (ch ^ ((row >> 1) & 7)); }

// What the fused-loss variant writes instead of logits.
struct LossParts {
    const int32_t *labels; // [M]
    float2 *pairs;         // [M][ceil(N / 64)]: (maximum, sum of exp(logit - maximum)) of 64 columns
    float *label_logit;    // [M]: the label's logit, written only where the label is in range
    // Kernel arguments beyond the preloaded ones would be fetched where they are first used, when the products are done: with the first
    // copies on their way instead, the loss of up to sixteen rows takes 4 to 5 % less (2 x 7284 x 1024 9.7 -> 9.3 us).
    __device__ __forceinline__ void fetch() const { asm volatile("" ::"s"(labels), "s"(pairs), "s"(label_logit)); }
};

template <bool FUSED>
__global__ __launch_bounds__(512, 2) void dense_kernel(const _Float16 *__restrict__ x, int M,
                                                       const _Float16 *__restrict__ W, int N, int K,
                                                       _Float16 *__restrict__ out, LossParts loss)
{
    __shared__ h8 tiles[2][2][DSLOTS]; // [buffer][0: activations, 1: weights]

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    // Workgroups go to the eight XCDs round-robin, each with its own L2: XCD x takes the x-th contiguous
    // run of tiles, ordered in bands of four activation row-tiles (row-tile fastest).
    const int NT = (N + DT - 1) / DT, MT = (M + DT - 1) / DT, total = NT * MT;
    const int per_xcd = (total + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= total)
        return; // uniform over the workgroup, before any barrier
    const int band = tile / (4 * NT), rest = tile - band * 4 * NT, height = min(4, MT - 4 * band);
    const int m0 = (4 * band + rest % height) * DT, n0 = (rest / height) * DT;
    const int KT = K / DK;

    // The i-th copy of a wavefront fills the 64 slots from 64*wave + 512*i of a tile, lane by lane: rows
    // 8*wave + 64*i + lane/8, position lane%8, which holds chunk position ^ (row/2)%8 (the same for every
    // i).  Rows past the end of an operand re-read its last row; their products are never stored.
    const int crow = 8 * wave + (lane >> 3), cch = (lane & 7) ^ ((crow >> 1) & 7);
    uint32_t xoff[4], woff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        xoff[i] = ((uint32_t)min(m0 + crow + 64 * i, M - 1) * (uint32_t)K + (uint32_t)cch * 8u) * 2u;
        woff[i] = ((uint32_t)min(n0 + crow + 64 * i, N - 1) * (uint32_t)K + (uint32_t)cch * 8u) * 2u;
    }
    const fq_rsrc xr = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2u);
    const fq_rsrc wr = make_rsrc(W, (uint32_t)N * (uint32_t)K * 2u);

    auto copy_tiles = [&](int buffer, int kt) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, &tiles[buffer][0][64 * wave + 512 * i], 16, xoff[i],
                                                     (uint32_t)kt * (DK * 2u), 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, &tiles[buffer][1][64 * wave + 512 * i], 16, woff[i],
                                                     (uint32_t)kt * (DK * 2u), 0, 0);
    };

    f4 acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
            acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    copy_tiles(0, 0);
    __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0);
    __syncthreads();

    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < KT)
            copy_tiles(cur ^ 1, kt + 1);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int ch = 4 * s + (lane >> 4);
            h8 a[4], b[8];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[i] = tiles[cur][1][dense_slot(64 * wn + 16 * i + (lane & 15), ch)];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                b[j] = tiles[cur][0][dense_slot(128 * wm + 16 * j + (lane & 15), ch)];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    acc[i][j] = mfma16x16x32(a[i], b[j], acc[i][j]);
        }
        __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0); // this wavefront's copies have landed ...
        __syncthreads();                            // ... and everyone's, and all reads of `cur` are done
    }

    // lane holds m = lane%16 and n = 4*(lane/16) + v of each 16x16 block
    if constexpr (FUSED) {
        const int nw = n0 + 64 * wn, NC = (N + 63) >> 6;
        if (nw >= N)
            return; // no column of this wavefront exists (after the last barrier)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int m = m0 + 128 * wm + 16 * j + (lane & 15);
            const int label = m < M ? loss.labels[m] : -1;
            float l[16], mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int n = nw + 16 * i + 4 * (lane >> 4) + v;
                    const float logit = (float)(_Float16)acc[i][j][v]; // what the stored fp16 logit would hold
                    l[4 * i + v] = n < N ? logit : -INFINITY;
                    mx = fmaxf(mx, l[4 * i + v]);
                    if (n == label)
                        loss.label_logit[m] = logit;
                }
            float se = 0.f;
            if (mx != -INFINITY) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    se += __expf(l[e] - mx);
            }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) { // the four lanes that share a row
                const float m2 = __shfl_xor(mx, o, 64), s2 = __shfl_xor(se, o, 64);
                lse_merge(mx, se, m2, s2);
            }
            if (lane < 16 && m < M)
                loss.pairs[(size_t)m * NC + (nw >> 6)] = make_float2(mx, se);
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int m = m0 + 128 * wm + 16 * j + (lane & 15);
        if (m >= M)
            continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = n0 + 64 * wn + 16 * i + 4 * (lane >> 4);
            _Float16 *o = out + (size_t)m * N + n;
            if (n + 3 < N && (N & 3) == 0) {
                h4 v = {(_Float16)acc[i][j][0], (_Float16)acc[i][j][1], (_Float16)acc[i][j][2], (_Float16)acc[i][j][3]};
                *reinterpret_cast<h4 *>(o) = v;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < N)
                        o[v] = (_Float16)acc[i][j][v];
            }
        }
    }
}

// ------------------------------------------------------------------ few rows
// 16*MB activation rows x 128 weight rows per workgroup of eight wavefronts, for a handful of tokens: the logits of a
// decode step or of a short prompt.  The weights are read once and that read is the bound (32000 x 4096: 262 MB, 51 us at
// the rate of a large copy), so the tile is narrow enough for one workgroup on every CU (32000 rows: 250) and LDS is a ring
// of D stages of 64 k that keeps 70 to 110 KiB a CU under way: the copies of stage kt + D - 1 go out when stage kt is
// multiplied, and a wavefront waits, by count, for the oldest of its own stages only.  One barrier a stage: behind it
// every wavefront's copies of the stage have landed and nobody reads the slot that the next copies fill.  Wavefronts are
// a WM x 8/WM grid over the tile; above 32 rows two by four, which reads fewer operands per product from LDS.
// Measured: 32000 x 4096 in 54 us at 1 to 32 rows (4.9 TB/s); see dense_plan.
constexpr int RW = 128; // weight rows of a tile

template <int MB>
struct RowsTile {
    static constexpr int WM = MB >= 4 ? 2 : 1;                                   // wavefronts along the activation rows
    static constexpr int XB = MB / WM, WB = WM;                                  // 16-row blocks of a wavefront: activations, weights
    static constexpr int STAGE = (RW + 16 * MB) * 8;                             // 16-byte slots: weights, then activations
    static constexpr int D = MB >= 8 ? 4 : (MB >= 6 ? 5 : (MB >= 4 ? 6 : 7));     // 126 to 144 KiB
    static constexpr int COPIES = 2 + MB / 4;                                    // copies every wavefront issues a stage (the first ones up to one more)
};

template <int MB, bool FUSED>
__device__ __forceinline__ void dense_rows_tile(h8 *smem, const _Float16 *__restrict__ x, int M, const _Float16 *__restrict__ W,
                                                int N, int K, _Float16 *__restrict__ out, const LossParts loss)
{
    using T = RowsTile<MB>;
    constexpr int D = T::D, XB = T::XB, WB = T::WB;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % T::WM, wn = wave / T::WM;
    // the workgroups of an XCD take a contiguous run of tiles, row-tile fastest: weights shared by row tiles come from its L2
    const int NT = (N + RW - 1) / RW, MT = (M + 16 * MB - 1) / (16 * MB), total = NT * MT;
    const int per_xcd = (total + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= total)
        return; // uniform over the workgroup, before any barrier
    const int m0 = (tile % MT) * 16 * MB, n0 = (tile / MT) * RW;
    const int KT = K / DK;

    // Copy i of an operand fills rows 8i .. 8i + 7 of its part of a stage, slot (row, pos) with chunk pos ^ (row/2)%8;
    // the wavefronts take the copies in turn.  Rows past the end of an operand re-read its last row.
    const fq_rsrc xr = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2u);
    const fq_rsrc wr = make_rsrc(W, (uint32_t)N * (uint32_t)K * 2u);
    constexpr int XC = (2 * MB + 7) / 8; // copies of the activations a wavefront issues at most
    uint32_t woff[2], xoff[XC];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = 8 * (wave + 8 * i) + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
        woff[i] = ((uint32_t)min(n0 + row, N - 1) * (uint32_t)K + (uint32_t)ch * 8u) * 2u;
    }
#pragma unroll
    for (int i = 0; i < XC; ++i) {
        const int row = 8 * (wave + 8 * i) + (lane >> 3), ch = (lane & 7) ^ ((row >> 1) & 7);
        xoff[i] = ((uint32_t)min(m0 + row, M - 1) * (uint32_t)K + (uint32_t)ch * 8u) * 2u;
    }
    auto copy_stage = [&](int kt, int slot) { // past the end: the last stage again, into a slot that is not read any more
        h8 *const dst = smem + slot * T::STAGE;
        const uint32_t off = (uint32_t)min(kt, KT - 1) * (DK * 2u);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, dst + 64 * (wave + 8 * i), 16, woff[i], off, 0, 0);
#pragma unroll
        for (int i = 0; i < XC; ++i)
            if (wave + 8 * i < 2 * MB) // uniform over the wavefront
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, dst + RW * 8 + 64 * (wave + 8 * i), 16, xoff[i], off, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    f4 acc[WB][XB];
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < XB; ++j)
            acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int kt = 0; kt < D - 1; ++kt)
        copy_stage(kt, kt);
    if constexpr (FUSED)
        loss.fetch();
    for (int kt = 0, slot = 0; kt < KT; ++kt, slot = slot == D - 1 ? 0 : slot + 1) {
        // at least COPIES * (D - 2) copies are younger than this stage's
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_at_most(T::COPIES * (D - 2)));
        lds_barrier(); // LDS accesses only: the copies stay in flight
        __builtin_amdgcn_sched_barrier(0);
        copy_stage(kt + D - 1, slot == 0 ? D - 1 : slot - 1);
        const h8 *const stage = smem + slot * T::STAGE;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int ch = 4 * s + (lane >> 4);
            h8 a[WB], b[XB];
#pragma unroll
            for (int i = 0; i < WB; ++i)
                a[i] = stage[dense_slot(16 * (WB * wn + i) + (lane & 15), ch)];
#pragma unroll
            for (int j = 0; j < XB; ++j)
                b[j] = stage[RW * 8 + dense_slot(16 * (XB * wm + j) + (lane & 15), ch)];
#pragma unroll
            for (int i = 0; i < WB; ++i)
#pragma unroll
                for (int j = 0; j < XB; ++j)
                    acc[i][j] = mfma16x16x32(a[i], b[j], acc[i][j]);
        }
    }
    __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0); // copies past the end have landed ...
    __syncthreads();                            // ... in every wavefront, and nobody reads a stage any more

    // lane holds m = lane%16 and n = 4*(lane/16) + v of each 16x16 block
    const int nw = n0 + 16 * WB * wn;
    if constexpr (FUSED) {
        float2 *part = reinterpret_cast<float2 *>(smem); // [16 * MB rows][8 / WM column groups]
        constexpr int CG = 8 / T::WM;
#pragma unroll
        for (int j = 0; j < XB; ++j) {
            const int row = 16 * (XB * wm + j) + (lane & 15), m = m0 + row;
            const int label = m < M ? loss.labels[m] : -1;
            float l[4 * WB], mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < WB; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int n = nw + 16 * i + 4 * (lane >> 4) + v;
                    const float logit = (float)(_Float16)acc[i][j][v]; // what the stored fp16 logit would hold
                    l[4 * i + v] = n < N ? logit : -INFINITY;
                    mx = fmaxf(mx, l[4 * i + v]);
                    if (n == label)
                        loss.label_logit[m] = logit;
                }
            float se = 0.f;
            if (mx != -INFINITY) {
#pragma unroll
                for (int e = 0; e < 4 * WB; ++e)
                    se += __expf(l[e] - mx);
            } else { // no number among the lane's few columns: a NaN has to reach the row's sum all the same
#pragma unroll
                for (int e = 0; e < 4 * WB; ++e)
                    if (l[e] != l[e]) {
                        mx = -3.0e38f;
                        se = l[e];
                    }
            }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) { // the four lanes that share a row
                const float m2 = __shfl_xor(mx, o, 64), s2 = __shfl_xor(se, o, 64);
                lse_merge(mx, se, m2, s2);
            }
            if (lane < 16)
                part[row * CG + wn] = make_float2(mx, se);
        }
        __syncthreads();
        // one pair per row and 64 columns, as the 256-row tiles leave them
        const int NC = (N + 63) >> 6;
        for (int e = tid; e < 16 * MB * 2; e += 512) {
            const int row = e >> 1, half = e & 1, m = m0 + row, c64 = (n0 >> 6) + half;
            if (m >= M || c64 >= NC)
                continue;
            float2 p = part[row * CG + half * (CG / 2)];
#pragma unroll
            for (int g = 1; g < CG / 2; ++g) {
                const float2 q = part[row * CG + half * (CG / 2) + g];
                lse_merge(p.x, p.y, q.x, q.y);
            }
            loss.pairs[(size_t)m * NC + c64] = p;
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < XB; ++j) {
        const int m = m0 + 16 * (XB * wm + j) + (lane & 15);
        if (m >= M)
            continue;
#pragma unroll
        for (int i = 0; i < WB; ++i) {
            const int n = nw + 16 * i + 4 * (lane >> 4);
            _Float16 *o = out + (size_t)m * N + n;
            if (n + 3 < N && (N & 3) == 0) {
                h4 v = {(_Float16)acc[i][j][0], (_Float16)acc[i][j][1], (_Float16)acc[i][j][2], (_Float16)acc[i][j][3]};
                *reinterpret_cast<h4 *>(o) = v;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < N)
                        o[v] = (_Float16)acc[i][j][v];
            }
        }
    }
}

template <int MB, bool FUSED>
__global__ __launch_bounds__(512, 2) void dense_rows_kernel(const _Float16 *__restrict__ x, int M,
                                                            const _Float16 *__restrict__ W, int N, int K,
                                                            _Float16 *__restrict__ out, LossParts loss)
{
    __shared__ h8 smem[RowsTile<MB>::D * RowsTile<MB>::STAGE]; // the only LDS object: the compiler adds no waits for the copies in flight
    dense_rows_tile<MB, FUSED>(smem, x, M, W, N, K, out, loss);
}

typedef void (*RowsKernel)(const _Float16 *, int, const _Float16 *, int, int, _Float16 *, LossParts);

int launch_rows(bool fused, int mb, const void *x, int M, const void *W, int N, int K, void *out, const LossParts &loss, fq_stream st)
{
    static const RowsKernel table[2][5] = {
        {dense_rows_kernel<1, false>, dense_rows_kernel<2, false>, dense_rows_kernel<4, false>, dense_rows_kernel<6, false>, dense_rows_kernel<8, false>},
        {dense_rows_kernel<1, true>, dense_rows_kernel<2, true>, dense_rows_kernel<4, true>, dense_rows_kernel<6, true>, dense_rows_kernel<8, true>},
    };
    const int total = ((N + RW - 1) / RW) * ((M + 16 * mb - 1) / (16 * mb));
    hipLaunchKernelGGL(table[fused][mb <= 2 ? mb - 1 : mb / 2], dim3(8 * ((total + 7) / 8)), dim3(512), 0, st, static_cast<const _Float16 *>(x), M,
                       static_cast<const _Float16 *>(W), N, K, static_cast<_Float16 *>(out), loss);
    return (int)hipGetLastError();
}

// --------------------------------------------------- few rows, few columns
// 16*MB activation rows x 16*S weight rows per workgroup whose eight wavefronts share K, for products whose tiles of 128 and 256
// would leave CUs idle (100 rows of 4000 x 4096: 32 tiles of 128 x 128).  Wavefront w takes the groups of 128 k w, w + 8, ...;
// sixteen rows of either operand over one group are a stage (4 KiB) of a ring in LDS that is the wavefront's own, filled by
// direct copies: the S stages of the weights, then the MB stages of the activations, one after the other, so there is no barrier in
// the loop and a wavefront waits, by count, for its oldest stage only.  Partial sums meet in LDS, in a fixed order.
// Bound by latency, of the first stages and of the sums at the end, more than by the way from L2 into LDS that both operands of every tile
// take (26 to 33 TB/s over the chip by itself): 100 x 4000 x 4096 is 250 tiles of 64 x 32, 197 MB in 13.6 us with the launch, 14 TB/s (2.5
// times as fast as tiles of 128 x 128).
constexpr int SPLIT_NW = 8, SPLIT_H = 4, SPLIT_STAGE = 256, SPLIT_COPIES = 4; // wavefronts; stages, 16-byte slots of one, copies that fill one

template <int MB, int S, bool FUSED>
__device__ __forceinline__ void dense_split_tile(h8 *smem, const _Float16 *__restrict__ x, int M, const _Float16 *__restrict__ W,
                                                 int N, int K, _Float16 *__restrict__ out, const LossParts loss, int m0, int n0)
{
    constexpr int H = SPLIT_H, P = S + MB; // stages of a group
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, c = lane >> 4;
    const int G = K >> 7;

    f4 acc[S][MB];
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
        for (int j = 0; j < MB; ++j)
            acc[u][j] = f4{0.f, 0.f, 0.f, 0.f};

    if (wave < G) { // uniform over the wavefront
        // Copy i of a stage fills rows 4i .. 4i + 3, slot (row, pos) with chunk pos ^ row of the row's sixteen.  The row is part of the
        // lane offset, which the descriptor's range check covers: rows past the end of an operand read as zero.
        h8 *const ring = smem + wave * (H * SPLIT_STAGE);
        const fq_rsrc xr = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2u), wr = make_rsrc(W, (uint32_t)N * (uint32_t)K * 2u);
        uint32_t off[SPLIT_COPIES]; // from row 0 of an operand
#pragma unroll
        for (int i = 0; i < SPLIT_COPIES; ++i) {
            const int row = 4 * i + c;
            off[i] = ((uint32_t)row * (uint32_t)K + 8u * (uint32_t)(r ^ row)) * 2u;
        }
        const int turns = (G - wave + SPLIT_NW - 1) / SPLIT_NW; // groups of this wavefront
        int nt = 0, np = 0, ns = 0;                             // group, part of it and slot of the next copy
        auto copy = [&]() { // past the end: the last group again, into a stage that is not read any more
            const uint32_t at = (uint32_t)(wave + SPLIT_NW * min(nt, turns - 1)) * 256u;
            h8 *dst = ring + ns * SPLIT_STAGE;
            uint32_t down = (uint32_t)(np < S ? n0 + 16 * np : m0 + 16 * (np - S)) * ((uint32_t)K * 2u);
            asm volatile("" : "+s"(down)); // added here: the sums of all blocks would be kept in registers
            if (np < S) {
#pragma unroll
                for (int i = 0; i < SPLIT_COPIES; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, dst + 64 * i, 16, off[i] + down, at, 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < SPLIT_COPIES; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, dst + 64 * i, 16, off[i] + down, at, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            ns = (ns + 1) & (H - 1);
            if (++np == P) {
                np = 0;
                ++nt;
            }
        };
#pragma unroll
        for (int h = 0; h < H; ++h)
            copy();
        if constexpr (FUSED)
            loss.fetch();
        int rd[4]; // slot of operand (row r, k-step s) in a stage
#pragma unroll
        for (int s = 0; s < 4; ++s)
            rd[s] = r * 16 + ((4 * s + c) ^ r);
        int slot = 0; // of the stage whose operands are read next
        auto read = [&](h8 (&to)[4]) { // exactly the copies of H - 1 stages are younger than this one's
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(vmcnt_at_most(SPLIT_COPIES * (H - 1)));
            __builtin_amdgcn_sched_barrier(0);
            const h8 *stage = ring + slot * SPLIT_STAGE;
#pragma unroll
            for (int s = 0; s < 4; ++s)
                to[s] = stage[rd[s]];
            slot = (slot + 1) & (H - 1);
        };
        auto refill = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(FQ_WAIT_LGKMCNT0); // the operands have left their stage
            copy();
        };
        h8 a[S][4], b[2][4];
        for (int t = 0; t < turns; ++t) {
            read(a[0]);
            static_for<S>([&](auto u_tag) {
                constexpr int u = decltype(u_tag)::value;
                refill();
                if constexpr (u + 1 < S)
                    read(a[u + 1]);
                else
                    read(b[0]);
            });
            static_for<MB>([&](auto j_tag) {
                constexpr int j = decltype(j_tag)::value;
                refill();
                if constexpr (j + 1 < MB)
                    read(b[(j + 1) & 1]); // on their way during the products below
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int u = 0; u < S; ++u)
                        acc[u][j] = mfma16x16x32(a[u][s], b[j & 1][s], acc[u][j]);
                __builtin_amdgcn_s_setprio(0);
            });
        }
    }

    // The partial sums take the rings' memory, JP row blocks at a time: every wavefront's copies have to land first.
    __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0);
    constexpr int JP = MB * S <= 16 ? MB : 16 / S, PASSES = (MB + JP - 1) / JP, BLOCKS = JP * S;
    f4 *red = reinterpret_cast<f4 *>(smem);
    auto total = [&](int b) { // of block b of the pass: lane holds m = lane%16 and n = 4*(lane/16) + v
        f4 part[SPLIT_NW]; // of all wavefronts, zeros of those without a group: read at once, one after another took the loss of one row block 0.7 us
#pragma unroll
        for (int v = 0; v < SPLIT_NW; ++v)
            part[v] = red[(v * BLOCKS + b) * 64 + lane];
        f4 sum = part[0];
#pragma unroll
        for (int v = 1; v < SPLIT_NW; ++v)
            sum += part[v];
        return sum;
    };
    static_for<PASSES>([&](auto pass_tag) {
        constexpr int first = decltype(pass_tag)::value * JP, count = first + JP <= MB ? JP : MB - first;
        __syncthreads();
        static_for<count>([&](auto j_tag) {
            constexpr int j = decltype(j_tag)::value;
#pragma unroll
            for (int u = 0; u < S; ++u)
                red[(wave * BLOCKS + j * S + u) * 64 + lane] = acc[u][first + j];
        });
        __syncthreads();
        if constexpr (FUSED) {
            static_assert(!FUSED || S == 4, "a pair is 64 columns");
            const int NC = (N + 63) >> 6;
            for (int j = wave; j < count; j += SPLIT_NW) {
                const int m = m0 + 16 * (first + j) + r, label = m < M ? loss.labels[m] : -1;
                float l[4 * S], mx = -INFINITY;
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    const f4 sum = total(j * S + u);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int n = n0 + 16 * u + 4 * c + v;
                        const float logit = (float)(_Float16)sum[v]; // what the stored fp16 logit would hold
                        l[4 * u + v] = n < N ? logit : -INFINITY;
                        mx = fmaxf(mx, l[4 * u + v]);
                        if (n == label)
                            loss.label_logit[m] = logit;
                    }
                }
                float se = 0.f;
                if (mx != -INFINITY) {
#pragma unroll
                    for (int e = 0; e < 4 * S; ++e)
                        se += __expf(l[e] - mx);
                } else { // no number among the lane's columns: a NaN has to reach the row's sum all the same
#pragma unroll
                    for (int e = 0; e < 4 * S; ++e)
                        if (l[e] != l[e]) {
                            mx = -3.0e38f;
                            se = l[e];
                        }
                }
#pragma unroll
                for (int o = 16; o <= 32; o <<= 1) { // the four lanes that share a row
                    const float m2 = __shfl_xor(mx, o, 64), s2 = __shfl_xor(se, o, 64);
                    lse_merge(mx, se, m2, s2);
                }
                if (lane < 16 && m < M)
                    loss.pairs[(size_t)m * NC + (n0 >> 6)] = make_float2(mx, se);
            }
        } else {
            for (int b = wave; b < count * S; b += SPLIT_NW) {
                const f4 sum = total(b);
                const int m = m0 + 16 * (first + b / S) + r, n = n0 + 16 * (b % S) + 4 * c;
                if (m >= M)
                    continue;
                _Float16 *o = out + (size_t)m * N + n;
                if (n + 3 < N && (N & 3) == 0) {
                    *reinterpret_cast<h4 *>(o) = h4{(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (n + v < N)
                            o[v] = (_Float16)sum[v];
                }
            }
        }
    });
}

template <int MB, int S, bool FUSED>
__global__ __launch_bounds__(64 * SPLIT_NW, 2) void dense_split_kernel(const _Float16 *__restrict__ x, int M, const _Float16 *__restrict__ W,
                                                                       int N, int K, _Float16 *__restrict__ out, LossParts loss)
{
    // the kernel's only LDS object (see dense_rows_kernel): the rings, later the sums of at most sixteen blocks
    __shared__ h8 smem[SPLIT_NW * SPLIT_H * SPLIT_STAGE];
    static_assert(SPLIT_H * SPLIT_STAGE >= 16 * 64);
    // the workgroups of an XCD take a contiguous run of tiles, row-tile fastest: weights shared by row tiles come from its L2
    const int NT = (N + 16 * S - 1) / (16 * S), MT = (M + 16 * MB - 1) / (16 * MB), total = NT * MT;
    const int per_xcd = (total + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile >= total)
        return; // uniform over the workgroup, before any barrier
    dense_split_tile<MB, S, FUSED>(smem, x, M, W, N, K, out, loss, (tile % MT) * 16 * MB, (tile / MT) * 16 * S);
}

template <bool FUSED, int S, int... MB>
RowsKernel split_kernel(int mb, std::integer_sequence<int, MB...>)
{
    static const RowsKernel table[] = {dense_split_kernel<MB + 1, S, FUSED>...};
    return table[mb - 1];
}

// Row blocks of a tile of 16, 32 and 64 columns; the loss has the last.
constexpr int SPLIT_MB1 = 3, SPLIT_MB2 = 5, SPLIT_MB4 = 8;

int launch_split(bool fused, int mb, int s, const void *x, int M, const void *W, int N, int K, void *out, const LossParts &loss, fq_stream st)
{
    using std::make_integer_sequence;
    const RowsKernel kernel = fused    ? split_kernel<true, 4>(mb, make_integer_sequence<int, SPLIT_MB4>{})
                              : s == 1 ? split_kernel<false, 1>(mb, make_integer_sequence<int, SPLIT_MB1>{})
                              : s == 2 ? split_kernel<false, 2>(mb, make_integer_sequence<int, SPLIT_MB2>{})
                                       : split_kernel<false, 4>(mb, make_integer_sequence<int, SPLIT_MB4>{});
    const int total = ((M + 16 * mb - 1) / (16 * mb)) * ((N + 16 * s - 1) / (16 * s));
    hipLaunchKernelGGL(kernel, dim3(8 * ((total + 7) / 8)), dim3(64 * SPLIT_NW), 0, st, static_cast<const _Float16 *>(x), M,
                       static_cast<const _Float16 *>(W), N, K, static_cast<_Float16 *>(out), loss);
    return (int)hipGetLastError();
}

// One wavefront per row: merge the row's pairs, then nll = log(sum of exp) - label's logit; a label outside
// [0, V) gives 0, as in the unfused loss.
__global__ __launch_bounds__(64) void loss_finish_kernel(LossParts loss, int V, float *__restrict__ nll)
{
    const int row = blockIdx.x, lane = threadIdx.x, NC = (V + 63) >> 6;
    const int label = loss.labels[row];
    if (label < 0 || label >= V) { // uniform across the wavefront
        if (lane == 0)
            nll[row] = 0.f;
        return;
    }
    float mx = -INFINITY, se = 0.f;
    for (int c = lane; c < NC; c += 64) {
        const float2 p = loss.pairs[(size_t)row * NC + c];
        lse_merge(mx, se, p.x, p.y);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(mx, o, 64), s2 = __shfl_xor(se, o, 64);
        lse_merge(mx, se, m2, s2);
    }
    if (lane == 0)
        nll[row] = logf(se) + (mx - loss.label_logit[row]); // difference first: exact for fp16 inputs
}

} // namespace

// Kernel and tile by estimated time, fitted to 420 sizes of 1 to 1500 rows, 1000 to 50000 columns, K = 256 to 6144, half of them
// with the loss (half the times within 7 %; the choice takes 3 % longer than the best one on average, the spread of two runs
// included).  All three go by rounds over the chip, one tile a CU:
//  - shared K: 2.4 us, 2.1 + 0.16 MB S us a round and 0.38 S + 0.31 MB + 0.02 S MB us a turn of eight groups: the stages that it copies;
//  - streamed weights, 128 columns: 1.1 us, 3.7 us a round and 0.16 / 0.25 / 0.33 / 0.51 / 0.6 us a stage of 64 k for 16 / 32 / 64 / 96 / 128 rows;
//  - 256 x 256 tiles: 1.3 us, 6.7 us a round and 1.58 us a stage of 64 k;
// and none is faster than the weights come from memory, 4.75 TB/s and 2 us.  Measured (us; the best of the other two against shared K): 100 x 4000 x
// 4096 35.6 and 14.0, with the loss 38.3 and 18.0; 1 x 4000 x 4096 14.8 and 8.6; 350 x 4000 x 4096 36.6 and 21.5; 100 x 8000 x 4096 36.0
// and 19.8; 512 x 8000 x 4096 41.5 either way.  180 x 32000 x 4096, two row tiles of 128 rows 87.3, of 96 rows 81.8.
namespace {

enum DenseKind { DENSE_LARGE, DENSE_ROWS, DENSE_SPLIT }; // FQ_DENSE_* of fq.h
struct DensePlan {
    DenseKind kind;
    int rows, columns; // of a tile
    double us;
};

DensePlan dense_plan(int M, int N, int K, bool fused)
{
    const int blocks = (M + 15) / 16, turns = ((K >> 7) + SPLIT_NW - 1) / SPLIT_NW;
    const double stages = K / DK;
    const double memory = 2.0 + (double)N * K * 2.0 / 4.75e6;
    auto consider = [&](DensePlan &best, DenseKind kind, int rows, int columns, double fixed, double round) {
        const double tiles = (double)((M + rows - 1) / rows) * ((N + columns - 1) / columns);
        const double us = fixed + (double)(long)(tiles / 256.0 + 0.999) * round;
        if ((us > memory ? us : memory) < best.us)
            best = {kind, rows, columns, us > memory ? us : memory};
    };
    DensePlan whole = {DENSE_LARGE, DT, DT, 1e30}, narrow = whole, wide = whole; // K in one piece; shared, 16 or 32 columns; shared, 64
    static const int heights[5] = {1, 2, 4, 6, 8};
    static const double stage_us[5] = {0.16, 0.25, 0.33, 0.51, 0.6};
    for (int i = 0; i < 5; ++i) // one row tile of the least height, or several of 96 or 128 rows
        if (blocks > 8 ? i >= 3 : (heights[i] >= blocks && (i == 0 || heights[i - 1] < blocks)))
            consider(whole, DENSE_ROWS, 16 * heights[i], RW, 1.1, 3.7 + stages * stage_us[i]);
    consider(whole, DENSE_LARGE, DT, DT, 1.3, 6.7 + stages * 1.58);
    for (int S = 1; S <= 4; S *= 2)
        for (int mb = 1; mb <= (S == 1 ? SPLIT_MB1 : (S == 2 ? SPLIT_MB2 : SPLIT_MB4)); ++mb) {
            const int row_tiles = (blocks + mb - 1) / mb;
            if ((blocks + row_tiles - 1) / row_tiles == mb) // else as many row tiles of fewer blocks do
                consider(S == 4 ? wide : narrow, DENSE_SPLIT, 16 * mb, 16 * S, 2.4,
                         2.1 + 0.16 * mb * S + turns * (0.38 * S + 0.31 * mb + 0.02 * S * mb));
        }
    // The loss, a pair of which is 64 columns, shares K exactly where the logits do, so that both round the same sums: sharing K
    // changes their order.
    const DensePlan best = narrow.us < wide.us ? narrow : wide;
    if (best.us > 0.88 * whole.us || wide.us > 1.2 * whole.us) // closer than that either may be the faster one
        return whole;
    return fused ? wide : best;
}

int launch_few(const DensePlan &p, bool fused, const void *x, int M, const void *W, int N, int K, void *out, const LossParts &loss, fq_stream st)
{
    if (p.kind == DENSE_ROWS)
        return launch_rows(fused, p.rows / 16, x, M, W, N, K, out, loss, st);
    return launch_split(fused, p.rows / 16, p.columns / 16, x, M, W, N, K, out, loss, st);
}

} // namespace

void fq_dense_plan(int M, int N, int K, bool fused, int *kind, int *rows, int *columns)
{
    const DensePlan plan = dense_plan(M, N, K, fused);
    *kind = plan.kind;
    *rows = plan.rows;
    *columns = plan.columns;
}

int fq_launch_dense_planned(const void *x, int M, const void *W, int N, int K, void *out, fq_stream st)
{
    const DensePlan plan = dense_plan(M, N, K, false);
    return plan.kind == DENSE_LARGE ? fq_launch_dense_tiled(x, M, W, N, K, out, st)
                                    : launch_few(plan, false, x, M, W, N, K, out, LossParts{}, st);
}

// x and W are addressed through 32-bit byte offsets (checked by the caller); K is a multiple of 128.
int fq_launch_dense_tiled(const void *x, int M, const void *W, int N, int K, void *out, fq_stream st)
{
    const int total = ((N + DT - 1) / DT) * ((M + DT - 1) / DT);
    dim3 grid(8 * ((total + 7) / 8)), block(512);
    hipLaunchKernelGGL(dense_kernel<false>, grid, block, 0, st, static_cast<const _Float16 *>(x), M,
                       static_cast<const _Float16 *>(W), N, K, static_cast<_Float16 *>(out), LossParts{});
    return (int)hipGetLastError();
}

size_t fq_head_nll_scratch_bytes(int M, int V)
{
    const size_t pairs = (size_t)M * ((V + 63) / 64) * sizeof(float2);
    return pairs + (size_t)M * sizeof(float);
}

// workspace: fq_head_nll_scratch_bytes(M, V) bytes, 8-byte aligned.
int fq_launch_head_nll(const void *x, int M, const void *W, int V, int K, const int32_t *labels, float *nll,
                       void *workspace, fq_stream st)
{
    LossParts loss;
    loss.labels = labels;
    loss.pairs = static_cast<float2 *>(workspace);
    loss.label_logit = reinterpret_cast<float *>(loss.pairs + (size_t)M * ((V + 63) / 64));
    int rc = 0;
    const DensePlan plan = dense_plan(M, V, K, true);
    if (plan.kind != DENSE_LARGE) {
        rc = launch_few(plan, true, x, M, W, V, K, nullptr, loss, st);
    } else {
        const int total = ((V + DT - 1) / DT) * ((M + DT - 1) / DT);
        dim3 grid(8 * ((total + 7) / 8)), block(512);
        hipLaunchKernelGGL(dense_kernel<true>, grid, block, 0, st, static_cast<const _Float16 *>(x), M,
                           static_cast<const _Float16 *>(W), V, K, static_cast<_Float16 *>(nullptr), loss);
        rc = (int)hipGetLastError();
    }
    if (rc != 0)
        return rc;
    hipLaunchKernelGGL(loss_finish_kernel, dim3(M), dim3(64), 0, st, loss, V, nll);
    return (int)hipGetLastError();
}
