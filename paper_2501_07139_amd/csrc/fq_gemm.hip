// Calibration-forward path: dequant-GEMM for many rows of activations, and the
// unquantized fp16 head GEMM.
//
// Scoring one candidate hybrid model means a full forward of the calibration
// sequences (FlexQuant, arXiv 2501.07139, Algorithm 1, calibrationEval), which is
// a dense contraction, so it runs on the matrix cores: 16x16x32 fp16 MFMA with
// fp32 accumulation.
//
// Quantized kernel.  Workgroup tile: BM=128 activation rows x BN=128 weight rows,
// one group of 128 k per iteration, 256 threads = 4 wavefronts side by side along
// N (each 128 x 32), two workgroups resident per CU.  The packed format stores a lane's 32 weights of a group as
// the A operands of four consecutive MFMA k-steps, so every wavefront loads its
// own packed chunks straight from global memory into registers (1 KiB contiguous
// per load), dequantizes them there and feeds the matrix core: weights never
// touch LDS and are unpacked once per workgroup.  Activations are shared by the
// four wavefronts through a double-buffered LDS tile, row-major with 16-byte
// chunks XOR-swizzled by row so that the coalesced copy and the operand reads are
// both free of bank conflicts; the copy goes from global memory straight into LDS.  Loads for group g+1 are issued
// before the MFMAs of group g; one barrier per iteration.
//
// The linears of a block that share their input (q/k/v, gate/up) go out as one launch whose workgroups
// each look up their matrix: a matrix whose tiles do not fill the workgroup slots a whole number of times
// shares its last round with the next one.
//
// The unquantized head runs the same kernel: its fp16 weights are read from the row-major matrix
// directly into the operand registers (sixteen rows by 64 contiguous bytes per load).
#include "fq_device.h"
#include "fq_internal.h"

#include <algorithm>
#include <climits>
#include <type_traits>
#include <utility>

namespace {

// ------------------------------------------------------------ quantized GEMM
constexpr int QBM = 128, QMB = QBM / 16; // per wave: QNB weight blocks (template) x QMB activation blocks

constexpr int DENSE = 16; // BITS value of the unquantized fp16 weight path (the vocabulary head)

template <int BITS>
struct WChunk {
    uint32_t c[BITS];
    uint32_t scale, zero; // fp16 bits in the low half, as loaded: nothing touches them before their use
};

// fp16 weights: a lane's operands of the four k-steps, read straight from the row-major matrix
template <>
struct WChunk<DENSE> {
    h8 f[4];
};

// Descriptors of the kernel's arrays (see make_rsrc).
struct GemmBuffers {
    fq_rsrc x, packed, scales, zeros;
};

template <int BITS>
__device__ __forceinline__ void load_wchunk(WChunk<BITS> &w, const GemmBuffers &buf, int rb16, int Np16, int G, int K,
                                            int g, int lane)
{
    if constexpr (BITS == DENSE) {
        // packed is the fp16 matrix [N,K]; Np16 carries N here.  Rows past the end re-read the last row.
        const int row = min(rb16 * 16 + (lane & 15), Np16 - 1);
        const uint32_t lo = ((uint32_t)row * (uint32_t)K + 8u * (uint32_t)(lane >> 4)) * 2u;
#pragma unroll
        for (int s = 0; s < 4; ++s)
            w.f[s] = __builtin_bit_cast(h8, buf_load_b128(buf.packed, lo + 64u * s, (uint32_t)g * 256u));
    } else {
        constexpr int SUB = Fmt<BITS>::SUB;
        // blocks past the end of the matrix re-read the last block: their results are never stored, and
        // loads without a branch keep the count of loads in flight known to the compiler
        const int rb = min(rb16, Np16 - 1);
        const uint32_t tile_off = (uint32_t)((rb / SUB) * G + g) * (uint32_t)(tile_dwords<BITS>() * 4);
        buf_load_chunk<BITS>(buf.packed, tile_off, rb % SUB, lane, w.c);
        const uint32_t meta_off = (uint32_t)(rb * G + g) * 32u, lo = (uint32_t)(lane & 15) * 2u;
        w.scale = buf_load_u16(buf.scales, lo, meta_off);
        w.zero = buf_load_u16(buf.zeros, lo, meta_off);
    }
}

// One output tile of one matrix.  Xs: the workgroup's two activation tiles in LDS, [2][QBM * 16], chunk ch of
// row r at r*16 + (ch ^ (r & 15)).  `tile` numbers the matrix's tiles in bands of four activation row-tiles
// (row-tile fastest): tiles with consecutive numbers share weight tiles and a few activation row-tiles.
template <int BITS, int QNB>
__device__ __forceinline__ void qgemm_tile(h8 (*Xs)[QBM * 16], const _Float16 *__restrict__ x, int M,
                                           const uint32_t *__restrict__ packed, const _Float16 *__restrict__ scales,
                                           const _Float16 *__restrict__ zeros, int N, int K,
                                           _Float16 *__restrict__ out, int ld, int tile)
{
    constexpr int QBN = 64 * QNB;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NT = (N + QBN - 1) / QBN, MT = (M + QBM - 1) / QBM;
    const int band = tile / (4 * NT), rest = tile - band * 4 * NT, height = min(4, MT - 4 * band);
    const int m0 = (4 * band + rest % height) * QBM, n0 = (rest / height) * QBN;
    const int G = K >> 7;
    const int Np16 = BITS == DENSE ? N : ((N + 63) / 64 * 64) >> 4; // sixteen-row blocks present (dense: rows)
    const int rb0 = (n0 >> 4) + wave * QNB; // first sixteen-row weight block of this wave

    // activation copy, global memory straight into LDS (no register hop): the i-th load of a wavefront
    // fills the 64 consecutive 16-byte slots from 64*wave + 256*i, lane by lane; slot (row, pos) holds
    // chunk pos ^ (row & 15) of its row, so each lane fetches that chunk.  Rows past M re-read row M-1.
    // Source addresses are the group's byte offset in a row (uniform) plus a 32-bit lane offset.
    const int xrow = 4 * wave + (lane >> 4), xch = (lane & 15) ^ (xrow & 15);
    uint32_t xoff[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        xoff[i] = ((uint32_t)min(m0 + xrow + 16 * i, M - 1) * (uint32_t)K + (uint32_t)xch * 8u) * 2u;
    GemmBuffers buf;
    buf.x = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2u);
    if constexpr (BITS == DENSE) {
        buf.packed = make_rsrc(packed, (uint32_t)N * (uint32_t)K * 2u);
        buf.scales = buf.zeros = buf.packed; // unused
    } else {
        const uint32_t Np = (uint32_t)(N + 63) / 64u * 64u;
        buf.packed = make_rsrc(packed, Np / 8u * (uint32_t)K * (uint32_t)BITS);
        buf.scales = make_rsrc(scales, Np * (uint32_t)G * 2u);
        buf.zeros = make_rsrc(zeros, Np * (uint32_t)G * 2u);
    }

    f4 acc[QNB][QMB];
#pragma unroll
    for (int i = 0; i < QNB; ++i)
#pragma unroll
        for (int j = 0; j < QMB; ++j)
            acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    WChunk<BITS> wc[QNB];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buf.x, &Xs[0][64 * wave + 256 * i], 16, xoff[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < QNB; ++i)
        load_wchunk<BITS>(wc[i], buf, rb0 + i, Np16, G, K, 0, lane);
    __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0); // the copies into LDS have landed ...
    __syncthreads();                            // ... in every wavefront

    // Integer zeros (what the quantizer produces) let bias and zero leave a pair in one addition: look
    // at the zeros of this workgroup's weight rows once and take the matching copy of the main loop.
    bool intz = true;
    if constexpr (BITS != DENSE && QNB != 4) {
        const uint32_t first = (uint32_t)(n0 >> 4) * (uint32_t)G * 16u, count = (QBN / 16) * (uint32_t)G * 16u;
        int frac = 0;
        for (uint32_t i = (uint32_t)tid * 8u; i < count; i += 256u * 8u) { // past the array: zeros
            const h8 z = __builtin_bit_cast(h8, buf_load_b128(buf.zeros, (first + i) * 2u, 0));
#pragma unroll
            for (int e = 0; e < 8; ++e)
                frac |= z[e] != __builtin_truncf16(z[e]);
        }
        intz = !__syncthreads_or(frac);
    }

    auto main_loop = [&](auto intz_tag) {
    constexpr bool INTZ = decltype(intz_tag)::value;
    for (int g = 0; g < G; ++g) {
        const int cur = g & 1;
        // dequantize this group's weights into operands: (code - zero) * scale
        h8 a[QNB][4];
#pragma unroll
        for (int i = 0; i < QNB; ++i) {
            if constexpr (BITS == DENSE) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    a[i][s] = wc[i].f[s];
            } else {
                h2 q[16];
                unpack_dequant<BITS, INTZ>(wc[i].c, as_h2(wc[i].zero * 0x10001u), as_h2(wc[i].scale * 0x10001u), q);
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    a[i][s] = make_h8(q[4 * s], q[4 * s + 1], q[4 * s + 2], q[4 * s + 3]);
            }
        }
        // prefetch the next group
        const bool more = g + 1 < G;
        if (more) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(buf.x, &Xs[cur ^ 1][64 * wave + 256 * i], 16, xoff[i],
                                                         (uint32_t)(g + 1) * 256u, 0, 0);
#pragma unroll
            for (int i = 0; i < QNB; ++i)
                load_wchunk<BITS>(wc[i], buf, rb0 + i, Np16, G, K, g + 1, lane);
        }
        // contraction
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            h8 b[QMB];
#pragma unroll
            for (int j = 0; j < QMB; ++j) {
                const int row = j * 16 + (lane & 15), ch = 4 * s + (lane >> 4);
                b[j] = Xs[cur][row * 16 + (ch ^ (row & 15))];
            }
#pragma unroll
            for (int i = 0; i < QNB; ++i)
#pragma unroll
                for (int j = 0; j < QMB; ++j)
                    acc[i][j] = mfma16x16x32(a[i][s], b[j], acc[i][j]);
        }
        __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0);
        __syncthreads();
    }
    };
    // Narrow quantized tiles: the same loop, software-pipelined inside the wavefront.  Matrix and vector
    // instructions leave through one issue port, so a wavefront that unpacks first and multiplies afterwards
    // leaves the matrix pipe idle while it unpacks, whatever the other resident wavefront does; here the
    // operands of group g+1 are unpacked between the MFMAs of group g (each MFMA occupies the pipe for four
    // issue slots and needs one).  Two chunk buffers and two operand buffers; the loads of group g+2 go out at
    // the top of iteration g, so everything the end-of-iteration wait covers was issued an iteration ago.
    auto pipelined_loop = [&](auto intz_tag) {
        constexpr bool INTZ = decltype(intz_tag)::value;
        if constexpr (BITS != DENSE) {
            WChunk<BITS> wd[QNB];
            h8 a0[QNB][4], a1[QNB][4];
            auto unpack_all = [&](WChunk<BITS> (&w)[QNB], h8 (&a)[QNB][4]) {
#pragma unroll
                for (int i = 0; i < QNB; ++i) {
                    h2 q[16];
                    unpack_dequant<BITS, INTZ>(w[i].c, as_h2(w[i].zero * 0x10001u), as_h2(w[i].scale * 0x10001u), q);
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        a[i][s] = make_h8(q[4 * s], q[4 * s + 1], q[4 * s + 2], q[4 * s + 3]);
                }
            };
            auto load_all = [&](WChunk<BITS> (&w)[QNB], int g) {
#pragma unroll
                for (int i = 0; i < QNB; ++i)
                    load_wchunk<BITS>(w[i], buf, rb0 + i, Np16, G, K, min(g, G - 1), lane);
            };
            auto body = [&](int g, h8 (&ac)[QNB][4], h8 (&an)[QNB][4], WChunk<BITS> (&wn)[QNB], WChunk<BITS> (&wl)[QNB]) {
                const int cur = g & 1;
                // past the last group both prefetches repeat it (nobody reads them): no branch in the iteration
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(buf.x, &Xs[cur ^ 1][64 * wave + 256 * i], 16, xoff[i],
                                                             (uint32_t)min(g + 1, G - 1) * 256u, 0, 0);
                load_all(wl, g + 2);
                unpack_all(wn, an); // ahead of the MFMAs in program order: the scheduler fills their shadows with it
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    h8 b[QMB];
#pragma unroll
                    for (int j = 0; j < QMB; ++j) {
                        const int row = j * 16 + (lane & 15), ch = 4 * s + (lane >> 4);
                        b[j] = Xs[cur][row * 16 + (ch ^ (row & 15))];
                    }
#pragma unroll
                    for (int i = 0; i < QNB; ++i)
#pragma unroll
                        for (int j = 0; j < QMB; ++j)
                            acc[i][j] = mfma16x16x32(ac[i][s], b[j], acc[i][j]);
                }
                __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0);
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0); // nothing moves from one iteration into the other
            };
            unpack_all(wc, a0);
            load_all(wc, 1);
            int g = 0;
            for (; g + 1 < G; g += 2) {
                body(g, a0, a1, wc, wd);
                body(g + 1, a1, a0, wd, wc);
            }
            if (g < G)
                body(g, a0, a1, wc, wd);
        }
    };
    if constexpr (QNB == 4 || BITS == DENSE)
        main_loop(std::false_type{}); // the wide tile has no registers to spare for a second copy of the loop
    else if (intz)
        pipelined_loop(std::true_type{});
    else
        pipelined_loop(std::false_type{});

    // store: lane holds m = lane%16 and n = 4*(lane/16) + v of each 16x16 block; four values at once where
    // every row of the output (a column range of a wider array when ld > N) starts 8-byte aligned
    const bool vec_ok = (ld & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 7) == 0;
#pragma unroll
    for (int j = 0; j < QMB; ++j) {
        const int m = m0 + j * 16 + (lane & 15);
        if (m >= M)
            continue;
#pragma unroll
        for (int i = 0; i < QNB; ++i) {
            const int n = (rb0 + i) * 16 + 4 * (lane >> 4);
            _Float16 *o = out + (size_t)m * ld + n;
            if (n + 3 < N && vec_ok) {
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

// Workgroups are dealt to the eight XCDs round-robin and each XCD has its own L2: XCD x takes the x-th
// contiguous run of `total` tiles.  Returns -1 for the workgroups past the end (uniform over a workgroup).
__device__ __forceinline__ int xcd_tile(int total)
{
    const int per_xcd = (total + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    return tile < total ? tile : -1;
}

// Two workgroups per CU (two wavefronts per SIMD): a single wavefront cannot keep the matrix pipe
// busy, and two independent workgroups overlap one's unpack/copy phase with the other's MFMAs.
template <int BITS, int QNB>
__global__ __launch_bounds__(256, 2) void qgemm_kernel(const _Float16 *__restrict__ x, int M,
                                                       const uint32_t *__restrict__ packed,
                                                       const _Float16 *__restrict__ scales,
                                                       const _Float16 *__restrict__ zeros, int N, int K,
                                                       _Float16 *__restrict__ out)
{
    __shared__ h8 Xs[2][QBM * 16];
    constexpr int QBN = 64 * QNB;
    const int tile = xcd_tile(((N + QBN - 1) / QBN) * ((M + QBM - 1) / QBM));
    if (tile < 0)
        return; // before any barrier
    qgemm_tile<BITS, QNB>(Xs, x, M, packed, scales, zeros, N, K, out, N, tile);
}

// Up to three matrices with the same input in one launch (q/k/v, gate/up): their tiles form one list, so
// a matrix whose tiles do not fill the chip's workgroup slots a whole number of times shares its last
// round with the next matrix.  Each workgroup looks up its matrix and runs the tile code of that matrix's
// bit-width and tile width.
struct GemmJob {
    const uint32_t *packed;
    const _Float16 *scales, *zeros;
    _Float16 *out;
    int N, bits;
    int ld;  // elements between consecutive rows of out
    int qnb; // 128-row tiles: width, see qgemm_tile
};
struct GemmJobs {
    GemmJob j[3];
};

// The scalars of both kernels below are preloaded into registers at wavefront start; the matrix that they select is then one round of
// loads from the argument buffer.  first1, first2: first tile of the second and third matrix, beyond the last tile where there is none.
constexpr int GEMM_JOBS_AT = 32; // bytes of the arguments ahead of the jobs: a pointer and five numbers

__device__ __forceinline__ GemmJob gemm_job(int &tile, int first1, int first2)
{
    const int index = (tile >= first1) + (tile >= first2);
    tile -= index == 0 ? 0 : (index == 1 ? first1 : first2);
    return kernel_argument<GemmJobs>(GEMM_JOBS_AT)->j[index];
}

__global__ __launch_bounds__(256, 2) void qgemm_multi_kernel(const _Float16 *__restrict__ x, int M, int K, int total, int first1, int first2,
                                                             GemmJobs)
{
    __shared__ h8 Xs[2][QBM * 16];
    int tile = xcd_tile(total);
    if (tile < 0)
        return;
    const GemmJob job = gemm_job(tile, first1, first2);
    switch (job.bits * 8 + job.qnb) {
    case 2 * 8 + 4: qgemm_tile<2, 4>(Xs, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile); break;
    case 4 * 8 + 4: qgemm_tile<4, 4>(Xs, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile); break;
    case 2 * 8 + 2: qgemm_tile<2, 2>(Xs, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile); break;
    case 3 * 8 + 2: qgemm_tile<3, 2>(Xs, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile); break;
    case 4 * 8 + 2: qgemm_tile<4, 2>(Xs, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile); break;
    default: qgemm_tile<8, 2>(Xs, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile); break;
    }
}

// ------------------------------------------------------------ tall tiles
// Up to 256 activation rows x 128 weight rows per workgroup of eight wavefronts, one workgroup per CU, for products
// with many rows.  In the 128-row kernels every unpacked weight operand feeds 8 MFMAs and the unpacking is the
// largest share of what a wavefront issues beside its MFMAs; here a wavefront owns 256 x 32 outputs (128
// accumulator registers), so an operand feeds 16.  A 4096-column product at 2048 rows has only 256 such tiles,
// one per CU, so the second wavefront of every SIMD comes from splitting K inside the workgroup: wavefront
// (kh, nq) multiplies k-steps 2*kh and 2*kh+1 of every group with the weight rows 32*nq..+31, loads only that
// half of a chunk and unpacks only its eight pairs; the two partial sums meet in LDS at the end, in fp32.
// The loop is the narrow tiles' software pipeline (loads two groups ahead, operands of the next group
// unpacked ahead of this group's MFMAs in program order, one barrier per group).
//
// The two activation buffers are two LDS arrays on purpose.  A kernel with more than one LDS object has its LDS
// accesses tagged with alias scopes, and the compiler then waits for every direct-to-LDS load in flight before
// a read that may touch the same object: with both buffers in one array the reads of one buffer wait for the
// copies into the other right after they were issued, and the copy's whole latency (0.6 us per group here)
// lands on the wavefront.  With separate arrays, selected at compile time, the copies stay in flight until the
// wait at the end of the iteration.  As measured on MI355X (2048 rows, 4096 x 4096 and 4096 x 11008, same
// harness): 6-13 % faster than the 128-row kernels at every bit-width.
constexpr int TBM = 256, TBN = 128, TMB = TBM / 16, TNB = 2;

// The dwords of a chunk that hold k-steps 2*KH and 2*KH+1 (3 bits: all three, the last pair's bits sit on
// top of every dword), with the row's scale and zero; the other entries of w.c stay unset and unread.
template <int BITS, int KH>
__device__ __forceinline__ void load_whalf(WChunk<BITS> &w, const GemmBuffers &buf, int rb16, int Np16, int G, int g,
                                           int lane)
{
    constexpr int SUB = Fmt<BITS>::SUB;
    const int rb = min(rb16, Np16 - 1); // blocks past the end re-read the last block (see load_wchunk)
    const uint32_t tile_off = (uint32_t)((rb / SUB) * G + g) * (uint32_t)(tile_dwords<BITS>() * 4);
    const int u = rb % SUB;
    const uint32_t lo = (uint32_t)lane * 16u;
    if constexpr (BITS == 2) {
        w.c[KH] = buf_load_b32(buf.packed, lo + 8u * (uint32_t)u + 4u * KH, tile_off);
    } else if constexpr (BITS == 4) {
        const u2v v = buf_load_b64(buf.packed, lo + 8u * KH, tile_off);
        w.c[2 * KH] = v.x; w.c[2 * KH + 1] = v.y;
    } else if constexpr (BITS == 8) {
        const u4v v = buf_load_b128(buf.packed, lo + 1024u * KH, tile_off);
        w.c[4 * KH] = v.x; w.c[4 * KH + 1] = v.y; w.c[4 * KH + 2] = v.z; w.c[4 * KH + 3] = v.w;
    } else {
        buf_load_chunk<BITS>(buf.packed, tile_off, u, lane, w.c);
    }
    const uint32_t meta_off = (uint32_t)(rb * G + g) * 32u, mlo = (uint32_t)(lane & 15) * 2u;
    w.scale = buf_load_u16(buf.scales, mlo, meta_off);
    w.zero = buf_load_u16(buf.zeros, mlo, meta_off);
}

// Sixteen-row blocks of activation row tile `row_tile` of MT: as even a cut of row_blocks as blocks allow, the first tiles one block higher.
// Quotient and remainder: row_tile * row_blocks passes 2^31 from 2.97 million rows, which are taken up to K = 640.
struct TallCut {
    int block0, blocks;
};
__host__ __device__ constexpr TallCut tall_cut(int row_blocks, int MT, int row_tile)
{
    const int each = row_blocks / MT, rest = row_blocks % MT;
    return {row_tile * each + (row_tile < rest ? row_tile : rest), each + (row_tile < rest)};
}

// What a tall tile's body works on.
struct TallTile {
    GemmBuffers buf;
    _Float16 *out;
    uint32_t xoff0, xstep; // byte offset of the lane's part of copy 0, and from one copy to the next (32 rows)
    int rb0, Np16, G, K;   // first sixteen-row weight block of the wavefront, those that there are, groups
    int m0, m_end, N, ld;
};

// The main loop and the store of a tile of H sixteen-row blocks.  Xs0, Xs1: the two activation tiles (256 rows x 128 k each, laid out like
// the narrow tiles'); after the loop the same memory carries the second K half's partial sums to the first.
template <int BITS, int H, bool INTZ, int KH>
__device__ __forceinline__ void qgemm_tall_body(h8 *Xs0, h8 *Xs1, const TallTile &t)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nq = wave & 3;
    const int G = t.G, brow = lane & 15;
    f4 acc[TNB][H];
#pragma unroll
    for (int i = 0; i < TNB; ++i)
#pragma unroll
        for (int j = 0; j < H; ++j)
            acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    UnpackConsts<BITS> uc;
    uc.init();
    {
        WChunk<BITS> wc[TNB], wd[TNB];
        h8 a0[TNB][2], a1[TNB][2];
        auto unpack_all = [&](WChunk<BITS> (&w)[TNB], h8 (&a)[TNB][2]) {
#pragma unroll
            for (int i = 0; i < TNB; ++i)
                unpack_khalf<BITS, INTZ, true, KH>(w[i].c, as_h2(w[i].zero * 0x10001u), as_h2(w[i].scale * 0x10001u), uc, a[i]);
        };
        auto load_all = [&](WChunk<BITS> (&w)[TNB], int g) {
#pragma unroll
            for (int i = 0; i < TNB; ++i)
                load_whalf<BITS, KH>(w[i], t.buf, t.rb0 + i, t.Np16, G, min(g, G - 1), lane);
        };
        // Xc: this group's activations, Xn: the buffer the next group's are copied into.  Past the last group
        // both prefetches repeat it (nobody reads them): no branch in the iteration.
        auto body = [&](h8 *Xc, h8 *Xn, int g, h8 (&ac)[TNB][2], h8 (&an)[TNB][2], WChunk<BITS> (&wn)[TNB],
                        WChunk<BITS> (&wl)[TNB]) {
#pragma unroll
            for (int i = 0; i < (H + 1) / 2; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(t.buf.x, &Xn[64 * wave + 512 * i], 16, t.xoff0 + t.xstep * i,
                                                         (uint32_t)min(g + 1, G - 1) * 256u, 0, 0);
            __builtin_amdgcn_sched_barrier(0); // the copies go out first: they have the whole iteration to land
            load_all(wl, g + 2);
            unpack_all(wn, an); // ahead of the MFMAs in program order: the scheduler fills their shadows with it
            constexpr int JB = BITS == 3 ? 4 : (H < 16 ? (H + 1) / 2 : 8); // operand reads per batch (3 bits: the fewest registers to spare)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
#pragma unroll
                for (int jh = 0; jh < H; jh += JB) {
                    h8 b[JB];
#pragma unroll
                    for (int j = 0; j < JB && jh + j < H; ++j) {
                        const int ch = 4 * (2 * KH + s) + (lane >> 4);
                        b[j] = Xc[((jh + j) * 16 + brow) * 16 + (ch ^ brow)];
                    }
#pragma unroll
                    for (int i = 0; i < TNB; ++i)
#pragma unroll
                        for (int j = 0; j < JB && jh + j < H; ++j)
                            acc[i][jh + j] = mfma16x16x32(ac[i][s], b[j], acc[i][jh + j]);
                }
            }
            __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0); // this wavefront's copies into Xn have landed ...
            __syncthreads();                            // ... and everybody's; Xc is free
            __builtin_amdgcn_sched_barrier(0);          // nothing moves from one iteration into the other
        };
        load_all(wc, 0);
        unpack_all(wc, a0);
        load_all(wc, 1);
        int g = 0;
        for (; g + 1 < G; g += 2) {
            body(Xs0, Xs1, g, a0, a1, wc, wd);
            body(Xs1, Xs0, g + 1, a1, a0, wd, wc);
        }
        if (g < G)
            body(Xs0, Xs1, g, a0, a1, wc, wd);
    }

    // The second K half hands its sums over (every iteration ended with a wait for all loads and a barrier, so
    // both arrays are free): block (i, j) of column quarter nq at float4 (nq*16 + j)*64 + lane of array i.
    f4 *red0 = reinterpret_cast<f4 *>(Xs0), *red1 = reinterpret_cast<f4 *>(Xs1);
    if (KH == 1) {
#pragma unroll
        for (int j = 0; j < H; ++j) {
            red0[((nq * 16 + j) << 6) + lane] = acc[0][j];
            red1[((nq * 16 + j) << 6) + lane] = acc[1][j];
        }
    }
    __syncthreads();
    if (KH == 1)
        return;
    // store: lane holds m = lane%16 and n = 4*(lane/16) + v of each 16x16 block (see qgemm_tile)
    const int ld = t.ld, N = t.N;
    const bool vec_ok = (ld & 3) == 0 && (reinterpret_cast<uintptr_t>(t.out) & 7) == 0;
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const int m = t.m0 + j * 16 + (lane & 15);
#pragma unroll
        for (int i = 0; i < TNB; ++i) {
            const f4 r = acc[i][j] + (i ? red1 : red0)[((nq * 16 + j) << 6) + lane];
            const int n = (t.rb0 + i) * 16 + 4 * (lane >> 4);
            if (m >= t.m_end)
                continue;
            _Float16 *o = t.out + (size_t)m * ld + n;
            if (n + 3 < N && vec_ok) {
                h4 v = {(_Float16)r[0], (_Float16)r[1], (_Float16)r[2], (_Float16)r[3]};
                *reinterpret_cast<h4 *>(o) = v;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < N)
                        o[v] = (_Float16)r[v];
            }
        }
    }
}

template <int BITS, int H, bool INTZ>
__device__ __forceinline__ void qgemm_tall_halves(h8 *Xs0, h8 *Xs1, const TallTile &t, int kh)
{
    if (kh == 0)
        qgemm_tall_body<BITS, H, INTZ, 0>(Xs0, Xs1, t);
    else
        qgemm_tall_body<BITS, H, INTZ, 1>(Xs0, Xs1, t);
}

// One output tile of up to 256 x 128.
template <int BITS>
__device__ __forceinline__ void qgemm_tall_tile(h8 *Xs0, h8 *Xs1, const _Float16 *__restrict__ x, int M,
                                                const uint32_t *__restrict__ packed,
                                                const _Float16 *__restrict__ scales,
                                                const _Float16 *__restrict__ zeros, int N, int K,
                                                _Float16 *__restrict__ out, int ld, int tile, int MT)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave >> 2, nq = wave & 3; // half of every group's k-steps, quarter of the tile's weight rows
    // Tiles are numbered in bands of two row-tiles (row-tile fastest): the 32 tiles an XCD holds at a
    // time share up to 512 activation rows (4 MiB at k = 4096, the size of its L2) and 16 weight tiles
    const int NT = (N + TBN - 1) / TBN;
    const int band = tile / (2 * NT), rest = tile - band * 2 * NT, height = min(2, MT - 2 * band);
    const int row_tile = 2 * band + rest % height, n0 = (rest / height) * TBN;
    const TallCut cut = tall_cut((M + 15) / 16, MT, row_tile); // up to TMB blocks
    const int blocks = cut.blocks;
    TallTile t;
    t.m0 = 16 * cut.block0;
    t.m_end = min(M, t.m0 + 16 * blocks);
    t.G = K >> 7;
    t.Np16 = ((N + 63) / 64 * 64) >> 4;
    t.rb0 = (n0 >> 4) + nq * TNB;
    t.N = N;
    t.K = K;
    t.ld = ld;
    t.out = out;
    const int G = t.G;

    t.buf.x = make_rsrc(x, (uint32_t)t.m_end * (uint32_t)K * 2u);
    const uint32_t Np = (uint32_t)(N + 63) / 64u * 64u;
    t.buf.packed = make_rsrc(packed, Np / 8u * (uint32_t)K * (uint32_t)BITS);
    t.buf.scales = make_rsrc(scales, Np * (uint32_t)G * 2u);
    t.buf.zeros = make_rsrc(zeros, Np * (uint32_t)G * 2u);

    // Activation copies, global memory straight into LDS: copy i of a wavefront fills the 64 slots from
    // 64*wave + 512*i, i.e. rows 4*wave + 32*i + lane/16; slot (row, pos) holds chunk pos ^ (row & 15).  The
    // row is part of the lane offset, which the descriptor's range check covers (the scalar offset, which
    // carries the group's bytes within the row, is not checked): rows past the tile's read as zero and are never stored.
    const int xrow = 4 * wave + (lane >> 4), xch = (lane & 15) ^ (xrow & 15);
    t.xoff0 = ((uint32_t)(t.m0 + xrow) * (uint32_t)K + (uint32_t)xch * 8u) * 2u;
    t.xstep = 64u * (uint32_t)K; // 32 rows
#pragma unroll
    for (int i = 0; i < 8; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(t.buf.x, &Xs0[64 * wave + 512 * i], 16, t.xoff0 + t.xstep * i, 0, 0, 0);

    // integer zeros: one addition takes bias and zero away (see qgemm_tile)
    bool intz;
    {
        const uint32_t first = (uint32_t)(n0 >> 4) * (uint32_t)G * 16u, count = (TBN / 16) * (uint32_t)G * 16u;
        int frac = 0;
        for (uint32_t i = (uint32_t)tid * 8u; i < count; i += 512u * 8u) { // past the array: zeros
            const h8 z = __builtin_bit_cast(h8, buf_load_b128(t.buf.zeros, (first + i) * 2u, 0));
#pragma unroll
            for (int e = 0; e < 8; ++e)
                frac |= z[e] != __builtin_truncf16(z[e]);
        }
        __builtin_amdgcn_s_waitcnt(FQ_WAIT_VMCNT0); // the first activation tile has landed ...
        intz = !__syncthreads_or(frac);             // ... in every wavefront
    }

    auto of_height = [&](auto height) {
        constexpr int H = decltype(height)::value;
        if (intz)
            qgemm_tall_halves<BITS, H, true>(Xs0, Xs1, t, kh);
        else
            qgemm_tall_halves<BITS, H, false>(Xs0, Xs1, t, kh);
    };
    // the least height that holds the tile's blocks (see tall_height)
    if (blocks > 15)
        of_height(std::integral_constant<int, 16>{});
    else if (blocks > 14)
        of_height(std::integral_constant<int, 15>{});
    else if (blocks > 13)
        of_height(std::integral_constant<int, 14>{});
    else if (blocks > 12)
        of_height(std::integral_constant<int, 13>{});
    else if (blocks > 10)
        of_height(std::integral_constant<int, 12>{});
    else if (blocks > 8)
        of_height(std::integral_constant<int, 10>{});
    else
        of_height(std::integral_constant<int, 8>{});
}

// Eight wavefronts of 256 registers each: one workgroup per CU, two wavefronts per SIMD.
__global__ __launch_bounds__(512, 1) void qgemm_tall_kernel(const _Float16 *__restrict__ x, int M, int K, int total, int first1, int first2,
                                                            int row_tiles, GemmJobs)
{
    __shared__ h8 Xs0[TBM * 16];
    __shared__ h8 Xs1[TBM * 16];
    int tile = xcd_tile(total);
    if (tile < 0)
        return;
    const GemmJob job = gemm_job(tile, first1, first2);
    switch (job.bits) {
    case 2: qgemm_tall_tile<2>(Xs0, Xs1, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile, row_tiles); break;
    case 3: qgemm_tall_tile<3>(Xs0, Xs1, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile, row_tiles); break;
    case 4: qgemm_tall_tile<4>(Xs0, Xs1, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile, row_tiles); break;
    default: qgemm_tall_tile<8>(Xs0, Xs1, x, M, job.packed, job.scales, job.zeros, job.N, K, job.out, job.ld, tile, row_tiles); break;
    }
}

static_assert(last_argument_at(qgemm_multi_kernel) == GEMM_JOBS_AT && last_argument_at(qgemm_tall_kernel) == GEMM_JOBS_AT);

// Weight-tile width.  Wide tiles (each wavefront 128 x 64) halve the LDS reads and activation copies per
// MFMA but need at least two workgroups per CU to keep both wavefront slots of every SIMD filled.
int wide_tiles_pay(int M, int N)
{
    const long tiles = (long)((N + 255) / 256) * ((M + QBM - 1) / QBM);
    return tiles >= 2 * 256;
}

constexpr int CUS = 256;

// Row blocks that a tile of `blocks` is worked on as: the heights there are bodies for.  13 blocks take 4 % less than 14 (1 to 7 over four widths, K =
// 1024 to 11008, one and two rounds), 14 take 6 % less than 15 and 15 take 3 % less than 16; 9 and 11 would gain 1 to 3 on the next.
int tall_height(int blocks) { return blocks > 12 ? blocks : (blocks > 10 ? 12 : (blocks > 8 ? 10 : 8)); }

// Row tiles that a launch of tall tiles cuts M into, by estimated time (fitted to 29000 launches; from K = 2560 on 5 % off, shorter ones
// up to 20).  Rounds over the CUs, a tile each; a last round that is not full takes nearly as long as a full one.  A round takes, of every group
// of 128 k, a part that does not depend on the height (a tile's weights are unpacked whatever it is) and one that does.  Tiles of TBM rows are the
// fewest; more and lower ones are better where they fill the rounds better, and a launch's tiles are only as high as they have to be: at full
// height, rows that do not divide by TBM cost a last tile of a few rows as much as a whole one.  Measured, us, full height -> as chosen: 1500 x 11008 x 4096
// at 2 bits 158 -> 135 (eight of 192), 800 x 22016 x 4096 at 4 bits 168 -> 137 (four of 208); a call that was the 128-row kernel's, 1890 x 1420 x 6400 at 2
// bits, 70 -> 52 (fifteen of 128).  On rows shorter than 2048, whose kernel is chosen by full heights, the cut takes 8 % less than those over 300 sizes and
// nowhere over 2 % more.  Exactly as many tiles as whole rounds hold, by one more in some of the columns, gave 3 % more at one size in sixteen: a chip
// that is full clocks lower, and 2048 x 11008 x 4096 takes 166 us in 2.7 rounds of full height as in three of 240 rows.
int plan_tall(int M, const fq_packed_ref *w, int count, double *us)
{
    static const double whole[9] = {0, 0, 0.390, 0.812, 0.362, 0, 0, 0, 0.418}, block[9] = {0, 0, 0.063, 0.049, 0.067, 0, 0, 0, 0.066};
    int columns = 0;
    double fixed = 0.0, each = 0.0;
    for (int i = 0; i < count; ++i) {
        const int n = (w[i].N + TBN - 1) / TBN;
        columns += n;
        fixed += n * whole[w[i].bits];
        each += n * block[w[i].bits];
    }
    const int blocks = (M + 15) / 16, least = (blocks + TMB - 1) / TMB, G = w[0].K >> 7;
    int best = least;
    *us = 1e30;
    for (int k = least; k <= least + 16; ++k) {
        const int high = (blocks + k - 1) / k, H = tall_height(high);
        if (k > least && high < 7)
            break;
        const long tiles = (long)k * columns, whole_rounds = tiles / CUS;
        const double rest = (double)(tiles % CUS) / CUS;
        const double rounds = (double)whole_rounds + (rest == 0.0 ? 0.0 : (whole_rounds == 0 ? 0.83 + 0.16 * rest : 0.89 + 0.10 * rest));
        const double t = 2.5 + (double)(whole_rounds + (rest != 0.0)) * (0.92 + 0.658 * H) + G * rounds * (fixed + each * H) / columns;
        if (t < *us) {
            *us = t;
            best = k;
        }
    }
    return best;
}

// What the few-row kernel's estimate is held against (us), and what gives a call to the tall kernel by tiles of the full height (full_height).  The
// times: rounds over the 256 CUs, two 128-row tiles a CU or one tall one; measured over 32 groups, 512 to 2048 rows, 4096 to 22016 columns (us at 2 / 3 / 4 / 8
// bits) a full round of 128-row tiles 63 / 73 / 67 / 73, its last one 47 when at most one tile a CU is left and 4 under a full one otherwise; of tall ones
// 61 / 67 / 63 / 66, a last one 50 to 60.  Up to 256 128-row tiles, one a CU: 5.4 us and 1.31 us a group of 128 k; up to 512, 1.5 us (3 bits 1.8) a group and
// more the more CUs have two; beyond, the rounds above and 6 us, on rows shorter than 4096 up to 6 more.  Of that 0.92 (with a 3-bit matrix 0.9), up to
// 512 tiles from K = 4096 on, and the factors of the tall tiles below: without them the few-row kernel was taken for 29 of 300 sizes that it
// serves 2 to 26 % more slowly, with them for 10, up to 8 %.
//
// Rows shorter than 2048, where what a round takes beside its groups counts, go by full_height alone: a round of tall tiles keeps up to 1.5 us more (the
// two halves of its K meet through LDS): 229 rows of 20424 x 128 11.9 against 9.0 us, 1932 of 3144 x 384 15.8 against 13.9.  So do launches of 2- and
// 4-bit matrices only from 4096 rows on, whose 128 x 256 tiles run several full rounds and are level or 2-6 % ahead.
//
// The lower tall tiles are not in `us`: they would take calls from the few-row kernel, which applies a scale to sums in fp32 where they round it into
// every weight.  Over 1000 of its calls of 129 to 2200 rows from K = 2048 on, large tiles would take over 10 % less at 47 and over a quarter less at
// two (1282 x 6491 x 11008 at 3 bits 255 us against 414, 1363 x 1857 x 13824 at 4 bits 104 against 139; 1200 x 4096 x 11008 at 4 bits 107 against 159).
struct LargeTiles {
    double us;
    long tiles; // of 128 rows
    bool full_height, all_wide;
};
LargeTiles large_tiles(int M, const fq_packed_ref *w, int count)
{
    static const double full128[9] = {0, 0, 63, 73, 67, 0, 0, 0, 73}, full256[9] = {0, 0, 61, 67, 63, 0, 0, 0, 66};
    long tiles = 0, tall = 0;
    double f128 = 0.0, f256 = 0.0, three = 0.0;
    bool all_wide = M >= 4096;
    for (int i = 0; i < count; ++i) {
        const int t = ((w[i].N + 127) / 128) * ((M + 127) / 128);
        tiles += t;
        tall += ((w[i].N + TBN - 1) / TBN) * ((M + TBM - 1) / TBM);
        f128 += t * full128[w[i].bits];
        f256 += t * full256[w[i].bits];
        three = w[i].bits == 3 ? 0.3 : three;
        all_wide = all_wide && (w[i].bits == 2 || w[i].bits == 4) && wide_tiles_pay(M, w[i].N);
    }
    const int G = w[0].K >> 7;
    const double length = w[0].K / 4096.0; // of the rows, in those that the figures above were taken with
    const double brief = length < 1.0 ? 6.0 * (1.0 - length) : 0.0, long_part = three != 0.0 ? 0.9 : 0.92;
    f128 /= tiles;
    f256 /= tiles;
    const long r128 = tiles % 512, r256 = tall % 256;
    const double t128 = (tiles / 512) * f128 + (r128 == 0 ? 0.0 : (r128 <= 256 ? 47.0 : f128 - 4.0));
    const double t256 = (tall / 256) * f256 + (r256 == 0 ? 0.0 : 50.0 + 10.0 * r256 / 256);
    const double low = 5.4 + G * (tiles <= 256 ? 1.31 : 1.5 + three + 0.7 * (tiles - 256) / 256.0);
    const double us128 = tiles <= 256 ? low : (tiles <= 512 ? (low + brief) * (length < 1.0 ? 1.0 : long_part) : (6.0 + t128 * length + brief) * long_part);
    const double fixed256 = length < 1.0 ? 1.5 * (1.0 - length) * (tall / 256 + (r256 != 0)) : 0.0;
    const bool full_height = M > 128 && tiles > 256 && !all_wide && t256 * length + fixed256 < t128 * length;
    double us = us128;
    if (full_height)
        us = (3.0 + t256 * length + fixed256 + brief) * (three != 0.0 || length < 1.0 ? 1.0 : (tall <= 256 ? 0.9 : 0.95));
    return {us, tiles, full_height, all_wide};
}

// Estimated time of 128-row tiles that plan_tall's is held against, fitted to 2500 launches of 130 to 4096 rows from K = 2048 on (6.4 % off; the
// one in large_tiles, which the few-row kernel is held against, 7.8, up to 20 too high where 257 to 512 tiles nearly fill the chip and as much too
// low where they hardly start a second one a CU).  Rounds of 512 tiles, two a CU; a group of a full one takes 1.62 / 1.84 / 1.74 / 1.86 us at 2 / 3 / 4 / 8
// bits (at 3 the 1.77 below: plan_tall's is as much too low there; 5473 x 374 x 2816 37.1 us and 39.4 in tall tiles), of one that is not full the parts below.  A launch of 128 x 256 tiles and others takes a fifth longer: each XCD has as many tiles as the next
// (2174 rows of two 11008 x 4096 at 8 and 2 bits 478 us, 365 in tall tiles).
double us_128(int M, const fq_packed_ref *w, int count)
{
    static const double group[9] = {0, 0, 1.62, 1.77, 1.74, 0, 0, 0, 1.86};
    long tiles = 0;
    double each = 0.0;
    int wide = 0;
    for (int i = 0; i < count; ++i) {
        wide += (w[i].bits == 2 || w[i].bits == 4) && wide_tiles_pay(M, w[i].N);
        const long t = (long)((w[i].N + 127) / 128) * ((M + 127) / 128);
        tiles += t;
        each += t * group[w[i].bits];
    }
    const long whole = tiles / (2 * CUS), rest = tiles % (2 * CUS);
    const double x = (double)rest / CUS;
    double part = 0.0;
    if (rest != 0 && whole == 0)
        part = x <= 1.0 ? 0.71 : 0.65 + 0.20 * x;
    else if (rest != 0)
        part = x <= 1.0 ? 0.60 + 0.09 * x : 0.64 + 0.25 * x;
    const double us = 3.1 + 5.5 * (whole + (rest != 0)) + (w[0].K >> 7) * (each / tiles) * (whole + part);
    return wide != 0 && wide != count ? 1.2 * us : us;
}

// Row tiles of the tall kernel, or 0: the 128-row kernel.  From K = 2048 on by the two estimates above, except that calls of up to two 128-row tiles
// a CU that go to the tall kernel by tiles of the full height stay there, and with a margin for all that this choice gives to either kernel.  Over
// 2000 sizes of 130 to 16000 rows the calls take 9 % less on average than by full heights, 4 of them 5 to 9 % more (9, up to 22 %, by the estimate of
// large_tiles: 252 x 22016 x 4096 at 8 bits 51.4 us in tall tiles and 59.6 in the others, 578 x 12288 x 11008 at 2 bits 183 and 150); over 1500 launches
// of two or three matrices 7 % less, one over 5 % more (27, up to 46 %: 1223 rows of two 13824 x 4096 at 4 and 3 bits 295 and 373).
int tall_row_tiles(int M, const fq_packed_ref *w, int count, const LargeTiles &large)
{
    const bool by_full_height = w[0].K < 2048 || large.all_wide;
    if (M <= 128 || (by_full_height && !large.full_height))
        return 0;
    double us256;
    const int row_tiles = plan_tall(M, w, count, &us256);
    if (by_full_height || (large.full_height && large.tiles <= 2 * CUS))
        return row_tiles;
    return us256 < (large.full_height ? 1.03 : 0.98) * us_128(M, w, count) ? row_tiles : 0;
}

template <int BITS, int QNB>
int launch_tile(const void *x, int M, const void *packed, const void *scales, const void *zeros, int N, int K,
                void *out, fq_stream st)
{
    constexpr int QBN = 64 * QNB;
    const int total = ((N + QBN - 1) / QBN) * ((M + QBM - 1) / QBM);
    dim3 grid(8 * ((total + 7) / 8)), block(256);
    hipLaunchKernelGGL((qgemm_kernel<BITS, QNB>), grid, block, 0, st, static_cast<const _Float16 *>(x), M,
                       static_cast<const uint32_t *>(packed), static_cast<const _Float16 *>(scales),
                       static_cast<const _Float16 *>(zeros), N, K, static_cast<_Float16 *>(out));
    return (int)hipGetLastError();
}

template <int BITS>
int launch_q(const void *x, int M, const fq_packed_ref &w, void *out, fq_stream st)
{
    // 3- and 8-bit operands do not fit the register budget of a wide tile
    if ((BITS == 2 || BITS == 4) && wide_tiles_pay(M, w.N))
        return launch_tile<(BITS == 2 || BITS == 4) ? BITS : 4, 4>(x, M, w.packed, w.scales, w.zeros, w.N, w.K, out, st);
    return launch_tile<BITS, 2>(x, M, w.packed, w.scales, w.zeros, w.N, w.K, out, st);
}

} // namespace

// The kernels address x, the packed weights and the scales/zeros through 32-bit byte offsets.
static bool fits_32bit(size_t a, size_t b, size_t elem_bytes) { return a * b * elem_bytes < ((size_t)1 << 32); }

namespace {

// The jobs of a launch; tiles(i): tiles of matrix i; qnb(i): its tile width.
struct GemmLaunch {
    GemmJobs jobs = {};
    int first[4] = {0, INT_MAX, INT_MAX, INT_MAX}, total = 0;
    template <class T, class Q>
    GemmLaunch(const fq_packed_ref *w, void *const *outs, int count, T &&tiles, Q &&qnb)
    {
        for (int i = 0; i < count; ++i) {
            jobs.j[i] = GemmJob{static_cast<const uint32_t *>(w[i].packed), static_cast<const _Float16 *>(w[i].scales),
                                static_cast<const _Float16 *>(w[i].zeros), static_cast<_Float16 *>(outs[i]), w[i].N,
                                w[i].bits, w[i].ld ? w[i].ld : w[i].N, qnb(i)};
            first[i] = total;
            total += tiles(i);
        }
    }
};

} // namespace

// What the highest tiles of a launch of the tall kernel are worked on as.
static int highest_rows(int M, int row_tiles) { return 16 * tall_height(((M + 15) / 16 + row_tiles - 1) / row_tiles); }

int fq_gemm_tall_tile(int M, const fq_packed_ref *w, int count, int row_tile, int *first, int *rows, int *worked)
{
    double us;
    const int row_tiles = plan_tall(M, w, count, &us);
    if (row_tile >= 0 && row_tile < row_tiles) {
        const TallCut cut = tall_cut((M + 15) / 16, row_tiles, row_tile);
        *first = 16 * cut.block0;
        *rows = std::min(M - *first, 16 * cut.blocks);
        *worked = 16 * tall_height(cut.blocks);
    }
    return row_tiles;
}

// row_tiles: as planned; 0 where the caller pins the kernel.
static int launch_tall(const void *x, int M, const fq_packed_ref *w, void *const *outs, int count, fq_stream st, int row_tiles)
{
    double us;
    if (row_tiles == 0)
        row_tiles = plan_tall(M, w, count, &us);
    const GemmLaunch l(w, outs, count, [&](int i) { return row_tiles * ((w[i].N + TBN - 1) / TBN); }, [](int) { return 0; });
    hipLaunchKernelGGL(qgemm_tall_kernel, dim3(8 * ((l.total + 7) / 8)), dim3(512), 0, st,
                       static_cast<const _Float16 *>(x), M, w[0].K, l.total, l.first[1], l.first[2], row_tiles, l.jobs);
    return (int)hipGetLastError();
}

// Up to sixteen rows (the linears of a stack forward, which has no use for the streaming kernel then) the few-row kernel
// serves every launch whose offsets it can hold; beyond, the launches for which it is expected to be the faster one
// (measured in us: 77 rows of 4096 x 11008 at 3 bits 18 against 109, 300 35 against 116, 611 69 against 117; 300 of 11008 x 4096 45 against 50, 611 83
// against 57).  On short rows the estimate of the large tiles is too low, the more the shorter (300 x 2539 x 256 at 3 bits 7.6 us against
// 11.6 in large tiles, 55 x 15513 x 256 7.1 against 8.05, 2126 x 402 x 256 7.5 against 11.6): over 660 sizes both take the same time where
// the few-row kernel is expected to take 1.3 to 1.4 of the other's time at K = 256, 1.2 to 1.3 at 512 and 1.0 to 1.15 up to 1408 (many rounds
// of its sixteen-row tiles, 20 x 23466 x 256, are not ahead: 7.3 against 9.0).  Tiles of up to 32 columns have a tenth in their favour up
// to 1280: they keep the scales in fp32, the large ones round them into the weights.
fq_gemm_plan fq_plan_gemm(int M, const fq_packed_ref *w, int count)
{
    const LargeTiles large = large_tiles(M, w, count);
    fq_gemm_plan plan = {};
    if (fq_skinny_can(M, w[0].K)) {
        plan.few = fq_plan_skinny(M, w, count);
        if (M <= 16)
            return plan;
        const int K = w[0].K;
        const bool narrow = plan.few.s_log2 < 2;
        double level = 0.97;
        if (K <= 1280 && plan.few.mb == 1)
            level = narrow ? 1.02 : 0.97;
        else if (K <= 1280)
            level = K <= 256 ? 1.3 : (K <= 512 ? 1.2 : (narrow ? 1.1 : 1.03));
        if (plan.few.us < level * large.us)
            return plan;
    }
    plan.row_tiles = tall_row_tiles(M, w, count, large);
    plan.tile_rows = plan.row_tiles ? 256 : 128;
    plan.height = plan.row_tiles ? highest_rows(M, plan.row_tiles) : 128;
    return plan;
}

int fq_launch_gemm(const void *x, int M, const fq_packed_ref &w, void *out, fq_stream st, int tile_rows)
{
    const size_t Np = ((size_t)w.N + 63) / 64 * 64;
    if (!fits_32bit(M, w.K, 2) || Np / 8 * w.K * w.bits >= ((size_t)1 << 32))
        return (int)hipErrorInvalidValue;
    fq_gemm_plan plan = {};
    if (tile_rows == 0) {
        plan = fq_plan_gemm(M, &w, 1);
        tile_rows = plan.tile_rows;
    }
    if (tile_rows == 0)
        return fq_launch_skinny(x, M, &w, &out, 1, plan.few, st);
    if (tile_rows == 256)
        return launch_tall(x, M, &w, &out, 1, st, plan.row_tiles);
    if (w.ld && w.ld != w.N) // a column range of a wider output: the multi-matrix kernel carries the row pitch
        return fq_launch_gemm_multi(x, M, &w, &out, 1, st, 128);
    switch (w.bits) {
    case 2: return launch_q<2>(x, M, w, out, st);
    case 3: return launch_q<3>(x, M, w, out, st);
    case 4: return launch_q<4>(x, M, w, out, st);
    default: return launch_q<8>(x, M, w, out, st);
    }
}

// Matrices that share x (same K): one launch.  Shapes are validated by the caller like fq_launch_gemm's.
int fq_launch_gemm_multi(const void *x, int M, const fq_packed_ref *w, void *const *outs, int count, fq_stream st,
                         int tile_rows)
{
    if (count < 1 || count > 3)
        return (int)hipErrorInvalidValue;
    for (int i = 0; i < count; ++i) {
        const size_t Np = ((size_t)w[i].N + 63) / 64 * 64;
        if (w[i].K != w[0].K || !fits_32bit(M, w[i].K, 2) || Np / 8 * w[i].K * w[i].bits >= ((size_t)1 << 32))
            return (int)hipErrorInvalidValue;
    }
    fq_gemm_plan plan = {};
    if (tile_rows == 0) {
        plan = fq_plan_gemm(M, w, count);
        tile_rows = plan.tile_rows;
    }
    if (tile_rows == 0)
        return fq_launch_skinny(x, M, w, outs, count, plan.few, st);
    if (tile_rows == 256)
        return launch_tall(x, M, w, outs, count, st, plan.row_tiles);
    auto qnb = [&](int i) { return (w[i].bits == 2 || w[i].bits == 4) && wide_tiles_pay(M, w[i].N) ? 4 : 2; };
    const GemmLaunch l(w, outs, count, [&](int i) { return ((w[i].N + 64 * qnb(i) - 1) / (64 * qnb(i))) * ((M + QBM - 1) / QBM); }, qnb);
    hipLaunchKernelGGL(qgemm_multi_kernel, dim3(8 * ((l.total + 7) / 8)), dim3(256), 0, st,
                       static_cast<const _Float16 *>(x), M, w[0].K, l.total, l.first[1], l.first[2], l.jobs);
    return (int)hipGetLastError();
}

int fq_launch_dense(const void *x, int M, const void *W, int N, int K, void *out, fq_stream st)
{
    if (!fits_32bit(M, K, 2) || !fits_32bit(N, K, 2))
        return (int)hipErrorInvalidValue;
    return launch_tile<DENSE, 2>(x, M, W, nullptr, nullptr, N, K, out, st);
}
