// Row-wise kernels: the glue between the linears of the synthetic block, the
// dense dump of a packed matrix, and the fused log-softmax cross-entropy that
// turns head logits into the per-token loss behind the perplexity score
// (FlexQuant, arXiv 2501.07139, Algorithm 1, calibrationEval).  All are
// bandwidth-bound: one pass over their inputs with 128-bit loads.
#include "fq_device.h"
#include "fq_internal.h"
#include "fq_lse.h"

namespace {

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// ------------------------------------------------------------------ glue
// One workgroup of 256 threads per row; the row lives in registers between the
// sum-of-squares pass and the scaling pass (H <= 256*8*MAXC halves).
constexpr int GLUE_MAXC = 8;

template <int OP>
__global__ __launch_bounds__(256) void glue_kernel(const _Float16 *__restrict__ a, const _Float16 *__restrict__ b,
                                                   const _Float16 *__restrict__ c, int H,
                                                   _Float16 *__restrict__ out)
{
    const size_t row = (size_t)blockIdx.x * H;
    const int chunks = H >> 3;
    float t[GLUE_MAXC][8];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < GLUE_MAXC; ++i) {
        const int ch = threadIdx.x + 256 * i;
        if (ch < chunks) {
            const h8 va = *reinterpret_cast<const h8 *>(a + row + ch * 8);
            h8 vb = va, vc = va;
            if constexpr (OP != 0)
                vb = *reinterpret_cast<const h8 *>(b + row + ch * 8);
            if constexpr (OP == 1)
                vc = *reinterpret_cast<const h8 *>(c + row + ch * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v;
                if constexpr (OP == 0)
                    v = (float)va[e];
                else if constexpr (OP == 1)
                    v = (float)va[e] + (float)vb[e] + (float)vc[e];
                else if constexpr (OP == 2 || OP == 4)
                    v = (float)va[e] + (float)vb[e];
                else {
                    const float g = (float)va[e];
                    v = g / (1.0f + __expf(-g)) * (float)vb[e];
                }
                t[i][e] = v;
                ss += v * v;
            }
        }
    }
    float inv = 1.0f;
    if constexpr (OP != 2 && OP != 5) { // 2 and 5 have no norm
        __shared__ float part[4];
        ss = wave_sum(ss);
        if ((threadIdx.x & 63) == 0)
            part[threadIdx.x >> 6] = ss;
        __syncthreads();
        ss = part[0] + part[1] + part[2] + part[3];
        inv = 1.0f / sqrtf(ss / (float)H + 1e-5f);
    }
#pragma unroll
    for (int i = 0; i < GLUE_MAXC; ++i) {
        const int ch = threadIdx.x + 256 * i;
        if (ch < chunks) {
            h8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                o[e] = (_Float16)(t[i][e] * inv);
            *reinterpret_cast<h8 *>(out + row + ch * 8) = o;
        }
    }
}

// Two consecutive row-wise steps of the block in one pass (where they are launches of their own), each rounded to fp16 where the separate
// kernels would store it, so the values are those of the two calls:
//   OP 6: aux = a + b,       out = rms(aux)     the residual after the output projection and the FFN's input
//   OP 7: aux = rms(a + b),  out = rms(aux)     a block's output and the next block's first normalisation
template <int OP>
__global__ __launch_bounds__(256) void glue2_kernel(const _Float16 *__restrict__ a, const _Float16 *__restrict__ b, int H,
                                                    _Float16 *__restrict__ aux, _Float16 *__restrict__ out)
{
    const size_t row = (size_t)blockIdx.x * H;
    const int chunks = H >> 3;
    __shared__ float part[2][4];
    auto row_sum = [&](float ss, int which) {
        ss = wave_sum(ss);
        if ((threadIdx.x & 63) == 0)
            part[which][threadIdx.x >> 6] = ss;
        __syncthreads();
        return part[which][0] + part[which][1] + part[which][2] + part[which][3];
    };
    float t[GLUE_MAXC][8];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < GLUE_MAXC; ++i) {
        const int ch = threadIdx.x + 256 * i;
        if (ch < chunks) {
            const h8 va = *reinterpret_cast<const h8 *>(a + row + ch * 8), vb = *reinterpret_cast<const h8 *>(b + row + ch * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = (float)va[e] + (float)vb[e];
                if constexpr (OP == 6)
                    v = (float)(_Float16)v; // the stored sum is what the norm reads
                t[i][e] = v;
                ss += v * v;
            }
        }
    }
    if constexpr (OP == 7) { // first norm; its rounded result is the second one's input
        const float inv = 1.0f / sqrtf(row_sum(ss, 0) / (float)H + 1e-5f);
        ss = 0.f;
#pragma unroll
        for (int i = 0; i < GLUE_MAXC; ++i)
            if (threadIdx.x + 256 * i < chunks) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = (float)(_Float16)(t[i][e] * inv);
                    t[i][e] = v;
                    ss += v * v;
                }
            }
    }
    const float inv = 1.0f / sqrtf(row_sum(ss, 1) / (float)H + 1e-5f);
#pragma unroll
    for (int i = 0; i < GLUE_MAXC; ++i) {
        const int ch = threadIdx.x + 256 * i;
        if (ch < chunks) {
            h8 x, o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] = (_Float16)t[i][e]; // exact: already an fp16 value
                o[e] = (_Float16)(t[i][e] * inv);
            }
            *reinterpret_cast<h8 *>(aux + row + ch * 8) = x;
            *reinterpret_cast<h8 *>(out + row + ch * 8) = o;
        }
    }
}

// ------------------------------------------------------------------- NLL
// How a row of V logits is read (base pointers are 16-byte aligned, so a row is only if V % 8 == 0): in chunks of eight; in
// chunks from its first aligned element on, with up to seven elements before and behind them; or element by element.
enum RowMode { ROW_ALIGNED, ROW_ANY, ROW_ELEMENTS };

// Up to 512 elements are two loads a thread: the ends of a row that is not aligned would take as long (500 logits, 2048 rows:
// distance 3.1 us, 3.3 with chunks; 1001 logits 3.4 and 3.3).
RowMode row_mode(int V) { return (V & 7) == 0 ? ROW_ALIGNED : (V <= 512 ? ROW_ELEMENTS : ROW_ANY); }

template <RowMode MODE>
struct RowSpan {
    int head, chunks; // elements before the first chunk; chunks
    __device__ __forceinline__ RowSpan(int row, int V)
    {
        head = MODE == ROW_ANY ? min((int)((8u - (uint32_t)(((uint64_t)row * (uint64_t)V) & 7u)) & 7u), V) : 0;
        chunks = MODE == ROW_ELEMENTS ? 0 : (V - head) >> 3;
    }
    // use(i) for the elements outside the chunks: fewer than sixteen, one a thread, or all of the row
    template <int THREADS, class F>
    __device__ __forceinline__ void ends(int V, F &&use) const
    {
        if constexpr (MODE == ROW_ELEMENTS) {
            for (int i = threadIdx.x; i < V; i += THREADS)
                use(i);
        } else if constexpr (MODE == ROW_ANY) {
            const int i = threadIdx.x, e = i < head ? i : i + 8 * chunks;
            if (i < 16 && e < V)
                use(e);
        }
    }
};

// Chunks a thread loads before it uses the first, where a row has more than two a thread.  The last trip takes the loads it has
// no chunk for from the row's last one: with a loop of whole trips and another for the rest, the lanes of one wavefront
// part and it runs both, the rest load by load (loss of 2048 x 8000 logits 11.4 -> 9.9 us, 300 x 32000 9.7 -> 8.9; two chunks
// 10.4 and 9.3).  Shorter rows gain nothing by it (loss of 512 x 4096 logits 3.6 us against 3.45).
constexpr int ROW_UNROLL = 4;

// One workgroup per token row; each thread keeps a running (max, sum of
// exp(l - max)) over its 16-byte chunks, then the pairs are merged across the
// wavefront and the workgroup.  The label's logit is read directly.  Bound by the read; few rows take large
// workgroups (THREADS), so that the loads of a row are under way together.
// Measured (us): 2048 x 32000 27; 2048 x 31001, whose rows are not aligned, 27 (element by element 71).
template <int THREADS, RowMode MODE>
__global__ __launch_bounds__(THREADS) void nll_kernel(const _Float16 *__restrict__ logits,
                                                      const int32_t *__restrict__ labels, int V,
                                                      float *__restrict__ nll)
{
    const int row = blockIdx.x;
    const int label = labels[row];
    if (label < 0 || label >= V) { // uniform across the workgroup
        if (threadIdx.x == 0)
            nll[row] = 0.f;
        return;
    }
    const _Float16 *l = logits + (size_t)row * V;
    const RowSpan<MODE> span(row, V);
    const h8 *chunk = reinterpret_cast<const h8 *>(l + span.head);
    float mx = -INFINITY, se = 0.f;
    auto add = [&](h8 v) {
        float e8[8], cm, cs;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            e8[e] = (float)v[e];
        lse_pair(e8, cm, cs);
        lse_merge(mx, se, cm, cs);
    };
    if (span.chunks <= 2 * THREADS) {
        for (int ch = threadIdx.x; ch < span.chunks; ch += THREADS)
            add(chunk[ch]);
    } else {
        for (int ch = threadIdx.x; ch < span.chunks; ch += ROW_UNROLL * THREADS) {
            h8 v[ROW_UNROLL];
#pragma unroll
            for (int i = 0; i < ROW_UNROLL; ++i)
                v[i] = chunk[min(ch + i * THREADS, span.chunks - 1)];
#pragma unroll
            for (int i = 0; i < ROW_UNROLL; ++i)
                if (ch + i * THREADS < span.chunks)
                    add(v[i]);
        }
    }
    span.template ends<THREADS>(V, [&](int i) {
        const float e = (float)l[i]; // lse_pair of one logit: 1, or 0 for -inf, or NaN
        lse_merge(mx, se, fmaxf(e, LSE_FLOOR), e == -INFINITY ? 0.f : (e - e) + 1.f);
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(mx, o, 64), s2 = __shfl_xor(se, o, 64);
        lse_merge(mx, se, m2, s2);
    }
    constexpr int WAVES = THREADS / 64;
    __shared__ float pm[WAVES], ps[WAVES];
    if ((threadIdx.x & 63) == 0) {
        pm[threadIdx.x >> 6] = mx;
        ps[threadIdx.x >> 6] = se;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = pm[0], s = ps[0];
        for (int w = 1; w < WAVES; ++w)
            lse_merge(m, s, pm[w], ps[w]);
        nll[row] = logf(s) + (m - (float)l[label]); // difference first: exact for fp16 inputs
    }
}

// --------------------------------------------------------------- dequant
// Dense dump of a packed matrix, one thread per (sixteen-row block, group, lane)
// chunk: reads the format literally (integer field extraction), then
// float(scale) * (float(code) - float(zero)) with both steps rounded to fp32.
template <int BITS>
__global__ __launch_bounds__(64) void dequant_kernel(const uint32_t *__restrict__ packed,
                                                     const _Float16 *__restrict__ scales,
                                                     const _Float16 *__restrict__ zeros, int N, int K,
                                                     void *__restrict__ out, int out_is_fp16)
{
    constexpr int SUB = Fmt<BITS>::SUB;
    const int G = K >> 7;
    const int g = blockIdx.x, rb16 = blockIdx.y, lane = threadIdx.x;
    const int r = lane & 15, c = lane >> 4;
    const int n = rb16 * 16 + r;
    const uint32_t *tile = packed + ((size_t)(rb16 / SUB) * G + g) * tile_dwords<BITS>();
    uint32_t C[BITS];
    load_chunk<BITS>(tile, rb16 % SUB, lane, C);
    const size_t meta = ((size_t)rb16 * G + g) * 16 + r;
    const float z = (float)zeros[meta], sc = (float)scales[meta];
    if (n >= N)
        return;
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        const int s = t >> 3, e = t & 7;
        const int k = g * 128 + 32 * s + 8 * c + e;
        const float d = __fsub_rn((float)code_at<BITS>(C, t), z);
        const float w = __fmul_rn(sc, d);
        if (out_is_fp16)
            static_cast<_Float16 *>(out)[(size_t)n * K + k] = (_Float16)w;
        else
            static_cast<float *>(out)[(size_t)n * K + k] = w;
    }
}

} // namespace

int fq_launch_glue(int op, const void *a, const void *b, const void *c, int M, int H, void *out, fq_stream st)
{
    dim3 grid(M), block(256);
    const _Float16 *pa = static_cast<const _Float16 *>(a), *pb = static_cast<const _Float16 *>(b),
                   *pc = static_cast<const _Float16 *>(c);
    _Float16 *po = static_cast<_Float16 *>(out);
    switch (op) {
    case 0: hipLaunchKernelGGL(glue_kernel<0>, grid, block, 0, st, pa, pb, pc, H, po); break;
    case 1: hipLaunchKernelGGL(glue_kernel<1>, grid, block, 0, st, pa, pb, pc, H, po); break;
    case 2: hipLaunchKernelGGL(glue_kernel<2>, grid, block, 0, st, pa, pb, pc, H, po); break;
    case 3: hipLaunchKernelGGL(glue_kernel<3>, grid, block, 0, st, pa, pb, pc, H, po); break;
    case 4: hipLaunchKernelGGL(glue_kernel<4>, grid, block, 0, st, pa, pb, pc, H, po); break;
    default: hipLaunchKernelGGL(glue_kernel<5>, grid, block, 0, st, pa, pb, pc, H, po); break;
    }
    return (int)hipGetLastError();
}

int fq_launch_glue2(int op, const void *a, const void *b, int M, int H, void *aux, void *out, fq_stream st)
{
    dim3 grid(M), block(256);
    const _Float16 *pa = static_cast<const _Float16 *>(a), *pb = static_cast<const _Float16 *>(b);
    if (op == 6)
        hipLaunchKernelGGL(glue2_kernel<6>, grid, block, 0, st, pa, pb, H, static_cast<_Float16 *>(aux), static_cast<_Float16 *>(out));
    else
        hipLaunchKernelGGL(glue2_kernel<7>, grid, block, 0, st, pa, pb, H, static_cast<_Float16 *>(aux), static_cast<_Float16 *>(out));
    return (int)hipGetLastError();
}

// Workgroup size of the two row kernels: up to one row a CU, 1024 threads bring more loads of a long row under way (32000
// logits, 256 rows: distance 8.3 -> 6.4 us, loss 9.4 -> 6.7; 384 rows: level); shorter rows only pay for the larger
// reduction (loss of 8192 logits 3.8 -> 4.3 us, of 16384 level; the distance reads two rows: 8192 logits 3.2 -> 3.05).
static bool wide_rows(int M, int V, int longer) { return M <= 256 && V >= longer; }

// Row-wise Euclidean distance between two logit arrays (sensitivity analysis of the search, Section
// "Efficient Design Space Navigation").  One workgroup per row, one pass over both rows with 128-bit loads; differences and
// squares in fp32, four partial sums per thread, then a fixed-order reduction.  The two rows start at the same distance
// from a 16-byte boundary.  Measured (us): 2048 x 32000 43, 2048 x 31001 41 (element by element 70).
namespace {
template <int THREADS, RowMode MODE>
__global__ __launch_bounds__(THREADS) void logit_l2_kernel(const _Float16 *__restrict__ a, const _Float16 *__restrict__ b,
                                                           int V, float *__restrict__ dist)
{
    const int row = blockIdx.x;
    const _Float16 *ra = a + (size_t)row * V, *rb = b + (size_t)row * V;
    const RowSpan<MODE> span(row, V);
    const h8 *ca = reinterpret_cast<const h8 *>(ra + span.head), *cb = reinterpret_cast<const h8 *>(rb + span.head);
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    auto add = [&](h8 va, h8 vb) {
        float d[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            d[e] = (float)va[e] - (float)vb[e];
        s0 = fmaf(d[0], d[0], s0); s1 = fmaf(d[1], d[1], s1); s2 = fmaf(d[2], d[2], s2); s3 = fmaf(d[3], d[3], s3);
        s0 = fmaf(d[4], d[4], s0); s1 = fmaf(d[5], d[5], s1); s2 = fmaf(d[6], d[6], s2); s3 = fmaf(d[7], d[7], s3);
    };
    // two loads a chunk: with small workgroups, several on a CU, more in flight gain nothing up to 16384 logits (1024 x 8192
    // 5.6 us, 6.1 with four trips' loads at once; 300 x 32000 8.9 and 7.9)
    if (span.chunks <= (THREADS == 256 && MODE == ROW_ALIGNED ? 8 : 2) * THREADS) {
        for (int ch = threadIdx.x; ch < span.chunks; ch += THREADS)
            add(ca[ch], cb[ch]);
    } else {
        for (int ch = threadIdx.x; ch < span.chunks; ch += ROW_UNROLL * THREADS) {
            h8 va[ROW_UNROLL], vb[ROW_UNROLL];
#pragma unroll
            for (int i = 0; i < ROW_UNROLL; ++i) {
                const int at = min(ch + i * THREADS, span.chunks - 1);
                va[i] = ca[at];
                vb[i] = cb[at];
            }
#pragma unroll
            for (int i = 0; i < ROW_UNROLL; ++i)
                if (ch + i * THREADS < span.chunks)
                    add(va[i], vb[i]);
        }
    }
    span.template ends<THREADS>(V, [&](int i) {
        const float d = (float)ra[i] - (float)rb[i];
        s0 = fmaf(d, d, s0);
    });
    float ss = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        ss += __shfl_xor(ss, o, 64);
    constexpr int WAVES = THREADS / 64;
    __shared__ float part[WAVES];
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) {
        float sum = 0.f;
        for (int w = 0; w < WAVES; ++w)
            sum += part[w];
        dist[row] = sqrtf(sum);
    }
}
} // namespace

// [256 or 1024 threads][RowMode]; rows read element by element are never long enough for the larger workgroups
typedef void (*L2Kernel)(const _Float16 *, const _Float16 *, int, float *);
typedef void (*NllKernel)(const _Float16 *, const int32_t *, int, float *);
static const L2Kernel l2_kernels[2][3] = {
    {logit_l2_kernel<256, ROW_ALIGNED>, logit_l2_kernel<256, ROW_ANY>, logit_l2_kernel<256, ROW_ELEMENTS>},
    {logit_l2_kernel<1024, ROW_ALIGNED>, logit_l2_kernel<1024, ROW_ANY>, nullptr}};
static const NllKernel nll_kernels[2][3] = {
    {nll_kernel<256, ROW_ALIGNED>, nll_kernel<256, ROW_ANY>, nll_kernel<256, ROW_ELEMENTS>},
    {nll_kernel<1024, ROW_ALIGNED>, nll_kernel<1024, ROW_ANY>, nullptr}};

template <class Kernel, class... Args>
static void launch_rows(const Kernel (&kernels)[2][3], int M, int V, bool wide, fq_stream st, Args... args)
{
    hipLaunchKernelGGL(kernels[wide][row_mode(V)], dim3(M), dim3(wide ? 1024 : 256), 0, st, args...);
}

int fq_launch_logit_l2(const void *a, const void *b, int M, int V, float *dist, fq_stream st)
{
    const _Float16 *pa = static_cast<const _Float16 *>(a), *pb = static_cast<const _Float16 *>(b);
    launch_rows(l2_kernels, M, V, wide_rows(M, V, 8192), st, pa, pb, V, dist);
    return (int)hipGetLastError();
}

int fq_launch_nll(const void *logits, const int32_t *labels, int M, int V, float *nll, fq_stream st)
{
    const _Float16 *l = static_cast<const _Float16 *>(logits);
    launch_rows(nll_kernels, M, V, wide_rows(M, V, 16384), st, l, labels, V, nll);
    return (int)hipGetLastError();
}

int fq_launch_dequant(const fq_packed_ref &w, void *out, int out_is_fp16, fq_stream st)
{
    const int Np16 = (w.N + 63) / 64 * 4;
    dim3 grid(w.K >> 7, Np16), block(64);
    const uint32_t *p = static_cast<const uint32_t *>(w.packed);
    const _Float16 *s = static_cast<const _Float16 *>(w.scales), *z = static_cast<const _Float16 *>(w.zeros);
    switch (w.bits) {
    case 2: hipLaunchKernelGGL(dequant_kernel<2>, grid, block, 0, st, p, s, z, w.N, w.K, out, out_is_fp16); break;
    case 3: hipLaunchKernelGGL(dequant_kernel<3>, grid, block, 0, st, p, s, z, w.N, w.K, out, out_is_fp16); break;
    case 4: hipLaunchKernelGGL(dequant_kernel<4>, grid, block, 0, st, p, s, z, w.N, w.K, out, out_is_fp16); break;
    default: hipLaunchKernelGGL(dequant_kernel<8>, grid, block, 0, st, p, s, z, w.N, w.K, out, out_is_fp16); break;
    }
    return (int)hipGetLastError();
}

// ------------------------------------------------------------ streaming read
// Reads `bytes` once with 128-bit loads, eight independent loads per lane and round, and keeps one word
// per workgroup: what a kernel that does nothing but read reaches on this device, the practical ceiling
// beside which the decode path's bytes per second are reported (Section "Introduction": single-batch
// decoding streams every weight once per token and is bound by that).
namespace {
__global__ __launch_bounds__(256) void stream_read_kernel(const u4v *__restrict__ src, size_t n16, uint32_t *sink)
{
    const size_t stride = (size_t)gridDim.x * 256;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    u4v acc = {0u, 0u, 0u, 0u};
    for (; i + 7 * stride < n16; i += 8 * stride) {
        u4v v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            v[k] = __builtin_nontemporal_load(src + i + k * stride);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            acc ^= v[k];
    }
    for (; i < n16; i += stride)
        acc ^= __builtin_nontemporal_load(src + i);
    uint32_t w = acc.x ^ acc.y ^ acc.z ^ acc.w;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        w ^= __shfl_xor(w, o, 64);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0)
        sink[blockIdx.x] = part[0] ^ part[1] ^ part[2] ^ part[3];
}
} // namespace

int fq_launch_stream_read(const void *src, size_t bytes, uint32_t *sink, int blocks, fq_stream st)
{
    hipLaunchKernelGGL(stream_read_kernel, dim3(blocks), dim3(256), 0, st, static_cast<const u4v *>(src), bytes / 16, sink);
    return (int)hipGetLastError();
}

