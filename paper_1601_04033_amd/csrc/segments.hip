// B-FASGD as the paper states it: one transmit decision per push from v
// averaged over all parameters (Sec. 2.3), or one per tensor segment from
// that segment's mean (the per-tensor direction of Sec. 5), and the server
// apply of a push decided that way.
//
// Segments are handled in groups of up to kSegGroup whose offsets and block
// counts travel in the kernel arguments, so the host never copies to the
// device.  A group is as large as its offsets fit the kernel arguments (2 KB
// of 4): a server with 100 tensors decides in two launches and applies in
// one.  Every segment is cut into blocks:
//   seg_partial  one fp64 partial sum of v per block of kSegSpan parameters,
//                in a fixed order;
//   seg_decide   one block of 1024 threads per segment folds its partials in
//                a fixed order, divides by the length and decides in fp64;
//   seg_apply    the FASGD update on the blocks of transmitted segments.
// Sums are deterministic run to run (fixed assignment and reduction order).
#include "kernels.hpp"

namespace fasgd {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kThreads = 256;
constexpr int kPerThread = 16;                         // 4 vectors of 4
constexpr int64_t kSegSpan = int64_t(kThreads) * kPerThread;

// The segment of the group that block b belongs to (wave-uniform; every lane
// of the wave calls): the number of segments whose blocks all come before b.
// A walk over the prefixes for a few segments; beyond, the wave compares 64
// of them at a time (the walk's dependent scalar loads cost about as much as
// the block's own work at 100 segments).
constexpr int kWalkSegments = 8;
__device__ __forceinline__ int segment_of(const SegGroup& g, int64_t b)
{
    int i = 0;
    if (g.n <= kWalkSegments) {
        while (i + 1 < g.n && b >= g.block_prefix[i + 1]) ++i;
        return i;
    }
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int k = 0; k < kSegGroup; k += kWave) {
        if (k + 1 < g.n) {
            const int at = k + lane + 1;
            i += __popcll(__builtin_amdgcn_ballot_w64(at < g.n && b >= g.block_prefix[at < g.n ? at : 0]));
        }
    }
    return i;
}

// block b of the group -> (segment i of the group, first parameter, end)
__device__ __forceinline__ void block_range(const SegGroup& g, int64_t b, int& i, int64_t& lo, int64_t& hi)
{
    i = segment_of(g, b);
    lo = g.start[i] + (b - g.block_prefix[i]) * kSegSpan;
    hi = lo + kSegSpan < g.start[i + 1] ? lo + kSegSpan : g.start[i + 1];
}

constexpr int kDecideThreads = 1024;   // one block folds a segment's partials
constexpr int kDecideAcc = 4;          // independent accumulators per thread
static_assert(kDecideAcc == 4, "the fold below combines four sums");

template <int THREADS>
__device__ __forceinline__ double block_sum(double x)
{
    __shared__ double wave_sum[THREADS / kWave];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) x += __shfl_xor(x, d, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) wave_sum[threadIdx.x / kWave] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < THREADS / kWave; ++w) s += wave_sum[w];
    return s;
}

__global__ __launch_bounds__(kThreads) void seg_partial(const SegGroup g, const float* __restrict__ v,
                                                        double* __restrict__ partial)
{
    int i;
    int64_t lo, hi;
    block_range(g, blockIdx.x, i, lo, hi);
    double acc = 0.0;
    if ((lo & 3) == 0 && (reinterpret_cast<uintptr_t>(v) & 15) == 0 && hi - lo == kSegSpan) {
#pragma unroll
        for (int k = 0; k < kPerThread / 4; ++k) {
            const f4 x = __builtin_nontemporal_load(reinterpret_cast<const f4*>(v + lo) + k * kThreads + threadIdx.x);
            acc += static_cast<double>(x[0]) + static_cast<double>(x[1]) + static_cast<double>(x[2]) +
                   static_cast<double>(x[3]);
        }
    } else {
        // every load of the span before the first sum
        float x[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int64_t j = lo + threadIdx.x + k * kThreads;
            x[k] = j < hi ? v[j] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) acc += static_cast<double>(x[k]);
    }
    const double s = block_sum<kThreads>(acc);
    if (threadIdx.x == 0) partial[g.partial_base + blockIdx.x] = s;
}

__global__ __launch_bounds__(kDecideThreads) void seg_decide(const SegGroup g, const double* __restrict__ partial,
                                                       float c, float eps_c, uint32_t key0, uint32_t key1,
                                                       uint32_t ctr_T, uint32_t ctr_client,
                                                       uint8_t* __restrict__ transmit)
{
    const int i = blockIdx.x;
    // thread t folds partials t, t + 1024, ... into kDecideAcc running sums
    // (loads of one round issued together), then the sums in a fixed order
    double acc[kDecideAcc] = {0.0, 0.0, 0.0, 0.0};
    const int64_t end = g.block_prefix[i + 1];
    for (int64_t b = g.block_prefix[i] + threadIdx.x; b < end; b += kDecideAcc * kDecideThreads) {
#pragma unroll
        for (int q = 0; q < kDecideAcc; ++q) {
            const int64_t bq = b + q * kDecideThreads;
            if (bq < end) acc[q] += partial[g.partial_base + bq];
        }
    }
    const double sum = block_sum<kDecideThreads>((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if (threadIdx.x == 0) {
        const int64_t s = g.first_seg + i;
        const double mean = sum / static_cast<double>(g.start[i + 1] - g.start[i]);
        const uint4 w = philox4x32_10(
            make_uint4(static_cast<uint32_t>(s), 0x80000000u | static_cast<uint32_t>(static_cast<uint64_t>(s) >> 32),
                       ctr_T, ctr_client),
            key0, key1);
        const double r = static_cast<double>(w.x >> 8) * 0x1p-24;
        const double t = mean + static_cast<double>(eps_c);
        const double u = t + static_cast<double>(c);
        transmit[s] = fma(r, u, -t) < 0.0 ? 1 : 0;
    }
}

// The FASGD update on a block of VECS x 256 chunks of 4 parameters (chunks at
// multiples of 4 of the parameter index, so every segment's inside is read in
// 16-byte vectors wherever it starts), every load of the block before the
// first update.  Bound by HBM (40 bytes per parameter of a sent segment).
// A state that the L2 caches hold (kStreamBytes) takes 4 parameters per
// thread and plain stores, as the next call reads it again; a larger one 16
// per thread and non-temporal accesses.  Measured against one loop of 4
// chunks per thread, loads and stores alternating, one parameter at a time
// where a segment starts off a multiple of 4 (decision and apply together,
// same box): 25M in 16 segments 220 -> 188 us, 40M whole 334 -> 306, 5M in
// 50 79.7 -> 64.6, the MLP's 6 tensors 21.6 -> 20.2, 300k in 6 14.4 -> 13.8
// (15.2 in the streaming form; the MLP 21.0 in the other).  Only these two of
// the four combinations were timed.
constexpr int64_t kStreamBytes = int64_t(32) << 20;   // the eight L2 caches together
typedef int i4 __attribute__((ext_vector_type(4)));

template <bool STREAM, typename T>
__device__ __forceinline__ T load(const T* p)
{
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}
template <bool STREAM, typename T>
__device__ __forceinline__ void store(T x, T* p)
{
    if (STREAM)
        __builtin_nontemporal_store(x, p);
    else
        *p = x;
}

template <int MODE, int VECS, bool STREAM>
__global__ __launch_bounds__(kThreads) void seg_apply(const SegGroup g, const SegApplyArgs a)
{
    constexpr int64_t kChunks = int64_t(kThreads) * VECS;
    const int64_t blk = blockIdx.x;
    const int i = segment_of(g, blk);
    if (!a.transmit[g.first_seg + i]) return;
    const int64_t lo = g.start[i], hi = g.start[i + 1];
    const int64_t q0 = (lo >> 2) + (blk - g.block_prefix[i]) * kChunks;   // the block's first chunk
    const Hyper h = a.h;
    const int32_t T = a.last_T_value;
    if (a.aligned && q0 * 4 >= lo && (q0 + kChunks) * 4 <= hi) {
        f4 th[VECS], n[VECS], b[VECS], v[VECS], gr[VECS];
#pragma unroll
        for (int k = 0; k < VECS; ++k) {
            const int64_t o = (q0 + k * kThreads + threadIdx.x) * 4;
            th[k] = load<STREAM>(reinterpret_cast<const f4*>(a.theta + o));
            n[k] = load<STREAM>(reinterpret_cast<const f4*>(a.n + o));
            b[k] = load<STREAM>(reinterpret_cast<const f4*>(a.b + o));
            v[k] = load<STREAM>(reinterpret_cast<const f4*>(a.v + o));
            gr[k] = load<true>(reinterpret_cast<const f4*>(a.grad + o));
        }
#pragma unroll
        for (int k = 0; k < VECS; ++k) {
            const int64_t o = (q0 + k * kThreads + threadIdx.x) * 4;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                float t = th[k][cc], nn = n[k][cc], bb = b[k][cc], vv = v[k][cc];
                fasgd_step<MODE>(t, nn, bb, vv, gr[k][cc], a.coef, h);
                th[k][cc] = t; n[k][cc] = nn; b[k][cc] = bb; v[k][cc] = vv;
            }
            store<STREAM>(th[k], reinterpret_cast<f4*>(a.theta + o));
            store<STREAM>(n[k], reinterpret_cast<f4*>(a.n + o));
            store<STREAM>(b[k], reinterpret_cast<f4*>(a.b + o));
            store<STREAM>(v[k], reinterpret_cast<f4*>(a.v + o));
            store<STREAM>(i4{T, T, T, T}, reinterpret_cast<i4*>(a.last_T + o));
        }
        return;
    }
    // a block that reaches past its segment (its first and last), or arrays
    // that are only 4-byte aligned: one parameter per lane, 4 at a time
#pragma unroll
    for (int k = 0; k < VECS; ++k) {
        float th[4], n[4], b[4], v[4], gr[4];
        const int64_t j0 = (q0 + k * kThreads) * 4 + threadIdx.x;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = j0 + u * kThreads;
            if (j >= lo && j < hi) { th[u] = a.theta[j]; n[u] = a.n[j]; b[u] = a.b[j]; v[u] = a.v[j]; gr[u] = a.grad[j]; }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = j0 + u * kThreads;
            if (j >= lo && j < hi) {
                fasgd_step<MODE>(th[u], n[u], b[u], v[u], gr[u], a.coef, h);
                a.theta[j] = th[u]; a.n[j] = n[u]; a.b[j] = b[u]; a.v[j] = v[u];
                a.last_T[j] = T;
            }
        }
    }
}

// seg_apply with the group's blocks counted in its own shape.
template <int MODE, int VECS, bool STREAM>
void launch_apply_shape(SegGroup& g, const SegApplyArgs& a, hipStream_t s)
{
    constexpr int64_t kChunks = int64_t(kThreads) * VECS;
    int64_t blocks = 0;
    for (int i = 0; i < g.n; ++i) {
        g.block_prefix[i] = blocks;
        blocks += (((g.start[i + 1] + 3) >> 2) - (g.start[i] >> 2) + kChunks - 1) / kChunks;
    }
    g.block_prefix[g.n] = blocks;
    seg_apply<MODE, VECS, STREAM><<<static_cast<unsigned>(blocks), kThreads, 0, s>>>(g, a);
}

template <int MODE>
void launch_apply(SegGroup& g, const SegApplyArgs& a, hipStream_t s)
{
    if (a.P * 20 > kStreamBytes)   // theta, n, b, v and last_T
        launch_apply_shape<MODE, 4, true>(g, a, s);
    else
        launch_apply_shape<MODE, 1, false>(g, a, s);
}

}  // namespace

int64_t seg_blocks(int64_t length) { return (length + kSegSpan - 1) / kSegSpan; }

size_t segments_workspace_bytes(int64_t P, int32_t S)
{
    const int64_t blocks = (P + kSegSpan - 1) / kSegSpan + S;
    return ((size_t(blocks) * sizeof(double)) + 255) & ~size_t(255);
}

hipError_t launch_seg_decide(const SegGroup& g, const float* v, double* partial, float c, float eps_c,
                             uint64_t seed, uint32_t ctr_T, uint32_t ctr_client, uint8_t* transmit,
                             hipStream_t s)
{
    const unsigned blocks = static_cast<unsigned>(g.block_prefix[g.n]);
    seg_partial<<<blocks, kThreads, 0, s>>>(g, v, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    seg_decide<<<static_cast<unsigned>(g.n), kDecideThreads, 0, s>>>(g, partial, c, eps_c, static_cast<uint32_t>(seed),
                                                              static_cast<uint32_t>(seed >> 32), ctr_T, ctr_client,
                                                              transmit);
    return hipGetLastError();
}

hipError_t launch_seg_apply(SegGroup& g, const SegApplyArgs& a, int variant, hipStream_t s)
{
    switch (variant) {
    case kernel_variant(MATH_FAST, 0): launch_apply<kernel_variant(MATH_FAST, 0)>(g, a, s); break;
    case kernel_variant(MATH_IEEE, 0): launch_apply<kernel_variant(MATH_IEEE, 0)>(g, a, s); break;
    case kernel_variant(MATH_FAST, 1): launch_apply<kernel_variant(MATH_FAST, 1)>(g, a, s); break;
    case kernel_variant(MATH_IEEE, 1): launch_apply<kernel_variant(MATH_IEEE, 1)>(g, a, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace fasgd
