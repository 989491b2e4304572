// B-FASGD push selection with deterministic ordered compaction, and the
// sparse server apply of the compacted list.
//
// Work is cut into wave tiles of kTileSegs segments of 64 chunks (one chunk is
// 4 consecutive parameters, one 16-byte vector).  Every wave owns one tile and
// never waits on another wave, so no launch has a block barrier in its
// streaming part.  Selection runs in three launches (calls of up to about 50M
// parameters: two, described at select_mark_totals):
//   mark     the wave loads its tile of v, draws one Philox4x32-10 call per
//            chunk (the counter is the global chunk index, so one call feeds
//            one vector of v), forms four ballots per segment (1 bit per
//            parameter), stores the tile's ballot words in one store and its
//            transmit count;
//   scan     one block per 1024 tiles scans their counts (offsets within the
//            group) and records the group total;
//   scatter  the wave sums the totals of the groups before its own, loads its
//            tile of gradients, reads its ballot words (scalar loads), places
//            every transmitted (index, value) pair in an LDS stage at the
//            popcount of the bits before it (ascending index order), and
//            writes the staged run at group position + tile offset in
//            contiguous stores.
// When the mark step ran inside the preceding dense pass (which leaves the
// ballot words but no tile counts), the scan counts each tile's ballot bits
// (in the two-launch range, a count launch does, for the direct scatter).
// Several pushes selected together run as one set of launches with the push
// as the grid's y index, each with its own gradient, counter words, output
// slice and workspace slice.
// The result depends only on (seed, T, client, v, grad), never on timing.
#include <string.h>

#include "kernels.hpp"

// v_writelane_b32: write a wave-uniform value into one lane of a VGPR.  The
// LLVM intrinsic is reached through its symbol name (this compiler has no
// clang builtin for it), so the backend still schedules it and handles its
// hazards as for any other instruction.
__device__ int amdgcn_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace fasgd {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kSelBlock = 256;                // 4 independent waves
constexpr int kWavesPerBlock = kSelBlock / kWave;
constexpr int kTileSegs = 4;                  // 64-chunk segments per wave tile
constexpr int kTileWords = 4 * kTileSegs;     // ballot words per tile
constexpr int64_t kChunksPerTile = int64_t(kTileSegs) * kWave;  // 256 chunks = 1024 parameters
constexpr int kScanBlock = 1024;              // tiles per scan group
constexpr int kMaxGroups = 4096;              // 2^31 parameters need 2048
constexpr int kEarlyGroups = 64;              // up to 64 groups: the scatter's EARLY form

__host__ __device__ inline int64_t n_chunks(int64_t P) { return (P + 3) / 4; }
int64_t n_tiles(int64_t P) { return (n_chunks(P) + kChunksPerTile - 1) / kChunksPerTile; }
size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

__device__ __forceinline__ uint64_t lanes_below(int lane)
{
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// The 4 values of chunk q, one load each; parameters at or past P read as
// NaN, which never transmits (mark) and is never written (scatter).
__device__ __forceinline__ f4 load_chunk(const float* p, int64_t q, int64_t P)
{
    const int64_t j = q * 4;
    f4 x;
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = (j + c < P) ? p[j + c] : __builtin_nanf("");
    return x;
}

// wave tile of this wave (wave-uniform)
__device__ __forceinline__ int64_t wave_tile()
{
    return static_cast<int64_t>(blockIdx.x) * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
}

// The arguments of push b of a batch: its gradient, counter words, list,
// count, list index and workspace slice.
__device__ __forceinline__ SelectArgs push_args(const SelectArgs& a0, const SelectBatch& bt, int b)
{
    if (b == 0) return a0;
    SelectArgs a = a0;
    a.grad = bt.grad[b];
    a.ctr_T = bt.ctr_T[b];
    a.ctr_client = bt.ctr_client[b];
    if (a0.out_idx) a.out_idx = a0.out_idx + b * bt.list_stride;
    if (a0.out_val) a.out_val = a0.out_val + b * bt.list_stride;
    a.d_count = a0.d_count + b;
    if (a0.seg_start) a.seg_start = a0.seg_start + b * bt.index_stride;
    const size_t off = b * bt.ws_stride;
    a.ballots = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(a0.ballots) + off);
    a.tile_count = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(a0.tile_count) + off);
    a.tile_offset = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(a0.tile_offset) + off);
    a.group_total = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(a0.group_total) + off);
    return a;
}

// Mark one tile and return its transmit count (wave-uniform).  FULL: the
// tile lies inside [0, P) and v is 16-byte aligned, so no lane needs a bounds
// check (every tile but the last).  STORE_COUNT: also store the count for the
// scan launch.
template <bool FULL, bool STORE_COUNT>
__device__ __forceinline__ uint32_t mark_tile(const SelectArgs& a, int64_t tile, int lane)
{
    const int64_t nch = n_chunks(a.P);
    const int64_t q0 = tile * kChunksPerTile + lane;
    // every load of the tile before any arithmetic
    f4 v[kTileSegs];
#pragma unroll
    for (int s = 0; s < kTileSegs; ++s) {
        const int64_t q = q0 + s * kWave;
        if (FULL)
            v[s] = *reinterpret_cast<const f4*>(a.v + q * 4);
        else if (q < nch)
            v[s] = load_chunk(a.v, q, a.P);
    }
    // lane k < kTileWords holds ballot word k of the tile (low, high halves)
    int word_lo = 0, word_hi = 0;
    uint32_t count = 0;
#pragma unroll
    for (int s = 0; s < kTileSegs; ++s) {
        const int64_t q = q0 + s * kWave;
        uint32_t nib = 0;
        if (FULL || q < nch) {
            const uint64_t qg = a.chunk_base + static_cast<uint64_t>(q);   // global chunk index
            const uint4 w = philox4x32_10(
                make_uint4(static_cast<uint32_t>(qg), static_cast<uint32_t>(qg >> 32), a.ctr_T, a.ctr_client),
                a.key0, a.key1);
            nib = transmit_bit(w.x, v[s][0], a.c, a.eps_c) | (transmit_bit(w.y, v[s][1], a.c, a.eps_c) << 1) |
                  (transmit_bit(w.z, v[s][2], a.c, a.eps_c) << 2) |
                  (transmit_bit(w.w, v[s][3], a.c, a.eps_c) << 3);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t bk = __builtin_amdgcn_ballot_w64(((nib >> k) & 1u) != 0);
            count += static_cast<uint32_t>(__popcll(bk));
            word_lo = amdgcn_writelane(static_cast<int>(bk), 4 * s + k, word_lo);
            word_hi = amdgcn_writelane(static_cast<int>(bk >> 32), 4 * s + k, word_hi);
        }
    }
    if (lane < kTileWords)
        a.ballots[tile * kTileWords + lane] =
            (static_cast<uint64_t>(static_cast<uint32_t>(word_hi)) << 32) | static_cast<uint32_t>(word_lo);
    if (STORE_COUNT && lane == 0) a.tile_count[tile] = count;
    return count;
}

// Several pushes decided from one v: a wave marks its tile for pushes
// [b0, b0 + nb), so v is read once for all of them and both sides of the
// transmit test are formed once.  The tile must be full and aligned and its
// global chunk indexes must share their high word (shared_tile); the counts
// go to the pushes' tile counts (STORE_COUNT) or to s_cnt[(b - b0) * stride].
// Per push the bits are mark_tile's.
__device__ __forceinline__ bool shared_tile(const SelectArgs& a, int64_t tile, bool aligned)
{
    const uint32_t q_lo = static_cast<uint32_t>(a.chunk_base + static_cast<uint64_t>(tile * kChunksPerTile));
    return aligned && (tile + 1) * kChunksPerTile * 4 <= a.P && q_lo <= 0xffffffffu - (kChunksPerTile - 1);
}

template <bool STORE_COUNT>
__device__ __forceinline__ void mark_tile_shared(const SelectArgs& a, const SelectBatch& bt, int b0, int nb,
                                                 int64_t tile, int lane, uint32_t* s_cnt, int stride)
{
    const int64_t q0 = tile * kChunksPerTile + lane;
    f4 v[kTileSegs];
    float t[kTileSegs][4], u[kTileSegs][4];
#pragma unroll
    for (int s = 0; s < kTileSegs; ++s) v[s] = *reinterpret_cast<const f4*>(a.v + (q0 + s * kWave) * 4);
#pragma unroll
    for (int s = 0; s < kTileSegs; ++s)
#pragma unroll
        for (int k = 0; k < 4; ++k) transmit_sides(v[s][k], a.c, a.eps_c, t[s][k], u[s][k]);
    const uint64_t qg = a.chunk_base + static_cast<uint64_t>(tile * kChunksPerTile);   // wave-uniform
    const uint32_t q_hi = static_cast<uint32_t>(qg >> 32);
    const uint32_t q_lo = static_cast<uint32_t>(qg) + static_cast<uint32_t>(lane);
    for (int g = 0; g < nb; ++g) {
        const int b = b0 + g;
        int word_lo = 0, word_hi = 0;   // as in mark_tile
        uint32_t count = 0;
#pragma unroll
        for (int s = 0; s < kTileSegs; ++s) {
            const uint4 w = philox4x32_10(make_uint4(q_lo + s * kWave, q_hi, bt.ctr_T[b], bt.ctr_client[b]), a.key0,
                                          a.key1);
            const uint32_t word[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t bk = __builtin_amdgcn_ballot_w64(transmit_test(word[k], t[s][k], u[s][k]));
                count += static_cast<uint32_t>(__popcll(bk));
                word_lo = amdgcn_writelane(static_cast<int>(bk), 4 * s + k, word_lo);
                word_hi = amdgcn_writelane(static_cast<int>(bk >> 32), 4 * s + k, word_hi);
            }
        }
        const size_t off = b * bt.ws_stride;
        uint64_t* ballots = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(a.ballots) + off);
        if (lane < kTileWords)
            ballots[tile * kTileWords + lane] =
                (static_cast<uint64_t>(static_cast<uint32_t>(word_hi)) << 32) | static_cast<uint32_t>(word_lo);
        if (lane == 0) {
            if (STORE_COUNT)
                reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(a.tile_count) + off)[tile] = count;
            else
                s_cnt[g * stride] = count;
        }
    }
}

// Mark one segment, with bounds, and return its transmit count: the tiles
// that are not shared_tile (rolled, so that they cost the kernels no
// registers).
__device__ __forceinline__ uint32_t mark_segment(const SelectArgs& a, int64_t seg, int lane)
{
    const int64_t q = seg * kWave + lane;
    uint32_t nib = 0;
    if (q < n_chunks(a.P)) {
        const f4 v = load_chunk(a.v, q, a.P);
        const uint64_t qg = a.chunk_base + static_cast<uint64_t>(q);
        const uint4 w = philox4x32_10(
            make_uint4(static_cast<uint32_t>(qg), static_cast<uint32_t>(qg >> 32), a.ctr_T, a.ctr_client), a.key0,
            a.key1);
        nib = transmit_bit(w.x, v[0], a.c, a.eps_c) | (transmit_bit(w.y, v[1], a.c, a.eps_c) << 1) |
              (transmit_bit(w.z, v[2], a.c, a.eps_c) << 2) | (transmit_bit(w.w, v[3], a.c, a.eps_c) << 3);
    }
    uint32_t count = 0;
    uint64_t mine = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint64_t bk = __builtin_amdgcn_ballot_w64(((nib >> k) & 1u) != 0);
        count += static_cast<uint32_t>(__popcll(bk));
        if (lane == k) mine = bk;
    }
    if (lane < 4) a.ballots[seg * 4 + lane] = mine;
    return count;
}

// One tile for pushes [b0, b0 + nb) of a batch.
template <bool STORE_COUNT>
__device__ __forceinline__ void mark_pushes(const SelectArgs& a0, const SelectBatch& bt, int b0, int nb, int64_t tile,
                                            int lane, bool aligned, uint32_t* s_cnt, int stride)
{
    if (shared_tile(a0, tile, aligned)) {
        mark_tile_shared<STORE_COUNT>(a0, bt, b0, nb, tile, lane, s_cnt, stride);
        return;
    }
#pragma clang loop unroll(disable)
    for (int g = 0; g < nb; ++g) {
        const SelectArgs a = push_args(a0, bt, b0 + g);
        uint32_t count = 0;
#pragma clang loop unroll(disable)
        for (int s = 0; s < kTileSegs; ++s) count += mark_segment(a, tile * kTileSegs + s, lane);
        if (lane == 0) {
            if (STORE_COUNT)
                a.tile_count[tile] = count;
            else
                s_cnt[g * stride] = count;
        }
    }
}

// Pushes a wave marks together (the grid's y index counts such groups).  From
// 4M parameters on, where v and the gradients no longer share the caches
// (the saved reads of v are HBM traffic); below, the vector ALU bounds the
// mark and fewer, longer waves balance worse.  Selection and apply of B
// pushes, one at a time against groups of 2, 4 and 8, same box:
//   P, B, transmitted    1       2       4       8
//   1.8M, 16, 20 %      75.7    75.3    76.9    80.0 us
//   3M, 3, 20 %         44.1    43.7    44.6    44.5
//   3M, 16, 20 %        123     120     118     120
//   6M, 2, 10 %         64.3    62.4    62.4    62.0
//   6M, 8, 10 %         126     123     121     123
//   12M, 32, 10 %       725     693     678     672
//   39M, 8, 10 %        791     755     744     745
constexpr int kMarkPushes = 4;
constexpr int64_t kMarkSharedFrom = 4'000'000;
int mark_group(int64_t P, int B, bool aligned)
{
    return aligned && P >= kMarkSharedFrom ? (B < kMarkPushes ? B : kMarkPushes) : 1;
}

__global__ __launch_bounds__(kSelBlock) void select_mark_shared(const SelectArgs a0, const SelectBatch bt, int B, int G)
{
    const int b0 = blockIdx.y * G;
    const int nb = B - b0 < G ? B - b0 : G;
    const int64_t tile = wave_tile();
    if (tile >= a0.n_tiles) return;
    mark_pushes<true>(a0, bt, b0, nb, tile, threadIdx.x & (kWave - 1), true, nullptr, 0);
}

__global__ __launch_bounds__(kSelBlock) void select_mark(const SelectArgs a0, const SelectBatch bt, bool aligned)
{
    const SelectArgs a = push_args(a0, bt, blockIdx.y);
    const int64_t tile = wave_tile();
    if (tile >= a.n_tiles) return;
    const int lane = threadIdx.x & (kWave - 1);
    if (aligned && (tile + 1) * kChunksPerTile * 4 <= a.P)
        mark_tile<true, true>(a, tile, lane);
    else
        mark_tile<false, true>(a, tile, lane);
}

// Inclusive prefix sum over the wave's 64 lanes in register-to-register
// DPP adds: row shifts by 1, 2, 4 and 8 give each 16-lane row its own
// prefix sums (lanes shifted in from outside the row read 0), then the last
// lane of row 0 is broadcast into row 1 and of row 2 into row 3, and the
// last lane of row 1 (the sum of lanes 0-31) into rows 2 and 3.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x)
{
    constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
    constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowShr1, 0xf, 0xf, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowShr2, 0xf, 0xf, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowShr4, 0xf, 0xf, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowShr8, 0xf, 0xf, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowBcast15, 0xa, 0xf, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kRowBcast31, 0xc, 0xf, false));
    return x;
}

// Block-wide exclusive scan of one value per thread (kScanBlock threads).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* total)
{
    __shared__ uint32_t wave_total[kScanBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const uint32_t inc = wave_inclusive_scan(x);
    if (lane == kWave - 1) wave_total[wave] = inc;
    __syncthreads();
    if (wave == 0) {
        const uint32_t t = wave_inclusive_scan(lane < kScanBlock / kWave ? wave_total[lane] : 0u);
        if (lane < kScanBlock / kWave) wave_total[lane] = t;
    }
    __syncthreads();
    *total = wave_total[kScanBlock / kWave - 1];
    return inc - x + (wave > 0 ? wave_total[wave - 1] : 0u);
}

// Group g of 1024 tiles: offsets of its tiles within the group and the group
// total; select_scatter sums the totals of the groups before its own.
// FROM_BALLOTS: the tile counts were not written (the mark step ran inside
// another pass); count the tiles' ballot bits instead.  The wave's 64 tiles
// are 8 KB of ballot words, read in 8 rounds of one 16-byte piece per lane
// (8 lanes per tile, contiguous), summed over each group of 8 lanes and
// passed through LDS to the lane of the tile.
__device__ __forceinline__ uint32_t wave_tile_bits(const SelectArgs& a, int64_t wave_first_tile, int lane)
{
    __shared__ uint32_t s_cnt[kScanBlock / kWave][kWave];
    const int w = threadIdx.x / kWave;
    constexpr int kPieces = kTileWords / 2;                 // 16-byte pieces per tile
    constexpr int kTilesPerRound = kWave / kPieces;
    const ulonglong2* base = reinterpret_cast<const ulonglong2*>(a.ballots + wave_first_tile * kTileWords);
#pragma unroll
    for (int r = 0; r < kPieces; ++r) {
        const int t = r * kTilesPerRound + lane / kPieces;  // tile of this lane's piece, within the wave's 64
        uint32_t n = 0;
        if (wave_first_tile + t < a.n_tiles) {
            const ulonglong2 piece = base[r * kWave + lane];
            n = __popcll(piece.x) + __popcll(piece.y);
        }
#pragma unroll
        for (int d = 1; d < kPieces; d <<= 1) n += __shfl_xor(n, d, kWave);
        if (lane % kPieces == 0) s_cnt[w][t] = n;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return s_cnt[w][lane];
}

template <bool FROM_BALLOTS>
__global__ __launch_bounds__(kScanBlock) void select_scan(const SelectArgs a0, const SelectBatch bt)
{
    const SelectArgs a = push_args(a0, bt, blockIdx.y);
    const int64_t t = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x;
    uint32_t c = 0;
    if (FROM_BALLOTS) {
        const int64_t wave_first = t - (threadIdx.x & (kWave - 1));
        c = wave_tile_bits(a, wave_first, threadIdx.x & (kWave - 1));
        if (t >= a.n_tiles) c = 0;
    } else if (t < a.n_tiles) {
        c = a.tile_count[t];
    }
    uint32_t total;
    const uint32_t off = block_exclusive_scan(c, &total);
    if (t < a.n_tiles) a.tile_offset[t] = off;
    if (threadIdx.x == 0) a.group_total[blockIdx.x] = total;
}

// Scatter one tile; FULL as for mark_tile.  The tile's entries are staged
// in output order in the wave's LDS slice and leave in contiguous full-wave
// stores (a lane storing its own entries directly issues four sparse masked
// stores per segment).  The slice holds kStageEntries; a segment that would
// overflow it flushes it first, so the slice stays small enough for full
// occupancy while a tile at any transmit fraction up to about 1/4 leaves in
// one flush.
constexpr int kStageEntries = 4 * kWave;     // one segment's worth

__device__ __forceinline__ void wave_lds_order()
{
    // the wave's LDS operations execute in order; keep the compiler from
    // moving the reads of other lanes' entries above the writes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// entries [0, n) of the stage to output positions [base, base + n)
__device__ __forceinline__ void drain(const SelectArgs& a, const int32_t* s_idx, const float* s_val, uint32_t n,
                                      int64_t base, int lane)
{
    for (uint32_t e = lane; e < n; e += kWave) {
        const int64_t pos = base + e;
        if (pos < a.capacity) {
            a.out_idx[pos] = s_idx[e];
            a.out_val[pos] = s_val[e];
        }
    }
}

// Every gradient load of the tile, issued before anything waits on them (at
// any transmit fraction worth compacting every line holds a transmitted
// value, so loading the whole tile costs no traffic).
template <bool FULL>
__device__ __forceinline__ void load_tile_grad(const SelectArgs& a, int64_t tile, int lane, f4 (&g)[kTileSegs])
{
    const int64_t nch = n_chunks(a.P);
    const int64_t q0 = tile * kChunksPerTile + lane;
#pragma unroll
    for (int s = 0; s < kTileSegs; ++s) {
        const int64_t q = q0 + s * kWave;
        if (FULL)
            g[s] = *reinterpret_cast<const f4*>(a.grad + q * 4);
        else if (q < nch)
            g[s] = load_chunk(a.grad, q, a.P);
    }
}

// The tile's ballot words (wave-uniform, scalar loads).  Loaded together
// with the gradients, ahead of any use: loading them segment by segment
// left up to three dependent scalar round trips in each wave's lifetime.
__device__ __forceinline__ void load_tile_ballots(const SelectArgs& a, int64_t tile, uint64_t (&bw)[kTileWords])
{
    const uint64_t* tb = a.ballots + tile * kTileWords;
#pragma unroll
    for (int k = 0; k < kTileWords; ++k) bw[k] = tb[k];
}

// The tile's entries, with gradients g and ballot words bw (loaded into
// registers already, or the tile's words in the workspace), to list
// positions from `base` on.  Chunks past P carry no ballot bits, so their
// (unloaded) gradients are never read.
__device__ __forceinline__ void scatter_loaded(const SelectArgs& a, int64_t tile, int lane, const f4 (&g)[kTileSegs],
                                               const uint64_t* bw, int64_t base, int32_t* s_idx, float* s_val)
{
    const int64_t q0 = tile * kChunksPerTile + lane;
    const uint64_t below = lanes_below(lane);
    uint32_t staged = 0;
    uint32_t seg_pos = 0;   // lane s < kTileSegs: list position of segment s's first entry
#pragma unroll
    for (int s = 0; s < kTileSegs; ++s) {
        const uint64_t b0 = bw[4 * s], b1 = bw[4 * s + 1], b2 = bw[4 * s + 2], b3 = bw[4 * s + 3];
        const uint32_t nib = static_cast<uint32_t>((b0 >> lane) & 1) | static_cast<uint32_t>(((b1 >> lane) & 1) << 1) |
                             static_cast<uint32_t>(((b2 >> lane) & 1) << 2) |
                             static_cast<uint32_t>(((b3 >> lane) & 1) << 3);
        const uint32_t n_seg = __popcll(b0) + __popcll(b1) + __popcll(b2) + __popcll(b3);
        if (lane == s) seg_pos = static_cast<uint32_t>(base + staged);
        if (staged + n_seg > static_cast<uint32_t>(kStageEntries)) {
            wave_lds_order();
            drain(a, s_idx, s_val, staged, base, lane);
            wave_lds_order();
            base += staged;
            staged = 0;
        }
        // entries of the lanes below come first; within a lane, ascending c
        uint32_t p = staged + __popcll(b0 & below) + __popcll(b1 & below) + __popcll(b2 & below) +
                     __popcll(b3 & below);
        const int64_t q = q0 + s * kWave;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if ((nib >> c) & 1u) {
                s_idx[p] = static_cast<int32_t>(q * 4 + c);
                s_val[p] = g[s][c];
                ++p;
            }
        }
        staged += n_seg;
    }
    wave_lds_order();
    drain(a, s_idx, s_val, staged, base, lane);
    if (a.seg_start) {
        static_assert(kTileSegs * kWave * 4 == kTileSegs * kPushSeg, "a tile segment is a list-index segment");
        const int64_t sg = tile * kTileSegs + lane;
        if (lane < kTileSegs && sg < a.n_segs) a.seg_start[sg] = seg_pos;
    }
}

// The list position of a tile's first entry: the totals of the groups before
// its own, 256 of them (one 16-byte load per lane) at a time, and the tile's
// offset within its group.  The first kGroupLoads loads are issued before the
// tile's gradient loads, so that waiting for them leaves the gradients in
// flight; 4 cover 1024 groups, 1.07e9 parameters.  Against a launch that
// scanned the totals (up to 64 groups: the last scan block to arrive did), the
// whole selection at 10 %, same box: 52M 91.9 -> 88.4 us, 100M 172.8 -> 165.5,
// 300M 519 -> 508; at 1e9 equal.
constexpr int kGroupLoads = 4;        // EARLY: 1

__device__ __forceinline__ uint4 load_totals(const SelectArgs& a, int k, int n, int lane)
{
    // groups at or past n do not count; a lane that holds none of the others reads nothing
    const int g = 4 * (lane + kWave * k);
    return g < n ? reinterpret_cast<const uint4*>(a.group_total)[lane + kWave * k] : make_uint4(0u, 0u, 0u, 0u);
}

__device__ __forceinline__ uint32_t sum_totals(const uint4& x, int k, int n, int lane)
{
    const int g = 4 * (lane + kWave * k);
    return (g < n ? x.x : 0u) + (g + 1 < n ? x.y : 0u) + (g + 2 < n ? x.z : 0u) + (g + 3 < n ? x.w : 0u);
}

template <int GL>
__device__ __forceinline__ int64_t group_position(const SelectArgs& a, const uint4 (&tv)[GL], int n, int lane)
{
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < GL; ++k)
        if (4 * kWave * k < n) s += sum_totals(tv[k], k, n, lane);   // wave-uniform
    for (int k = GL; 4 * kWave * k < n; ++k) s += sum_totals(load_totals(a, k, n, lane), k, n, lane);
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wave_inclusive_scan(s)), kWave - 1));
}

// The call's count (and the list index's last entry) from the last tile.
template <typename Words>
__device__ __forceinline__ void finish_list(const SelectArgs& a, int64_t tile, int lane, const Words& bw, int64_t base)
{
    if (tile == a.n_tiles - 1 && lane == 0) {
        uint32_t mine = 0;
#pragma unroll
        for (int k = 0; k < kTileWords; ++k) mine += __popcll(bw[k]);
        *a.d_count = base + mine;
        if (a.seg_start) a.seg_start[a.n_segs] = static_cast<uint32_t>(base + mine);
    }
}

// EARLY: every ballot word and the list position are loaded and waited for
// while the gradient loads are in flight.  In calls of at most
// kEarlyGroups groups (up to 67M parameters: the scan after a pass that
// took the decisions, and standalone calls past the two-launch form) every
// wave's latency is exposed, and this took the 25M selection, then in three
// launches, from 44.0-46.6 to 41.5-45.1 us (same box, lists identical).  Otherwise the compiler issues each part
// where it is first used (three dependent scalar round trips per tile),
// which was 3 % faster at 1e9 (1.63-1.65 against 1.70 ms), where many more
// waves are in flight to cover them.
template <bool FULL, bool EARLY>
__device__ __forceinline__ void scatter_tile(const SelectArgs& a, int64_t tile, int lane, int32_t* s_idx,
                                             float* s_val)
{
    const int n = static_cast<int>(tile / kScanBlock);   // groups before this tile's
    constexpr int GL = EARLY ? 1 : kGroupLoads;
    uint4 tv[GL];
#pragma unroll
    for (int k = 0; k < GL; ++k)
        tv[k] = 4 * kWave * k < n ? load_totals(a, k, n, lane) : make_uint4(0u, 0u, 0u, 0u);
    __builtin_amdgcn_sched_barrier(0);
    f4 g[kTileSegs];
    load_tile_grad<FULL>(a, tile, lane, g);
    const uint32_t tile_off = a.tile_offset[tile];
    if (EARLY && FULL) {
        uint64_t bw[kTileWords];
        load_tile_ballots(a, tile, bw);
        // uses that keep the compiler from sinking these loads to the first
        // use of each
#pragma unroll
        for (int k = 0; k < kTileWords; ++k) asm volatile("" ::"s"(bw[k]));
        asm volatile("" ::"s"(tile_off));
        const int64_t base = group_position(a, tv, n, lane) + tile_off;
        scatter_loaded(a, tile, lane, g, bw, base, s_idx, s_val);
        finish_list(a, tile, lane, bw, base);
    } else {
        const int64_t base = group_position(a, tv, n, lane) + tile_off;
        const uint64_t* bw = a.ballots + tile * kTileWords;
        scatter_loaded(a, tile, lane, g, bw, base, s_idx, s_val);
        finish_list(a, tile, lane, bw, base);
    }
}

// 64 VGPRs keep 8 waves per SIMD (the EARLY form needs 71 uncapped).
template <bool EARLY>
__global__ __launch_bounds__(kSelBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void select_scatter(
    const SelectArgs a0, const SelectBatch bt, bool aligned)
{
    const SelectArgs a = push_args(a0, bt, blockIdx.y);
    __shared__ int32_t s_idx[kWavesPerBlock][kStageEntries];
    __shared__ float s_val[kWavesPerBlock][kStageEntries];
    const int64_t tile = wave_tile();
    if (tile >= a.n_tiles) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    if (aligned && (tile + 1) * kChunksPerTile * 4 <= a.P)
        scatter_tile<true, EARLY>(a, tile, lane, s_idx[w], s_val[w]);
    else
        scatter_tile<false, EARLY>(a, tile, lane, s_idx[w], s_val[w]);
}

// Two-launch selection, for calls of at most kDirectMaxTiles tiles per push:
// no scan launch, and no wave waits for another.
//   select_mark_totals  blocks of TPB waves, one tile each, store the
//     tiles' ballot words as select_mark does and their counts in LDS; the
//     last wave to arrive (an LDS arrival counter) stores each tile's offset
//     within the block and the block total as 16 bits (at most 16 x 1024).
//   select_scatter_direct  every wave finds its own list position: the
//     totals of all blocks before its tile's block plus the tile's offset
//     within its block.  KT 16-byte loads per lane cover the totals of
//     512 KT blocks; they are issued before the gradient loads, so the wait
//     for them leaves the gradients in flight, and the wave sums them in
//     registers and across its lanes.
// The result is that of the three launches, bit for bit.  Against them on
// the same box (10 % transmitted, back to back): 8.4M 17.2 against 19.6 us,
// 12M 23.0 against 25.9, 25M 39.2 against 41.0, 33M 51.2 against 52.2 and
// 50M 86.0 against 91.3 us; at 1.8M the kernels take 8.2 us against 10.0 us
// for the two-launch form with 16-wave blocks and a block barrier in the
// scatter that this form replaced.  Blocks of 8 tiles are the faster shape
// where both fit (probes at 25M: 38.6 against 39.2 us with blocks of 16 and
// half the loads).  A mark block of 8 waves takes 1.1-1.4 us longer than one
// of 4 at 25M (it needs 8 free wave slots on a CU to start), but blocks of 4
// would need twice the loads and more registers than the scatter has.
constexpr int kDirectLoads = 6;                                  // 16-byte loads of block totals per lane, at most
constexpr int64_t kDirectMaxBlocks = int64_t(kDirectLoads) * kWave * 8;   // 3072 block totals (6 KB)
constexpr int64_t kDirectMaxTiles = 16 * kDirectMaxBlocks;       // 49,152 tiles: 50.3M parameters
static_assert(kDirectMaxBlocks * sizeof(uint16_t) <= kMaxGroups * sizeof(uint32_t),
              "16-bit block totals fit the group totals");

template <int TPB>
__global__ __launch_bounds__(TPB * kWave) void select_mark_totals(const SelectArgs a0, const SelectBatch bt,
                                                                  bool aligned)
{
    static_assert(TPB * kChunksPerTile * 4 < 65536 && TPB <= kWave, "a block total fits 16 bits");
    const SelectArgs a = push_args(a0, bt, blockIdx.y);
    __shared__ uint32_t s_cnt[TPB];
    __shared__ uint32_t s_arrived;
    if (threadIdx.x == 0) s_arrived = 0;
    __syncthreads();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * TPB;
    const int64_t tile = t0 + w;
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t count = 0;
    if (tile < a.n_tiles) {
        if (aligned && (tile + 1) * kChunksPerTile * 4 <= a.P)
            count = mark_tile<true, false>(a, tile, lane);
        else
            count = mark_tile<false, false>(a, tile, lane);
    }
    int last = 0;
    if (lane == 0) {
        s_cnt[w] = count;
        // release / acquire: the last wave to arrive sees every count
        last = __hip_atomic_fetch_add(&s_arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == TPB - 1;
    }
    if (__builtin_amdgcn_readfirstlane(last)) {
        const uint32_t c = lane < TPB ? s_cnt[lane] : 0u;
        const uint32_t inc = wave_inclusive_scan(c);
        if (lane < TPB && t0 + lane < a.n_tiles) a.tile_offset[t0 + lane] = inc - c;
        if (lane == TPB - 1) reinterpret_cast<uint16_t*>(a.group_total)[blockIdx.x] = static_cast<uint16_t>(inc);
    }
}

// The same for pushes [G blockIdx.y, G blockIdx.y + G) of a batch of B
// (16-byte aligned arrays), marked together.
template <int TPB>
__global__ __launch_bounds__(TPB * kWave) void select_mark_totals_shared(const SelectArgs a0, const SelectBatch bt,
                                                                         int B, int G)
{
    __shared__ uint32_t s_cnt[kMarkPushes][TPB];
    __shared__ uint32_t s_arrived;
    if (threadIdx.x == 0) s_arrived = 0;
    __syncthreads();
    const int b0 = blockIdx.y * G;
    const int nb = B - b0 < G ? B - b0 : G;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * TPB;
    const int64_t tile = t0 + w;
    const int lane = threadIdx.x & (kWave - 1);
    if (tile < a0.n_tiles)
        mark_pushes<false>(a0, bt, b0, nb, tile, lane, true, &s_cnt[0][w], TPB);
    else if (lane == 0)
        for (int g = 0; g < nb; ++g) s_cnt[g][w] = 0;
    int last = 0;
    if (lane == 0)   // release / acquire, after this lane's counts: the last wave to arrive sees every count
        last = __hip_atomic_fetch_add(&s_arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == TPB - 1;
    if (__builtin_amdgcn_readfirstlane(last)) {
        for (int g = 0; g < nb; ++g) {
            const size_t off = (b0 + g) * bt.ws_stride;
            uint32_t* tile_offset = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(a0.tile_offset) + off);
            uint16_t* totals = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(a0.group_total) + off);
            const uint32_t c = lane < TPB ? s_cnt[g][lane] : 0u;
            const uint32_t inc = wave_inclusive_scan(c);
            if (lane < TPB && t0 + lane < a0.n_tiles) tile_offset[t0 + lane] = inc - c;
            if (lane == TPB - 1) totals[blockIdx.x] = static_cast<uint16_t>(inc);
        }
    }
}

__device__ __forceinline__ uint32_t sum_halves(uint32_t x) { return (x & 0xffffu) + (x >> 16); }

// Mask of the 16-bit halves j < r of 32-bit word i (halves 2i, 2i + 1).
__device__ __forceinline__ uint32_t halves_below(int i, int r)
{
    return (2 * i + 1 < r) ? 0xffffffffu : (2 * i < r ? 0xffffu : 0u);
}

// The list position of the first entry of a tile whose block has
// `blocks_before` blocks before it: the sum of their 16-bit totals plus the
// tile's offset within its block.  Lane l holds the groups l + 64 k of 8
// totals (tv[k]); the group that holds the last totals that count is summed
// in part.
template <int KT>
__device__ __forceinline__ int64_t direct_position(const uint4 (&tv)[KT], int blocks_before, uint32_t tile_off,
                                                   int lane)
{
    const int whole = blocks_before >> 3;   // groups of 8 totals that count in full
    const int r = blocks_before & 7;        // totals of the next group that count
    const uint32_t m0 = halves_below(0, r), m1 = halves_below(1, r), m2 = halves_below(2, r),
                   m3 = halves_below(3, r);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int grp = lane + kWave * k;
        const bool all = grp < whole;
        const uint32_t x = sum_halves(tv[k].x & (all ? ~0u : m0)) + sum_halves(tv[k].y & (all ? ~0u : m1)) +
                           sum_halves(tv[k].z & (all ? ~0u : m2)) + sum_halves(tv[k].w & (all ? ~0u : m3));
        s += grp <= whole ? x : 0u;
    }
    const uint32_t inc = wave_inclusive_scan(s);
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), kWave - 1)) + tile_off;
}

// FULL as for mark_tile.  The partial tile (or every tile of misaligned
// arrays) finds its position before it loads its gradients, and reads its
// ballot words from the workspace where it uses them, which needs fewer
// registers.
template <bool FULL, int TPB, int KT>
__device__ __forceinline__ void scatter_direct_tile(const SelectArgs& a, int64_t tile, int lane, int32_t* s_idx,
                                                    float* s_val)
{
    const int nb = static_cast<int>(tile / TPB);   // blocks before this tile's block
    const uint4* tot = reinterpret_cast<const uint4*>(a.group_total);
    uint4 tv[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k)   // only the groups some lane needs (wave-uniform)
        tv[k] = kWave * k <= (nb >> 3) ? tot[lane + kWave * k] : make_uint4(0u, 0u, 0u, 0u);
    f4 g[kTileSegs];
    if (FULL) {
        // the loads above are issued before the gradients', so waiting for
        // them leaves the gradients in flight
        __builtin_amdgcn_sched_barrier(0);
        load_tile_grad<true>(a, tile, lane, g);
        const uint32_t tile_off = a.tile_offset[tile];
        uint64_t bw[kTileWords];
        load_tile_ballots(a, tile, bw);
        // uses that keep the compiler from sinking these (scalar) loads to
        // the first use of each
#pragma unroll
        for (int k = 0; k < kTileWords; ++k) asm volatile("" ::"s"(bw[k]));
        asm volatile("" ::"s"(tile_off));
        const int64_t base = direct_position<KT>(tv, nb, tile_off, lane);
        scatter_loaded(a, tile, lane, g, bw, base, s_idx, s_val);
        finish_list(a, tile, lane, bw, base);
    } else {
        const int64_t base = direct_position<KT>(tv, nb, a.tile_offset[tile], lane);
        load_tile_grad<false>(a, tile, lane, g);
        const uint64_t* bw = a.ballots + tile * kTileWords;
        scatter_loaded(a, tile, lane, g, bw, base, s_idx, s_val);
        finish_list(a, tile, lane, bw, base);
    }
}

template <int TPB, int KT>
__global__ __launch_bounds__(kSelBlock) __attribute__((amdgpu_waves_per_eu(8, 8))) void select_scatter_direct(
    const SelectArgs a0, const SelectBatch bt, bool aligned)
{
    const SelectArgs a = push_args(a0, bt, blockIdx.y);
    __shared__ int32_t s_idx[kWavesPerBlock][kStageEntries];
    __shared__ float s_val[kWavesPerBlock][kStageEntries];
    const int64_t tile = wave_tile();
    if (tile >= a.n_tiles) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    if (aligned && (tile + 1) * kChunksPerTile * 4 <= a.P)
        scatter_direct_tile<true, TPB, KT>(a, tile, lane, s_idx[w], s_val[w]);
    else
        scatter_direct_tile<false, TPB, KT>(a, tile, lane, s_idx[w], s_val[w]);
}

// After a pass that took the decisions (it leaves ballot words, no counts):
// each tile's offset within its block of TPB tiles and the blocks' 16-bit
// totals, for select_scatter_direct.  A wave counts 64 consecutive tiles,
// one per lane (as the scan from ballots does); a block of tiles is TPB
// consecutive lanes, so a scan within segments of TPB lanes gives both.
template <int TPB>
__global__ __launch_bounds__(kSelBlock) void select_count_totals(const SelectArgs a)
{
    static_assert(kWave % TPB == 0, "a block of tiles lies within one wave");
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t t = static_cast<int64_t>(blockIdx.x) * kSelBlock + threadIdx.x;
    uint32_t c = wave_tile_bits(a, t - lane, lane);
    if (t >= a.n_tiles) c = 0;
    uint32_t inc = c;
#pragma unroll
    for (int d = 1; d < TPB; d <<= 1) {
        const uint32_t up = __shfl_up(inc, d, kWave);
        if (lane % TPB >= d) inc += up;
    }
    if (t < a.n_tiles) a.tile_offset[t] = inc - c;
    if (lane % TPB == TPB - 1 && t - (TPB - 1) < a.n_tiles)
        reinterpret_cast<uint16_t*>(a.group_total)[t / TPB] = static_cast<uint16_t>(inc);
}

// The two-launch selection; from_ballots (one push): the decisions were
// taken by the preceding pass, so the first launch only counts.
template <int TPB>
hipError_t launch_direct(const SelectArgs& a, const SelectBatch& bt, int B, bool aligned, bool from_ballots,
                         hipStream_t s)
{
    const int64_t blocks = (a.n_tiles + TPB - 1) / TPB;
    const int kt = static_cast<int>((blocks + kWave * 8 - 1) / (kWave * 8));
    if (from_ballots) {
        select_count_totals<TPB><<<static_cast<unsigned>((a.n_tiles + kSelBlock - 1) / kSelBlock), kSelBlock, 0,
                                   s>>>(a);
    } else {
        const int G = mark_group(a.P, B, aligned);
        const dim3 mgrid(static_cast<unsigned>(blocks), static_cast<unsigned>((B + G - 1) / G));
        if (G > 1)
            select_mark_totals_shared<TPB><<<mgrid, TPB * kWave, 0, s>>>(a, bt, B, G);
        else
            select_mark_totals<TPB><<<mgrid, TPB * kWave, 0, s>>>(a, bt, aligned);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(static_cast<unsigned>((a.n_tiles + kWavesPerBlock - 1) / kWavesPerBlock), static_cast<unsigned>(B));
    switch (kt) {
    case 1: select_scatter_direct<TPB, 1><<<grid, kSelBlock, 0, s>>>(a, bt, aligned); break;
    case 2: select_scatter_direct<TPB, 2><<<grid, kSelBlock, 0, s>>>(a, bt, aligned); break;
    case 3: select_scatter_direct<TPB, 3><<<grid, kSelBlock, 0, s>>>(a, bt, aligned); break;
    case 4: select_scatter_direct<TPB, 4><<<grid, kSelBlock, 0, s>>>(a, bt, aligned); break;
    case 5: select_scatter_direct<TPB, 5><<<grid, kSelBlock, 0, s>>>(a, bt, aligned); break;
    case 6: select_scatter_direct<TPB, 6><<<grid, kSelBlock, 0, s>>>(a, bt, aligned); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

constexpr int kListBlock = 256;               // list kernels: 4 waves
constexpr int64_t kListMaxBlocks = 65536;     // grid cap of the list kernels (grid-stride)

// A wave owns 64 E consecutive list entries and lane l takes entries
// l, l + 64, ...: every gather instruction covers 64 consecutive entries
// (ascending indices, so few cache lines), and each thread issues all E of
// its gathers before the first update.  Bound by whole-line traffic of the
// state: at 10 % nearly every 128-byte line holds a listed parameter.
// STREAM: the scattered stores (and the list's loads) are non-temporal, so
// partly written lines leave the L2 caches at once instead of displacing
// lines still to be read; lines that two waves share are then written twice,
// which a longer run per wave (E = 6) makes rarer.  A whole push (selection
// and this), plain E = 2 against STREAM with E = 2 and 6, same box:
//   P, transmitted   plain    E = 2    E = 6
//   1.8M, 20 %       22.1     22.5     25.0 us
//   3.2M, 10 %       32.8     31.8     35.6
//   5M, 10 %         54.5     46.9     47.0
//   12M, 20 %        136      131      133
//   25M, 10 %        276      258      243
//   25M, 30 %        287      269      282
//   300M, 10 %       3280     3090     2800
//   300M, 2 %        1632     1566     1549
// (non-temporal loads of the state cost 30 %: a line's second reader misses).
// The lines are drawn at 10 %, by P alone: the launch does not know the count,
// and at 25M and 30 % E = 6 still beats the plain form.
template <int MODE, int E, bool STREAM>
__device__ __forceinline__ void sparse_runs(const SparseArgs& a, int64_t m)
{
    const Hyper h = a.h;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave_id = (static_cast<int64_t>(blockIdx.x) * kListBlock + threadIdx.x) / kWave;
    const int64_t n_waves = static_cast<int64_t>(gridDim.x) * (kListBlock / kWave);
    for (int64_t base = wave_id * kWave * E; base < m; base += n_waves * kWave * E) {
        int64_t j[E];
        float g[E], th[E], n[E], b[E], v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int64_t i = base + e * kWave + lane;
            j[e] = -1;
            if (i < m) {
                const int64_t x = STREAM ? __builtin_nontemporal_load(a.idx + i) : a.idx[i];
                if (x >= 0 && x < a.P) { j[e] = x; g[e] = STREAM ? __builtin_nontemporal_load(a.val + i) : a.val[i]; }
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (j[e] >= 0) { th[e] = a.theta[j[e]]; n[e] = a.n[j[e]]; b[e] = a.b[j[e]]; v[e] = a.v[j[e]]; }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (j[e] >= 0) {
                fasgd_step<MODE>(th[e], n[e], b[e], v[e], g[e], a.coef, h);
                if (STREAM) {
                    __builtin_nontemporal_store(th[e], a.theta + j[e]);
                    __builtin_nontemporal_store(n[e], a.n + j[e]);
                    __builtin_nontemporal_store(b[e], a.b + j[e]);
                    __builtin_nontemporal_store(v[e], a.v + j[e]);
                    __builtin_nontemporal_store(a.last_T_value, a.last_T + j[e]);
                } else {
                    a.theta[j[e]] = th[e]; a.n[j[e]] = n[e]; a.b[j[e]] = b[e]; a.v[j[e]] = v[e];
                    a.last_T[j[e]] = a.last_T_value;
                }
            }
        }
    }
}

// A list too short to give each of the 256 CUs two runs of 64 E entries goes
// in runs of 128: such an apply is bound by the latency of its gathers, and
// long runs leave CUs idle.  A whole push, plain E = 2 at every length (an
// earlier form), E = 6 at every length, and the line at 1, 2 and 4 runs per
// CU, same box:
//   P, transmitted          E = 2    E = 6     1       2       4
//   17M, 0.3 % (51k)         46.1     56.4    45.7    44.6    45.8 us
//   17M, 0.6 % (102k)        55.9     61.8    59.3    50.2    52.1
//   25M, 0.4 % (100k)        69.5     73.1    71.7    62.9    62.5
//   25M, 0.6 % (150k)        82.6     77.4    78.0    74.5    74.4
//   100M, 0.1 % (100k)        173      177     174     164     165
//   100M, 0.3 % (300k)        236      204     200     208     206
//   400M, 0.1 % (400k)        650      633     628     628     632
constexpr int kShortE = 2;
constexpr int64_t short_list(int E) { return int64_t(2 * 256) * kWave * E; }

template <int MODE, int E, bool STREAM>
__global__ __launch_bounds__(kListBlock) void sparse_apply(const SparseArgs a)
{
    int64_t m = *a.d_count;
    if (m > a.capacity) m = a.capacity;
    if (E > kShortE && m < short_list(E))
        sparse_runs<MODE, kShortE, STREAM>(a, m);
    else
        sparse_runs<MODE, E, STREAM>(a, m);
}

// The list's values into a dense array, one partial 32-byte sector per entry;
// a wave owns 64 E consecutive entries and loads them all first.  STREAM as
// for sparse_apply.  Selection and copy together, plain E = 1 (the former
// form), plain E = 2, STREAM with E = 2 and with E = 1, same box:
//   P, transmitted   E = 1    E = 2    E = 2 s. E = 1 s.
//   100k, 1 %        9.05     9.45 us
//   1M, 20 %         10.9     11.1
//   1.8M, 2 %        12.4     12.2
//   4M, 10 %         18.2     16.6     18.9     18.5 us
//   8M, 5 %          27.1     23.9     26.8     26.2
//   8M, 30 %         40.1     37.6     35.3     36.2
//   20M, 20 %        86.2     81.9     77.7     80.2
//   60M, 10 %        218      221      200      196
//   60M, 30 %        242      257      235      226
// (by P alone, as the launch does not know the count: at 8M and 30 % the
// streaming form would gain 6 %, at 5 % it would lose 12)
template <int E, bool STREAM>
__global__ __launch_bounds__(kListBlock) void scatter_list(float* __restrict__ dst, int64_t P,
                                                       const int32_t* __restrict__ idx,
                                                       const float* __restrict__ val,
                                                       const int64_t* __restrict__ d_count, int64_t capacity)
{
    int64_t m = *d_count;
    if (m > capacity) m = capacity;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave_id = (static_cast<int64_t>(blockIdx.x) * kListBlock + threadIdx.x) / kWave;
    const int64_t n_waves = static_cast<int64_t>(gridDim.x) * (kListBlock / kWave);
    for (int64_t base = wave_id * kWave * E; base < m; base += n_waves * kWave * E) {
        int64_t j[E];
        float x[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int64_t i = base + e * kWave + lane;
            j[e] = -1;
            if (i < m) {
                j[e] = STREAM ? __builtin_nontemporal_load(idx + i) : idx[i];
                x[e] = STREAM ? __builtin_nontemporal_load(val + i) : val[i];
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (j[e] >= 0 && j[e] < P) {
                if (STREAM)
                    __builtin_nontemporal_store(x[e], dst + j[e]);
                else
                    dst[j[e]] = x[e];
            }
        }
    }
}

}  // namespace

static_assert(kSelTileParams == kChunksPerTile * 4 && kSelTileWords == kTileWords && kSelMaxGroups == kMaxGroups,
              "the workspace size in kernels.hpp follows this file's layout");

size_t select_workspace_bytes(int64_t P) { return select_workspace_bytes_for(P); }

void select_workspace_layout(void* ws, int64_t P, SelectArgs& a)
{
    const int64_t nt = n_tiles(P);
    char* p = static_cast<char*>(ws);
    a.ballots = reinterpret_cast<uint64_t*>(p);
    p += align256(size_t(nt) * kTileWords * sizeof(uint64_t));
    a.tile_count = reinterpret_cast<uint32_t*>(p);
    p += align256(size_t(nt) * sizeof(uint32_t));
    a.tile_offset = reinterpret_cast<uint32_t*>(p);
    p += align256(size_t(nt) * sizeof(uint32_t));
    a.group_total = reinterpret_cast<uint32_t*>(p);
    a.n_tiles = nt;
}

hipError_t launch_select(const SelectArgs& a, const SelectBatch& bt, int B, bool aligned, hipStream_t s)
{
    const unsigned gx = static_cast<unsigned>((a.n_tiles + kWavesPerBlock - 1) / kWavesPerBlock);
    const unsigned groups = static_cast<unsigned>((a.n_tiles + kScanBlock - 1) / kScanBlock);
    if (groups > static_cast<unsigned>(kMaxGroups) || B < 1 || B > kMaxBatch) return hipErrorInvalidValue;
    if (a.n_tiles <= 8 * kDirectMaxBlocks) return launch_direct<8>(a, bt, B, aligned, false, s);
    if (a.n_tiles <= kDirectMaxTiles) return launch_direct<16>(a, bt, B, aligned, false, s);
    hipError_t e;
    const dim3 grid(gx, static_cast<unsigned>(B));
    const int G = mark_group(a.P, B, aligned);
    if (G > 1)
        select_mark_shared<<<dim3(gx, static_cast<unsigned>((B + G - 1) / G)), kSelBlock, 0, s>>>(a, bt, B, G);
    else
        select_mark<<<grid, kSelBlock, 0, s>>>(a, bt, aligned);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    select_scan<false><<<dim3(groups, B), kScanBlock, 0, s>>>(a, bt);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (groups <= static_cast<unsigned>(kEarlyGroups))
        select_scatter<true><<<grid, kSelBlock, 0, s>>>(a, bt, aligned);
    else
        select_scatter<false><<<grid, kSelBlock, 0, s>>>(a, bt, aligned);
    return hipGetLastError();
}

hipError_t launch_select_after_mark(const SelectArgs& a, bool aligned, hipStream_t s)
{
    const unsigned gx = static_cast<unsigned>((a.n_tiles + kWavesPerBlock - 1) / kWavesPerBlock);
    const unsigned groups = static_cast<unsigned>((a.n_tiles + kScanBlock - 1) / kScanBlock);
    if (groups > static_cast<unsigned>(kMaxGroups)) return hipErrorInvalidValue;
    SelectBatch bt;
    memset(&bt, 0, sizeof bt);
    if (a.n_tiles <= 8 * kDirectMaxBlocks) return launch_direct<8>(a, bt, 1, aligned, true, s);
    if (a.n_tiles <= kDirectMaxTiles) return launch_direct<16>(a, bt, 1, aligned, true, s);
    select_scan<true><<<groups, kScanBlock, 0, s>>>(a, bt);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (groups <= static_cast<unsigned>(kEarlyGroups))
        select_scatter<true><<<gx, kSelBlock, 0, s>>>(a, bt, aligned);
    else
        select_scatter<false><<<gx, kSelBlock, 0, s>>>(a, bt, aligned);
    return hipGetLastError();
}

// Enough lanes for `capacity` entries (the count is only known on the
// device); lanes past the count exit.
template <int MODE, int E, bool STREAM>
void launch_sparse_shape(const SparseArgs& a, hipStream_t s)
{
    int64_t g = (a.capacity + int64_t(kListBlock) * E - 1) / (int64_t(kListBlock) * E);
    if (E > kShortE) {   // the shorter runs of a short list
        const int64_t m = a.capacity < short_list(E) ? a.capacity : short_list(E);
        const int64_t g_short = (m + int64_t(kListBlock) * kShortE - 1) / (int64_t(kListBlock) * kShortE);
        if (g < g_short) g = g_short;
    }
    if (g > kListMaxBlocks) g = kListMaxBlocks;
    if (g < 1) g = 1;
    sparse_apply<MODE, E, STREAM><<<static_cast<unsigned>(g), kListBlock, 0, s>>>(a);
}

// By the size of the state (20 bytes per parameter): up to 3M parameters it
// stays in the caches between pushes; beyond 16M it is larger than the 256 MB
// Infinity Cache (see sparse_apply for both sides of each line).
template <int MODE>
void launch_sparse_variant(const SparseArgs& a, hipStream_t s)
{
    if (a.P <= 3'000'000)
        launch_sparse_shape<MODE, 2, false>(a, s);
    else if (a.P <= 16'000'000)
        launch_sparse_shape<MODE, 2, true>(a, s);
    else
        launch_sparse_shape<MODE, 6, true>(a, s);
}

hipError_t launch_sparse(const SparseArgs& a, int variant, hipStream_t s)
{
    switch (variant) {
    case kernel_variant(MATH_FAST, 0): launch_sparse_variant<kernel_variant(MATH_FAST, 0)>(a, s); break;
    case kernel_variant(MATH_IEEE, 0): launch_sparse_variant<kernel_variant(MATH_IEEE, 0)>(a, s); break;
    case kernel_variant(MATH_FAST, 1): launch_sparse_variant<kernel_variant(MATH_FAST, 1)>(a, s); break;
    case kernel_variant(MATH_IEEE, 1): launch_sparse_variant<kernel_variant(MATH_IEEE, 1)>(a, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int E, bool STREAM>
void launch_scatter_shape(float* dst, int64_t P, const int32_t* idx, const float* val, const int64_t* d_count,
                          int64_t capacity, hipStream_t s)
{
    int64_t g = (capacity + int64_t(kListBlock) * E - 1) / (int64_t(kListBlock) * E);
    if (g > kListMaxBlocks) g = kListMaxBlocks;
    if (g < 1) g = 1;
    scatter_list<E, STREAM><<<static_cast<unsigned>(g), kListBlock, 0, s>>>(dst, P, idx, val, d_count, capacity);
}

// By the size of dst: up to 6 MB, where most of the grid has no entry and one
// per lane is the shorter chain; up to 40 MB, about the L2 caches; and up to
// 160 MB, inside the Infinity Cache (see scatter_list for both sides of each
// line).  Where the next launch reads dst whole, lines that stay in a cache
// are not read from HBM again, and the stores are plain until dst is far
// larger than the Infinity Cache.  A cached push without an index, STREAM as
// by the lines above against plain E = 1 and 2, same box:
//   P, transmitted   STREAM   E = 1    E = 2
//   12M, 10 %        111      116      109 us
//   25M, 30 %        237      232      231
//   39M, 30 %        377      350      356
//   60M, 10 %        533      509      515
//   100M, 30 %       953      942      942
//   300M, 10 %       2649     2710     2712
hipError_t launch_scatter(float* dst, int64_t P, const int32_t* idx, const float* val,
                          const int64_t* d_count, int64_t capacity, bool read_next, hipStream_t s)
{
    if (P <= 1'500'000)
        launch_scatter_shape<1, false>(dst, P, idx, val, d_count, capacity, s);
    else if (P <= (read_next ? 30'000'000 : 10'000'000))
        launch_scatter_shape<2, false>(dst, P, idx, val, d_count, capacity, s);
    else if (read_next && P <= 150'000'000)
        launch_scatter_shape<1, false>(dst, P, idx, val, d_count, capacity, s);
    else if (P <= 40'000'000)
        launch_scatter_shape<2, true>(dst, P, idx, val, d_count, capacity, s);
    else
        launch_scatter_shape<1, true>(dst, P, idx, val, d_count, capacity, s);
    return hipGetLastError();
}

}  // namespace fasgd
