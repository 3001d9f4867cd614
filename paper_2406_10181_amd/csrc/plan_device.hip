// Device-side construction and maintenance of a projector plan.
//
// The plan is the column-sorted copy of the two ELL projectors that the compress kernels walk
// (layout: lsp_internal.h; the host builder in plan.cpp defines its contents).  The projectors
// change when MaybeUpdate (Alg. 1) replaces them, and their values change in every iteration of
// the fitting loop, so a plan has to be cheap to make where the projectors live: on the GPU.
//
// Build.  The same bytes as the host builder, from three kernels, asynchronously on one stream:
//   1. k_plan_sort: the stored entries of a tile of 2048 rows (a chunk of Q, or as many rows of P) in the order of the
//      host's counting sorts, (subspace column, row, k), by a stable counting sort in LDS;
//   2. k_plan_deal: owners per column of T (long lists are shared between lanes, spare lanes go to the longest
//      lists), virtual columns, slots; per chunk the lists dealt to the waves by length; the pieces of the rows of P^T;
//   3. k_plan_rows: the waves' stream positions, the interleaved (LDS offset, value) rows, the entries of P^T, the steps of the tiles.
// What bounds a build is not bytes (a few MB) but the chain of launches and of dependent loads inside them, so the
// work is cut into few kernels, and small sums are taken again by every workgroup that needs them.  The form before
// this one (64-bit keys, two device-wide radix sorts, 17 to 23 launches) took 96 us of host time alone for a
// 4096 x 4096 matrix with r = 512 and d = 8; this one is done after 23 us (4096 x 11008: 27, r = 2048: 34).  The tiles are part of every plan, whatever
// the type of G that comes later, and cost a build 0 to 2 us there, 4 at r = 2048 (without them: 23, 25.5 and 29.6 us, lists sorted by bitonic sorts).
// The sums that are taken again (all chunks' longest lists in k_plan_deal, all segments and all steps of tiles in k_plan_rows) grow with the square of
// the chunks, and show only far beyond weight matrices: n = 131072 (64 chunks) 77 us, 1M 0.63 ms, 4M 4.2 ms (r = 512, d = 8; the
// form before: 275 us, 1.0 ms, 3.6 ms), and 16.8M (8192 chunks, r = 64, d = 2) 27 ms against 11.1.  With the steps summed up per chunk that is 22 ms,
// but the builds of weight matrices take 0.4 us longer.
// Errors that only the data can show (an index outside [0, r), columns too skewed for a plan) are
// left in a device status word and invalidate the plan's magic, so that a later compress call
// with it fills S with NaN instead of following it.
//
// Values-only refresh.  The plan records, for every value it holds, the flat ELL position it came
// from, so new values are dropped in place by one small kernel.
#include <algorithm>

#include "lsp_internal.h"

namespace lsp {

// What bounds it is the launch and one chain of three trips to memory (header, positions, values), so a thread takes four values at a time
// and all are in flight: 4096 x 4096, d = 8 3.7 us from call to call, with the tiles as without them (one value a thread in the lists and four in the tiles: 4.7);
// 4096 x 131072 16 us, without tiles 7.7.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_plan_refresh(uint8_t* __restrict__ plan, const float* __restrict__ P_val,
                                                      const float* __restrict__ Q_val, int m, int n, int r, int d) {
    const LoadedHeader H = load_header(plan);
    if (!same_problem(H->magic, H->m, H->n, H->r, H->d, m, n, r, d)) return;   // not this problem's plan
    const int64_t nq = (int64_t)H->q_total_rows * kWave / 4, np = (int64_t)m * d, np4 = (np + 3) / 4;
    const int64_t nt = (int64_t)H->m_total_steps * kTileCols;
    uint2* rows = reinterpret_cast<uint2*>(plan + H->off_q_rows);
    const uint4* qsrc = reinterpret_cast<const uint4*>(plan + H->off_q_src);
    uint2* pent = reinterpret_cast<uint2*>(plan + H->off_p_ent);
    const uint32_t* psrc = reinterpret_cast<const uint32_t*>(plan + H->off_p_src);
    uint16_t* msteps = reinterpret_cast<uint16_t*>(plan + H->off_m_steps);
    const uint4* msrc = reinterpret_cast<const uint4*>(plan + H->off_m_src);
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < nt + nq + np4; k += (int64_t)gridDim.x * 256) {
        if (k < nt) {                                                // four entries of one list of a tile
            const uint4 x = msrc[k];                                 // [step][h][b]
            const uint32_t src[kStepEntries] = {x.x, x.y, x.z, x.w};
            if (src[0] == kNoSource) continue;                       // (a list's entries come first)
            uint16_t parts[kStepEntries][3];
            float val[kStepEntries];                                 // (loads without a condition, so that they do not wait for one another)
#pragma unroll
            for (int e = 0; e < kStepEntries; ++e) val[e] = Q_val[src[e] != kNoSource ? src[e] : 0u];
#pragma unroll
            for (int e = 0; e < kStepEntries; ++e) value_parts(src[e] != kNoSource ? val[e] : 0.0f, parts[e]);
            const int b = (int)(k % kSetCols), h = (int)(k / kSetCols % 2);
            uint16_t* out = msteps + k / kTileCols * kWave * 8 + h * 4;
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *reinterpret_cast<uint2*>(out + (4 * b + q) * 8) = make_uint2(parts[0][q] | (uint32_t)parts[1][q] << 16, parts[2][q] | (uint32_t)parts[3][q] << 16);
        } else if (k < nt + nq) {
            const uint4 x = qsrc[k - nt];
            const uint32_t src[4] = {x.x, x.y, x.z, x.w};
            float val[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = Q_val[src[e] != kNoSource ? src[e] : 0u];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (src[e] != kNoSource) rows[(k - nt) * 4 + e].y = __float_as_uint(val[e]);
        } else {
            const int64_t p0 = (k - nt - nq) * 4;
            uint32_t at[4];
            float val[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) at[e] = psrc[p0 + e < np ? p0 + e : np - 1];
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = P_val[at[e]];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p0 + e < np) pent[p0 + e].y = __float_as_uint(val[e]);
        }
    }
}

hipError_t launch_plan_refresh(uint8_t* plan, const float* P_val, const float* Q_val,
                               int64_t m, int64_t n, int32_t r, int32_t d, hipStream_t st) {
    const int64_t work = (int64_t)plan_max_rows(n, r, d) * kWave / 4 + (int64_t)plan_max_steps(n, r, d) * kTileCols + (m * d + 3) / 4;
    const unsigned blocks = (unsigned)std::min<int64_t>((work + 255) / 256, 2048);
    hipLaunchKernelGGL(k_plan_refresh, dim3(blocks), dim3(256), 0, st, plan, P_val, Q_val, (int)m, (int)n, (int)r, (int)d);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Build.  Scratch (device, caller's workspace), carved by build_scratch().  Tiles are the nchunks chunks of Q, then the
// ptiles runs of kChunk rows of P.
struct BuildScratch {
    uint32_t* sorted_q;    // n * d: flat ELL positions j * d + k, per chunk in the order (column, j, k)
    uint32_t* sorted_p;    // m * d: the same per tile of P
    uint32_t* start;       // [tile][r + 1]: first position of each column's list inside its tile
    int32_t*  bad;         // [tile][kSubTiles]: an index outside [0, r) was seen
    int32_t*  seg_lo;      // [chunk][slot][512]: first entry (of sorted_q) of the list thread t walks
    int32_t*  seg_n;       // ... and its length
    int32_t*  p_shift;     // [tile of P][r]: position of an entry in p_ent less its position in its tile
    int32_t*  by_len_lo;   // [chunk][kMaxSlots * 512]: first entry (of sorted_q) of the lists in the order of their length, longest first
    int32_t*  by_len_n;    // ... and their length
};
constexpr int kSubTiles = 8;                       // workgroups that share a tile in k_plan_sort
constexpr int kThreadsSort = 1024;
constexpr int kWavesSort = kThreadsSort / kWave;

static size_t build_scratch(uint8_t* base, int64_t m, int64_t n, int32_t r, int32_t d, BuildScratch* out) {
    const size_t nchunks = (size_t)((n + kChunk - 1) / kChunk), ptiles = (size_t)((m + kChunk - 1) / kChunk);
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes, 256); return base ? base + at : nullptr; };
    BuildScratch s;
    s.sorted_q = reinterpret_cast<uint32_t*>(take((size_t)n * (size_t)d * 4));
    s.sorted_p = reinterpret_cast<uint32_t*>(take((size_t)m * (size_t)d * 4));
    s.start = reinterpret_cast<uint32_t*>(take((nchunks + ptiles) * ((size_t)r + 1) * 4));
    s.bad = reinterpret_cast<int32_t*>(take((nchunks + ptiles) * kSubTiles * 4));
    s.seg_lo = reinterpret_cast<int32_t*>(take(nchunks * kMaxSlots * kThreadsGQ * 4));
    s.seg_n = reinterpret_cast<int32_t*>(take(nchunks * kMaxSlots * kThreadsGQ * 4));
    s.p_shift = reinterpret_cast<int32_t*>(take(ptiles * (size_t)r * 4));
    s.by_len_lo = reinterpret_cast<int32_t*>(take(nchunks * kMaxSlots * kThreadsGQ * 4));
    s.by_len_n = reinterpret_cast<int32_t*>(take(nchunks * kMaxSlots * kThreadsGQ * 4));
    if (out) *out = s;
    return o;
}

size_t plan_build_workspace_bytes(int64_t m, int64_t n, int32_t r, int32_t d) { return build_scratch(nullptr, m, n, r, d, nullptr); }

// Exclusive sum of x over the threads of the workgroup (NW waves); total: the sum of all.  `part` is LDS for NW words.
template <int NW>
__device__ __forceinline__ int32_t block_exclusive(int32_t x, int32_t* part, int32_t& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t inc = x;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t y = __shfl_up(inc, off);
        if (lane >= off) inc += y;
    }
    __syncthreads();                                                 // the last call's parts have been read
    if (lane == kWave - 1) part[w] = inc;
    __syncthreads();
    int32_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const int32_t y = part[k];
        before += k < w ? y : 0;
        all += y;
    }
    total = all;
    return before + inc - x;
}

// Stable counting sort of a tile's entries by column.  kSubTiles workgroups share a tile: each counts all of the tile's
// columns (LDS atomics; the counts do not depend on their order), which gives it the lists' first positions and what the
// parts before its own have put there, and then places its own part: every wave takes a contiguous run, counts it, and
// walks it 64 entries at a time; entries of one column among the 64 find their order by ballots over the column's bits.
// Sharing a tile shortens the serial walk to 2 steps of 64 at d = 8.  An index outside [0, r) is recorded and taken as 0.
// Workgroups past the tiles clear the parts of the plan that no later kernel fills completely.
__global__ __launch_bounds__(kThreadsSort) void k_plan_sort(uint8_t* __restrict__ plan, PlanLayout L, BuildScratch s, const int32_t* __restrict__ P_idx,
                                                            const int32_t* __restrict__ Q_idx, int m, int n, int r, int d,
                                                            int nchunks, int ptiles, int64_t max_rows) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ int32_t s_part[kWavesSort];
    touch_args<4>();
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tile = blockIdx.x / kSubTiles, sub = blockIdx.x % kSubTiles;
    if (tile >= nchunks + ptiles) {
        const int first = (nchunks + ptiles) * kSubTiles;
        const size_t rows_end = L.off_q_rows + (size_t)max_rows * kWave * sizeof(uint2), src_end = L.off_q_src + (size_t)max_rows * kWave * 4;
        const size_t np = (size_t)m * d;
        const size_t lo[] = {0, rows_end, L.off_p_ent + np * sizeof(uint2), src_end, L.off_p_src + np * 4};
        const size_t hi[] = {L.off_q_rows, L.off_p_ent, L.off_q_src, L.off_p_src, L.off_m_steps};
#pragma unroll
        for (int k = 0; k < 5; ++k)
            for (size_t at = lo[k] + ((size_t)(blockIdx.x - first) * kThreadsSort + tid) * 4; at < hi[k]; at += (size_t)(gridDim.x - first) * kThreadsSort * 4)
                *reinterpret_cast<uint32_t*>(plan + at) = 0u;
        return;
    }
    const bool is_q = tile < nchunks;
    const int t = is_q ? tile : tile - nchunks;
    const int32_t* __restrict__ idx = is_q ? Q_idx : P_idx;
    const int64_t base = (int64_t)t * kChunk * d;                    // first entry of the tile
    const int count = (int)(((int64_t)(is_q ? n : m) * d - base) < (int64_t)kChunk * d ? (int64_t)(is_q ? n : m) * d - base : (int64_t)kChunk * d);
    const int part = kChunk / kSubTiles * d;                         // entries of a workgroup's part
    const int run = (part / kWavesSort + kWave - 1) / kWave * kWave; // entries of a wave's run
    const int my_lo = min(sub * part, count), my_hi = min(my_lo + part, count);
    int32_t* after = reinterpret_cast<int32_t*>(smem);               // [r] entries of the tile behind this part
    int32_t* before = after + r;                                     // [r] and before it
    int32_t* mine = before + r;                                      // [wave][r] entries of the wave's run, then where the next one goes
    for (int k = tid; k < (2 + kWavesSort) * r; k += kThreadsSort) after[k] = 0;
    __syncthreads();
    bool bad = false;
    constexpr int kAhead = 8;                                        // loads in flight per thread
    for (int e0 = 0; e0 < count; e0 += kAhead * kThreadsSort) {
        int32_t b[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int e = e0 + k * kThreadsSort + tid;
            b[k] = idx[base + (e < count ? e : count - 1)];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int e = e0 + k * kThreadsSort + tid;
            if (e >= count) continue;
            if (b[k] < 0 || b[k] >= r) { bad = true; b[k] = 0; }
            int32_t* which = e < my_lo ? before : e < my_hi ? mine + ((e - my_lo) / run) * r : after;
            atomicAdd(&which[b[k]], 1);
        }
    }
    bad = __syncthreads_or(bad);
    if (tid == 0) s.bad[tile * kSubTiles + sub] = bad ? 1 : 0;
    uint32_t* start = s.start + (size_t)tile * (r + 1);
    int32_t carry = 0;
    for (int b0 = 0; b0 < r; b0 += kThreadsSort) {
        const int b = b0 + tid;
        int32_t len = 0;
        if (b < r) {
            len = before[b] + after[b];
#pragma unroll
            for (int v = 0; v < kWavesSort; ++v) len += mine[v * r + b];
        }
        int32_t total;
        int32_t at = carry + block_exclusive<kWavesSort>(len, s_part, total);
        carry += total;
        if (b < r) {
            if (sub == 0) start[b] = (uint32_t)at;
            at += before[b];
#pragma unroll
            for (int v = 0; v < kWavesSort; ++v) {
                const int32_t c = mine[v * r + b];
                mine[v * r + b] = at;
                at += c;
            }
        }
    }
    if (sub == 0 && tid == 0) start[r] = (uint32_t)carry;
    __syncthreads();
    uint32_t* out = (is_q ? s.sorted_q : s.sorted_p) + base;
    int32_t* next = mine + w * r;
    const int bits = 32 - __builtin_clz((unsigned)r);                // columns are < r < 2^bits
    for (int e0 = my_lo + w * run; e0 < min(my_lo + (w + 1) * run, my_hi); e0 += kWave) {
        const int e = e0 + lane;
        const bool live = e < my_hi;
        int32_t b = idx[base + (live ? e : my_hi - 1)];
        if (!live || b < 0 || b >= r) b = 0;
        uint64_t same = __ballot(live);
        for (int k = 0; k < bits; ++k) {
            const bool bit = (b >> k) & 1;
            const uint64_t with = __ballot(bit);
            same &= bit ? with : ~with;
        }
        const int rank = __builtin_popcountll(same & (((uint64_t)1 << lane) - 1));
        if (live) {
            const int32_t at = next[b];
            out[at + rank] = (uint32_t)(base + e);
            if (rank == 0) next[b] = at + __builtin_popcountll(same);
        }
        __builtin_amdgcn_wave_barrier();                             // the next 64 entries read what this step has left
    }
}

// share of owner o (of k) of the list [s0, s1): the same integer arithmetic as the host builder
__device__ __forceinline__ void share_of(uint32_t s0, uint32_t s1, int o, int k, int32_t& lo, int32_t& hi) {
    const int64_t len = (int64_t)s1 - (int64_t)s0;
    lo = (int32_t)s0 + (int32_t)(len * o / k);
    hi = (int32_t)s0 + (int32_t)(len * (o + 1) / k);
}

// Rows of P^T: pieces of at most kRowPiece entries (one workgroup).
__device__ __forceinline__ void deal_p(uint8_t* __restrict__ plan, const PlanLayout& L, const BuildScratch& s, int r, int nchunks, int ptiles, int32_t* part) {
    const int tid = threadIdx.x;
    const uint32_t* start = s.start + (size_t)nchunks * (r + 1);
    RowItem* items = reinterpret_cast<RowItem*>(plan + L.off_p_item);
    int32_t entries = 0, pieces = 0;
    int any = 0;
    for (int a0 = 0; a0 < r; a0 += kThreadsGQ) {
        const int a = a0 + tid;
        int32_t len = 0;
        if (a < r)
            for (int t0 = 0; t0 < ptiles; t0 += 4) {
                uint32_t lo[4], hi[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t* st = start + (size_t)min(t0 + u, ptiles - 1) * (r + 1) + a;
                    lo[u] = st[0]; hi[u] = st[1];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) len += t0 + u < ptiles ? (int32_t)(hi[u] - lo[u]) : 0;
            }
        int32_t total;
        const int32_t s0 = entries + block_exclusive<kWavesGQ>(len, part, total);
        entries += total;
        const int32_t cut = a < r ? max(1, (len + kRowPiece - 1) / kRowPiece) : 0;
        int32_t at = pieces + block_exclusive<kWavesGQ>(cut, part, total);
        pieces += total;
        if (a < r) {
            int32_t pos = s0;
            for (int t = 0; t < ptiles; ++t) {
                const uint32_t lo = start[(size_t)t * (r + 1) + a], hi = start[(size_t)t * (r + 1) + a + 1];
                s.p_shift[(size_t)t * r + a] = pos - (int32_t)lo;
                pos += (int32_t)(hi - lo);
            }
            const int split = len > kRowPiece;
            any |= split;
            if (len == 0) items[at] = RowItem{a, s0, 0, 0};
            for (int32_t x = 0; x < len; x += kRowPiece) items[at++] = RowItem{a, s0 + x, min((int32_t)kRowPiece, len - x), split};
        }
    }
    any = __syncthreads_or(any);
    if (tid == 0) {
        PlanHeader* H = reinterpret_cast<PlanHeader*>(plan);
        H->p_nitems = pieces; H->p_any_split = any ? 1 : 0;
    }
}

// Sorts the lists of a chunk by length, longest first and equal lengths in their order, as the host's stable sort does: a stable radix sort
// over the length, 8 bits at a time (lengths are at most `most`, hardly ever 256 or more).  Wave w has places (w per + i) 64 + lane, i < per, before and
// after; a key is length * kLists + list.  What bounds it is the chain of barriers (six a round).  The bitonic sorts before it had 45 stages for
// 512 lists and 66, a barrier each, for 2048: the build for 4096 x 4096, r = 2048, d = 8 took 53 us with them.
constexpr int kLists = kMaxSlots * kThreadsGQ, kSortBits = 8;
__device__ __forceinline__ void sort_by_length(uint32_t (&key)[kMaxSlots], int per, int most, uint32_t* s_key, int32_t* s_count, int32_t* part) {
    constexpr int kBins = 1 << kSortBits, kEach = kBins * kWavesGQ / kThreadsGQ;
    static_assert(kBins * kWavesGQ % kThreadsGQ == 0, "every thread sums up the same number of counts");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int shift = 0, bits = 32 - __builtin_clz(most | 1); bits > 0; shift += kSortBits, bits -= kSortBits) {
        const int now = min(bits, kSortBits);
        // counts by (digit, the largest first; wave)
        auto count_of = [&](uint32_t k) { return s_count + ((kBins - 1 - (int)((k / kLists) >> shift & (kBins - 1))) * kWavesGQ + w); };
        for (int k = tid; k < kBins * kWavesGQ; k += kThreadsGQ) s_count[k] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kMaxSlots; ++i)
            if (i < per) atomicAdd(count_of(key[i]), 1);
        __syncthreads();
        int32_t sum = 0, total;
#pragma unroll
        for (int k = 0; k < kEach; ++k) sum += s_count[tid * kEach + k];
        int32_t at = block_exclusive<kWavesGQ>(sum, part, total);
#pragma unroll
        for (int k = 0; k < kEach; ++k) {
            const int32_t x = s_count[tid * kEach + k];
            s_count[tid * kEach + k] = at;
            at += x;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kMaxSlots; ++i)
            if (i < per) {
                uint64_t same = ~(uint64_t)0;
                for (int k = 0; k < now; ++k) {
                    const bool bit = (key[i] / kLists) >> (shift + k) & 1;
                    const uint64_t with = __ballot(bit);
                    same &= bit ? with : ~with;
                }
                const int rank = __builtin_popcountll(same & (((uint64_t)1 << lane) - 1));
                int32_t* next = count_of(key[i]);
                const int32_t first = *next;
                s_key[first + rank] = key[i];
                __builtin_amdgcn_wave_barrier();
                if (rank == 0) *next = first + __builtin_popcountll(same);
                __builtin_amdgcn_wave_barrier();                     // the next 64 keys read what this step has left
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kMaxSlots; ++i)
            if (i < per) key[i] = s_key[(w * per + i) * kWave + lane];
    }
}

// The lanes left over go, as the host hands them out one at a time, to the column whose owners have the longest share (ties: the lower column), as long as that
// share is at least 64 pairs: the k-th owner of a column with a list of L pairs is given away for a share of L / k, so the lanes go to the `spare` greatest of the shares L / k,
// k = owners so far and up.  The level above which all of them are given away is searched, each wave with a level of its own; then the shares just below it, which are all
// equal, in the order of the columns.  A share is taken as floor(2^s L / k): k is at most the greatest L / 64, so with 2^s above the square of that shares
// that differ do so in this number too (two fractions are 1 / k k' apart).
// (One after the other in a wave, with eight divisions and six exchanges each, 256 lanes took 180 us: this kernel for 4096 x 4096, r = 256, d = 8 190 us, now 11, d = 16 250 and 12; a raw compress there 239 us, now 53.)
__device__ __forceinline__ void give_spare_lanes(int32_t* s_own, const int32_t* s_longest, int r, int spare, int32_t* s_level, int32_t* part) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    constexpr int kCols = kThreadsGQ / kWave;
    int own[kCols], longest[kCols], most = 0;
#pragma unroll
    for (int q = 0; q < kCols; ++q) {                                // every wave has all columns
        const int b = lane + kWave * q;
        own[q] = b < r ? s_own[b] : 1; longest[q] = b < r ? s_longest[b] : 0;
        most = max(most, longest[q]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off));
    if (most < 64) return;                                           // (uniform over the workgroup)
    const int scale = 2 * (32 - __builtin_clz((unsigned)most >> 6));
    auto shares_from = [&](int own, int longest, uint64_t level) {   // how many of a column's are at the level or above it
        // (both numbers are below 2^53, and a quotient that is no whole number is further from one than its rounding)
        return max(0, (int)((double)((uint64_t)longest << scale) / (double)level) - own + 1);
    };
    auto all_from = [&](uint64_t level) {
        int sum = 0;
#pragma unroll
        for (int q = 0; q < kCols; ++q) sum += shares_from(own[q], longest[q], level);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        return sum;
    };
    // the least level from 64 on with no more than `spare` shares at it or above it
    uint64_t low = (uint64_t)64 << scale, high = ((uint64_t)most << scale) + 1;
    const uint64_t least = low;
    for (int turn = 0; low < high; turn ^= kWavesGQ) {
        const uint64_t width = high - low;
        const int at_level = all_from(low + width * (unsigned)w / kWavesGQ);
        if (lane == 0) s_level[turn + w] = at_level;
        __syncthreads();
        uint64_t below = low, above = high;                          // levels with too many, and one more; with few enough
#pragma unroll
        for (int k = kWavesGQ - 1; k >= 0; --k) {
            const uint64_t level = low + width * (unsigned)k / kWavesGQ;
            if (s_level[turn + k] <= spare) above = level;
            else { below = level + 1; break; }
        }
        low = below; high = above;
    }
    const int mine = tid < r ? s_own[tid] : 1, length = tid < r ? s_longest[tid] : 0;
    const int given = shares_from(mine, length, high);
    const int next = high > least ? shares_from(mine, length, high - 1) - given : 0;   // one or none
    int32_t total, equal;
    (void)block_exclusive<kWavesGQ>(given, part, total);
    const int place = block_exclusive<kWavesGQ>(next, part, equal);
    if (tid < r) s_own[tid] = mine + given + (next && place < spare - total ? 1 : 0);
}

// One workgroup of 512 threads per chunk, one for P, and, if there are to be tiles, one more per chunk for their tables (in the first
// one they would be another 1.3 of then 10 us).  Every chunk's workgroup finds the owners of all columns (they
// depend on all chunks) and the virtual columns, then deals its chunk's lists to the waves, or sorts them into tiles; the first one also writes
// the tables and the header.  A plan that cannot be (an index outside [0, r), more lists than the lanes can carry) is
// left without its magic, so that compress calls with this buffer fill S with NaN.
__global__ __launch_bounds__(kThreadsGQ) void k_plan_deal(uint8_t* __restrict__ plan, PlanLayout L, BuildScratch s, int m, int n, int r, int d, int nchunks,
                                                          int ptiles, int cap, int32_t* __restrict__ status_out) {
    __shared__ int32_t s_own[LSP_MAX_R], s_first[LSP_MAX_R], s_part[kWavesGQ];
    __shared__ int16_t s_vcol[kLists], s_vown[kLists];
    __shared__ int32_t s_longest[kThreadsGQ];
    __shared__ int32_t s_start[LSP_MAX_R], s_end[LSP_MAX_R];         // this chunk's lists
    __shared__ uint32_t s_key[kLists];
    __shared__ int32_t s_count[(1 << kSortBits) * kWavesGQ];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if ((int)blockIdx.x == nchunks) { deal_p(plan, L, s, r, nchunks, ptiles, s_part); return; }
    const bool for_tiles = (int)blockIdx.x > nchunks;                 // this workgroup writes the chunk's tile tables, otherwise its lists'
    const int c = for_tiles ? (int)blockIdx.x - nchunks - 1 : (int)blockIdx.x;
    int bad = 0;
    for (int k = tid; k < (nchunks + ptiles) * kSubTiles; k += kThreadsGQ) bad |= s.bad[k];
    int32_t vneed = 0;
    for (int b0 = 0; b0 < r; b0 += kThreadsGQ) {
        const int b = b0 + tid;
        int32_t longest = 0;
        if (b < r) {
            constexpr int kAhead = 8;                                // (loads without a condition, so that they do not wait for one another)
            for (int k0 = 0; k0 < nchunks; k0 += kAhead) {
                int32_t lo[kAhead], hi[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const uint32_t* st = s.start + (size_t)min(k0 + u, nchunks - 1) * (r + 1) + b;
                    lo[u] = (int32_t)st[0]; hi[u] = (int32_t)st[1];
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    longest = max(longest, hi[u] - lo[u]);
                    if (k0 + u == c) { s_start[b] = lo[u]; s_end[b] = hi[u]; }
                }
            }
        }
        const int32_t own = b < r ? max(1, (longest + cap - 1) / cap) : 0;
        if (b < r) s_own[b] = own;
        if (b0 == 0) s_longest[tid] = longest;
        int32_t total;
        (void)block_exclusive<kWavesGQ>(own, s_part, total);
        vneed += total;
    }
    __syncthreads();
    if (vneed < kThreadsGQ) give_spare_lanes(s_own, s_longest, r, kThreadsGQ - vneed, s_count, s_part);   // (r < 512 here, because every column has an owner already)
    __syncthreads();
    int32_t V = 0;
    int shared = 0;
    for (int b0 = 0; b0 < r; b0 += kThreadsGQ) {                     // first virtual column of each column
        const int b = b0 + tid;
        const int32_t own = b < r ? s_own[b] : 0;
        int32_t total;
        const int32_t first = V + block_exclusive<kWavesGQ>(own, s_part, total);
        if (b < r) s_first[b] = first;
        V += total;
        shared |= own > 1;
    }
    shared = __syncthreads_or(shared);
    bad = __syncthreads_or(bad);
    const int32_t status = bad ? LSP_ERR_INDEX : V > kLists ? LSP_ERR_SKEW : LSP_OK;
    const bool first_one = c == 0 && !for_tiles;
    if (status_out && first_one && tid == 0) *status_out = status;
    if (status != LSP_OK) return;                                    // the magic has been cleared with the rest of the header
    for (int v = tid; v < kLists; v += kThreadsGQ) { s_vcol[v] = -1; s_vown[v] = 0; }
    __syncthreads();
    for (int b = tid; b < r; b += kThreadsGQ)
        for (int o = 0; o < s_own[b]; ++o) { s_vcol[s_first[b] + o] = (int16_t)b; s_vown[s_first[b] + o] = (int16_t)o; }
    __syncthreads();
    const int nslots = max(1, (V + kThreadsGQ - 1) / kThreadsGQ);
    if (first_one) {
        uint16_t* vcol = reinterpret_cast<uint16_t*>(plan + L.off_q_vcol);
        uint16_t* vcnt = reinterpret_cast<uint16_t*>(plan + L.off_q_vcnt);
        for (int v = tid; v < nslots * kThreadsGQ; v += kThreadsGQ) {
            const int b = s_vcol[v];
            vcol[v] = b < 0 ? (uint16_t)kNoColumn : (uint16_t)((uint32_t)b | (s_own[b] > 1 ? kSharedColumn : 0u));
            vcnt[v] = (b >= 0 && s_vown[v] == 0) ? (uint16_t)s_own[b] : (uint16_t)0;
        }
        if (tid == 0) {
            PlanHeader* H = reinterpret_cast<PlanHeader*>(plan);
            H->magic = kPlanMagic; H->m = m; H->n = n; H->r = r; H->d = d; H->nchunks = nchunks;
            H->nslots = nslots; H->nvcols = V; H->list_cap = cap;
            H->q_any_shared = shared ? 1 : 0; H->q_permuted = nslots == 1 ? 1 : 0;
            H->off_q_seg = L.off_q_seg; H->off_q_vcol = L.off_q_vcol; H->off_q_vcnt = L.off_q_vcnt; H->off_q_perm = L.off_q_perm;
            H->off_q_rows = L.off_q_rows; H->off_p_item = L.off_p_item; H->off_p_ent = L.off_p_ent; H->total_bytes = L.total;
            H->off_q_src = L.off_q_src; H->off_p_src = L.off_p_src;
            if (gridDim.x > (unsigned)nchunks + 1) {                 // (the header has been cleared)
                H->off_m_seg = L.off_m_seg; H->off_m_cols = L.off_m_cols; H->off_m_steps = L.off_m_steps; H->off_m_src = L.off_m_src;
            }
        }
    }
    // which virtual column each thread walks (lists dealt to the waves by length when there is one slot)
    uint32_t* seg = reinterpret_cast<uint32_t*>(plan + L.off_q_seg);
    uint16_t* perm = reinterpret_cast<uint16_t*>(plan + L.off_q_perm);
    auto list_of = [&](int v, int32_t& lo, int32_t& hi) {
        const int b = s_vcol[v];
        lo = hi = 0;
        if (b >= 0) share_of((uint32_t)s_start[b], (uint32_t)s_end[b], s_vown[v], s_own[b], lo, hi);
    };
    const bool permuted = nslots == 1;
    const int k_of_w = w < kWavesGQ / 2 ? w : kWavesGQ + kWavesGQ / 2 - 1 - w;      // group of 64 lists that wave w walks
    int32_t lo, hi;
    // by length: with one slot for both kinds of lists, with several for the tiles only
    if (permuted || for_tiles) {
        uint32_t key[kMaxSlots];
#pragma unroll
        for (int i = 0; i < kMaxSlots; ++i) {
            const int v = (w * nslots + i) * kWave + lane;
            lo = hi = 0;
            if (i < nslots) list_of(v, lo, hi);
            key[i] = (uint32_t)(hi - lo) * kLists + (uint32_t)v;
        }
        sort_by_length(key, nslots, min(cap, kChunk * d), s_key, s_count, s_part);
        __syncthreads();
    }
    auto by_len = [&](int place) -> int { return (int)(s_key[place] % kLists); };      // virtual column at a place of the sorted order
    if (!for_tiles) {
        const int walked_p = permuted ? by_len(k_of_w * kWave + lane) : k_of_w * kWave + lane;
        perm[(size_t)c * kThreadsGQ + tid] = (uint16_t)walked_p;
        for (int slot = 0; slot < nslots; ++slot) {
            list_of(permuted ? walked_p : slot * kThreadsGQ + tid, lo, hi);
            const size_t at = ((size_t)c * nslots + slot) * kThreadsGQ + tid;
            s.seg_lo[at] = lo;
            s.seg_n[at] = hi - lo;
            int32_t longest = hi - lo;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off));
            if (lane == 0) seg[((size_t)c * nslots + slot) * kWavesGQ + w] = (uint32_t)((longest + kSegBatch - 1) / kSegBatch * kSegBatch);
        }
        return;
    }
    // tiles of 32 lists
    const int ntiles = (V + kTileCols - 1) / kTileCols;
    for (int place = tid; place < ntiles * kTileCols; place += kThreadsGQ) {
        lo = hi = 0;
        if (place < V) list_of(by_len(place), lo, hi);
        const size_t at = (size_t)c * kLists + place;
        s.by_len_lo[at] = lo;
        s.by_len_n[at] = hi - lo;
    }
    uint32_t* cols = reinterpret_cast<uint32_t*>(plan + L.off_m_cols) + (size_t)c * kWavesMM * kSetCols * kWaveTiles;
    for (int k = tid; k < kWavesMM * kSetCols * kWaveTiles; k += kThreadsGQ) {
        const int i = k % kWaveTiles, b = k / kWaveTiles % kSetCols, wave = k / kWaveTiles / kSetCols, t = tile_of_wave(i, wave);
        uint32_t x = 0;
        if (t < ntiles) {
            const int p0 = t * kTileCols + b, p1 = p0 + kSetCols;
            x = (uint32_t)(p0 < V ? by_len(p0) : p0) | (uint32_t)(p1 < V ? by_len(p1) : p1) << 16;
        }
        cols[k] = x;
    }
    if (tid < kWavesMM) {
        TileSeg sg{};
#pragma unroll
        for (int i = 0; i < kWaveTiles; ++i) {
            const int t = tile_of_wave(i, tid);
            sg.len[i] = (uint16_t)(t < ntiles ? (s_key[t * kTileCols] / kLists + kStepEntries - 1) / kStepEntries : 0);
            sg.steps += sg.len[i];
        }
        reinterpret_cast<TileSeg*>(plan + L.off_m_seg)[(size_t)c * kWavesMM + tid] = sg;   // (first_step: k_plan_rows)
    }
}

// First row of segment cs of wave w's stream: the streams follow one another, each behind kStreamSlack padding rows of
// the one before.  (w = kWavesGQ, cs = 0: all rows.)  Summed anew by every workgroup, all of its threads together.
constexpr int kThreadsRows = 512;
__device__ __forceinline__ uint32_t stream_row(const uint32_t* __restrict__ seg, int ncs, int w, int cs, int32_t* part) {
    int32_t sum = 0;
    for (int k = threadIdx.x; k < ncs * kWavesGQ; k += kThreadsRows) {
        const int kw = k % kWavesGQ, kc = k / kWavesGQ;
        if (kw < w || (kw == w && kc < cs)) sum += (int32_t)seg[k];
    }
    int32_t total;
    (void)block_exclusive<kThreadsRows / kWave>(sum, part, total);
    return (uint32_t)total + (uint32_t)w * kStreamSlack;
}

// Sum over the calling thread's share of the steps of the tiles before wave w's in chunk c (all: w = 0, c = nchunks).
__device__ __forceinline__ int32_t steps_before(const TileSeg* __restrict__ seg, int w, int c) {
    int32_t sum = 0;
    for (int k = threadIdx.x; k < c * kWavesMM + w; k += kThreadsRows) sum += (int32_t)seg[k].steps;
    return sum;
}

// The steps of a wave's tiles in one chunk, dealt to kTileParts workgroups in runs of 16.  A thread makes the four entries of one list in
// one step.  What bounds this is the chain segment -> list -> entries -> values -> store, each link a trip to memory that another XCD
// has just written (1 us and more), so a thread has one chain only, and the sum that says where the steps go hides behind it.
constexpr int kTileParts = 2;
__device__ __forceinline__ void plan_tiles(uint8_t* __restrict__ plan, const PlanLayout& L, const BuildScratch& s, const float* __restrict__ Q_val, int d, int c, int w,
                                           int tile_part, int32_t* part) {
    constexpr int kRun = kThreadsRows / kTileCols;
    TileSeg* seg = reinterpret_cast<TileSeg*>(plan + L.off_m_seg);
    uint16_t* steps_out = reinterpret_cast<uint16_t*>(plan + L.off_m_steps);
    uint32_t* src_out = reinterpret_cast<uint32_t*>(plan + L.off_m_src);
    const TileSeg sg = seg[(size_t)c * kWavesMM + w];
    const int32_t sum = steps_before(seg, w, c);
    const uint32_t* sorted = s.sorted_q + (size_t)c * kChunk * d;
    const int bb = threadIdx.x % kTileCols, h = bb / kSetCols, b = bb % kSetCols;
    uint32_t first = 0;
    for (int step0 = tile_part * kRun; step0 == tile_part * kRun || step0 < (int)sg.steps; step0 += kTileParts * kRun) {
        const int step = step0 + (int)threadIdx.x / kTileCols;
        uint32_t src[kStepEntries] = {0, 0, 0, 0};
        bool has[kStepEntries] = {false, false, false, false};
        float val[kStepEntries];
        if (step < (int)sg.steps) {
            int tile = 0, before = 0, end = 0;                        // before: steps of the tiles before
#pragma unroll
            for (int i = 0; i < kWaveTiles - 1; ++i) {
                end += sg.len[i];
                if (step >= end) { tile = i + 1; before = end; }
            }
            const size_t place = (size_t)c * kLists + (size_t)tile_of_wave(tile, w) * kTileCols + bb;
            const int lo = s.by_len_lo[place], n = s.by_len_n[place], e0 = (step - before) * kStepEntries;
#pragma unroll
            for (int k = 0; k < kStepEntries; ++k) has[k] = e0 + k < n;
#pragma unroll
            for (int k = 0; k < kStepEntries; ++k) src[k] = sorted[has[k] ? lo + e0 + k : 0];
        }
#pragma unroll
        for (int k = 0; k < kStepEntries; ++k) val[k] = Q_val[src[k]];
#pragma unroll
        for (int k = 0; k < kStepEntries; ++k) {
            val[k] = has[k] ? val[k] : 0.0f;
            src[k] = has[k] ? src[k] : kNoSource;
        }
        if (step0 == tile_part * kRun) {                              // all threads are here
            int32_t total;
            (void)block_exclusive<kThreadsRows / kWave>(sum, part, total);
            first = (uint32_t)total;
            if (tile_part == 0 && threadIdx.x == 0) seg[(size_t)c * kWavesMM + w].first_step = first;
        }
        if (step >= (int)sg.steps) continue;
        uint16_t parts[kStepEntries][3];
#pragma unroll
        for (int k = 0; k < kStepEntries; ++k) value_parts(val[k], parts[k]);
        uint16_t* out = steps_out + (size_t)(first + step) * kWave * 8 + h * 4;                 // [lane][h][4]
#pragma unroll
        for (int q = 0; q < 3; ++q)
            *reinterpret_cast<uint2*>(out + (4 * b + q) * 8) = make_uint2(parts[0][q] | (uint32_t)parts[1][q] << 16, parts[2][q] | (uint32_t)parts[3][q] << 16);
#pragma unroll
        for (int k = 0; k < kStepEntries; ++k)
            out[(4 * (b / 4 * 4 + k) + 3) * 8 + b % 4] =
                (uint16_t)(src[k] != kNoSource ? chunk_unit_offset(src[k] / (uint32_t)d - (uint32_t)c * kChunk) : (uint32_t)kChunk * 8u);
        *reinterpret_cast<uint4*>(src_out + ((size_t)(first + step) * 2 + h) * kWave + b * 4) = make_uint4(src[0], src[1], src[2], src[3]);
    }
}

// The interleaved rows: workgroup cs * 8 + w writes one segment, the next eight the waves' slack rows (and the header's stream
// positions), `pblocks` the entries of P^T, nchunks * 16 the tiles' steps (if there are to be any), the rest clears what lies behind the last row and the last step.
__global__ __launch_bounds__(kThreadsRows) void k_plan_rows(uint8_t* __restrict__ plan, PlanLayout L, BuildScratch s, const int32_t* __restrict__ P_idx,
                                                            const float* __restrict__ P_val, const float* __restrict__ Q_val, int m, int r, int d,
                                                            int nchunks, int pblocks, int64_t max_rows, bool with_tiles, float* __restrict__ zero) {
    touch_args<4>();
    PlanHeader* H = reinterpret_cast<PlanHeader*>(plan);
    if (H->magic != kPlanMagic) {
        if (zero)
            for (int k = (int)blockIdx.x * kThreadsRows + threadIdx.x; k < r * r; k += (int)gridDim.x * kThreadsRows) zero[k] = 0.0f;
        return;
    }
    __shared__ int32_t s_part[kThreadsRows / kWave];
    __shared__ int32_t s_lo[kWave], s_n[kWave];
    const int tid = threadIdx.x;
    const int nslots = H->nslots, ncs = nchunks * nslots;
    const uint32_t* seg = reinterpret_cast<const uint32_t*>(plan + L.off_q_seg);
    uint2* rows = reinterpret_cast<uint2*>(plan + L.off_q_rows);
    uint32_t* qsrc = reinterpret_cast<uint32_t*>(plan + L.off_q_src);
    const uint32_t pad = (uint32_t)kChunk * 16u;
    int blk = blockIdx.x;
    const int segments = nchunks * kMaxSlots * kWavesGQ, slack = kWavesGQ;
    const int tiles = with_tiles ? nchunks * kWavesMM * kTileParts : 0;
    if (blk < segments) {
        if (blk >= ncs * kWavesGQ) return;
        const int cs = blk / kWavesGQ, w = blk % kWavesGQ, c = cs / nslots;
        if (tid < kWave) {
            const size_t at = (size_t)cs * kThreadsGQ + w * kWave + tid;
            s_lo[tid] = s.seg_lo[at]; s_n[tid] = s.seg_n[at];
        }
        const int len = (int)seg[(size_t)cs * kWavesGQ + w];
        const uint32_t row0 = stream_row(seg, ncs, w, cs, s_part);   // (its barriers also order s_lo and s_n)
        const uint32_t* sorted = s.sorted_q + (size_t)c * kChunk * d;
        // a thread takes rows 2 p and 2 p + 1 of a lane, eight entries in flight
        constexpr int kAhead = 4;
        for (int q0 = 0; q0 < len / 2 * kWave; q0 += kAhead * kThreadsRows) {
            uint32_t src[kAhead][2];
            float val[kAhead][2];
            bool has[kAhead][2];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const int q = q0 + k * kThreadsRows + tid, lane = q % kWave, e = q / kWave * 2;
                const bool in = e < len;
                const int lo = s_lo[lane], n = s_n[lane];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    has[k][h] = in && e + h < n;
                    src[k][h] = sorted[has[k][h] ? lo + e + h : 0];  // (loads without a condition, so that they do not wait for one another)
                }
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float v = Q_val[src[k][h]];
                    val[k][h] = has[k][h] ? v : 0.0f;
                    src[k][h] = has[k][h] ? src[k][h] : kNoSource;
                }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const int q = q0 + k * kThreadsRows + tid, lane = q % kWave, e = q / kWave * 2;
                if (e >= len) continue;
                uint32_t off[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) off[h] = src[k][h] != kNoSource ? chunk_col_offset(src[k][h] / (uint32_t)d - (uint32_t)c * kChunk) : pad;
                const size_t slot = ((size_t)((row0 + e) >> 1) * kWave + lane) * 2;
                *reinterpret_cast<uint4*>(rows + slot) = make_uint4(off[0], __float_as_uint(val[k][0]), off[1], __float_as_uint(val[k][1]));
                *reinterpret_cast<uint2*>(qsrc + slot) = make_uint2(src[k][0], src[k][1]);
            }
        }
        return;
    }
    blk -= segments;
    if (blk < slack) {                                               // slack rows behind wave w's stream
        const uint32_t first = stream_row(seg, ncs, blk, 0, s_part), next = stream_row(seg, ncs, blk + 1, 0, s_part);
        for (int q = tid; q < kStreamSlack / 2 * kWave; q += kThreadsRows) {
            const size_t slot = ((size_t)((next - kStreamSlack) >> 1) * kWave + q) * 2;
            *reinterpret_cast<uint4*>(rows + slot) = make_uint4(pad, 0u, pad, 0u);
            *reinterpret_cast<uint2*>(qsrc + slot) = make_uint2(kNoSource, kNoSource);
        }
        if (tid == 0) {
            H->q_stream_row[blk] = first;
            if (blk == kWavesGQ - 1) H->q_total_rows = (int32_t)next;
        }
        return;
    }
    blk -= slack;
    if (blk < pblocks) {
        uint2* pent = reinterpret_cast<uint2*>(plan + L.off_p_ent);
        uint32_t* psrc = reinterpret_cast<uint32_t*>(plan + L.off_p_src);
        const int64_t np = (int64_t)m * d;
        for (int64_t p = (int64_t)blk * kThreadsRows + tid; p < np; p += (int64_t)pblocks * kThreadsRows) {
            const uint32_t src = s.sorted_p[p];
            const int64_t t = p / ((int64_t)kChunk * d);
            const int64_t at = p - t * kChunk * d + s.p_shift[t * r + P_idx[src]];
            pent[at] = make_uint2(src / (uint32_t)d, __float_as_uint(P_val[src]));
            psrc[at] = src;
        }
        return;
    }
    blk -= pblocks;
    if (blk < tiles) {
        plan_tiles(plan, L, s, Q_val, d, blk / kTileParts / kWavesMM, blk / kTileParts % kWavesMM, blk % kTileParts, s_part);
        return;
    }
    blk -= tiles;
    const int zblocks = (int)gridDim.x - segments - slack - pblocks - tiles;
    // (both sums first: their barriers would wait for the stores)
    int32_t steps = with_tiles ? steps_before(reinterpret_cast<const TileSeg*>(plan + L.off_m_seg), 0, nchunks) : 0;
    const int64_t used = (int64_t)stream_row(seg, ncs, kWavesGQ, 0, s_part) * kWave, most = with_tiles ? max_rows * kWave : 0;
    (void)block_exclusive<kThreadsRows / kWave>(steps, s_part, steps);
    for (int64_t k = used / 2 + (int64_t)blk * kThreadsRows + tid; k < most / 2; k += (int64_t)zblocks * kThreadsRows) {
        reinterpret_cast<uint4*>(rows)[k] = make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint2*>(qsrc)[k] = make_uint2(0u, 0u);
    }
    if (!with_tiles) return;
    if (blk == 0 && tid == 0) H->m_total_steps = (uint32_t)(steps + kStepsAhead);
    uint4* msteps = reinterpret_cast<uint4*>(plan + L.off_m_steps);
    uint2* msrc = reinterpret_cast<uint2*>(plan + L.off_m_src);
    const int64_t steps_end = (int64_t)(L.off_m_src - L.off_m_steps) / 16, src_end = (int64_t)(L.total - L.off_m_src) / 8;
    for (int64_t k = (int64_t)steps * kWave + (int64_t)blk * kThreadsRows + tid; k < steps_end; k += (int64_t)zblocks * kThreadsRows) {
        msteps[k] = make_uint4(0u, 0u, 0u, 0u);
        const uint32_t none = k < (int64_t)(steps + kStepsAhead) * kWave ? kNoSource : 0u;
        if (k < src_end) msrc[k] = make_uint2(none, none);
    }
}

hipError_t launch_plan_build(const int32_t* P_idx, const float* P_val, const int32_t* Q_idx, const float* Q_val,
                             int64_t m, int64_t n, int32_t r, int32_t d, uint8_t* plan, uint8_t* workspace,
                             int32_t* status_out, hipStream_t st, bool with_tiles, float* zero) {
    BuildScratch s;
    build_scratch(workspace, m, n, r, d, &s);
    const PlanLayout L = plan_layout(m, n, r, d);
    const int nchunks = (int)((n + kChunk - 1) / kChunk), ptiles = (int)((m + kChunk - 1) / kChunk);
    const int64_t max_rows = (int64_t)plan_max_rows(n, r, d);
    hipError_t e;
    const size_t lds = (size_t)(2 + kWavesSort) * r * sizeof(int32_t);
    if ((e = allow_dynamic_lds<k_plan_sort, (size_t)(2 + kWavesSort) * LSP_MAX_R * sizeof(int32_t)>()) != hipSuccess) return e;
    const unsigned clear = (unsigned)std::min<size_t>((L.off_q_rows + (L.off_p_ent - L.off_p_item)) / (4 * kThreadsSort) + 1, 256);
    hipLaunchKernelGGL(k_plan_sort, dim3((unsigned)(nchunks + ptiles) * kSubTiles + clear), dim3(kThreadsSort), lds, st, plan, L, s, P_idx, Q_idx,
                       (int)m, (int)n, (int)r, (int)d, nchunks, ptiles, max_rows);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_plan_deal, dim3((unsigned)nchunks * (with_tiles ? 2 : 1) + 1), dim3(kThreadsGQ), 0, st, plan, L, s, (int)m, (int)n, (int)r, (int)d, nchunks, ptiles,
                       plan_list_cap(r, d), status_out);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int pblocks = (int)std::min<int64_t>((m * d + kThreadsRows - 1) / kThreadsRows, 512);
    // (a plan without tiles is used at once and never compared: nothing behind its last row is cleared)
    const int zblocks = with_tiles ? (int)std::min<int64_t>((max_rows * kWave / 2 + 4 * kThreadsRows - 1) / (4 * kThreadsRows), 512) : 1;
    const int segments = nchunks * kMaxSlots * kWavesGQ + kWavesGQ, tiles = with_tiles ? nchunks * kWavesMM * kTileParts : 0;
    hipLaunchKernelGGL(k_plan_rows, dim3((unsigned)(segments + pblocks + tiles + zblocks)), dim3(kThreadsRows), 0, st, plan, L, s,
                       P_idx, P_val, Q_val, (int)m, (int)r, (int)d, nchunks, pblocks, max_rows, with_tiles, zero);
    return hipGetLastError();
}

}  // namespace lsp
