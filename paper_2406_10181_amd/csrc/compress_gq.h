// Compress, kernel A: T = G Q, the template code; compress_gq_bf16.hip, compress_gq_f16.hip and compress_gq_f32.hip
// instantiate it.  See compress.hip for the path as a whole.
#pragma once

#include <algorithm>
#include <type_traits>

#include "compress_common.h"

namespace lsp {

// ----------------------------------------------------------------------------------------------
// G is staged as it is stored, in 16-byte LDS units of one column and the rows of a plane (8 rows of fp16 / bf16, 4 of fp32:
// [plane][column][rows]), so one 128-bit gather serves them all; 16-bit elements are widened in registers when they are
// used (exact: a shift or mask for bf16, a conversion for fp16).
// A workgroup has a block of one plane and holds two chunks, the one being consumed and the one being staged.  That is
// 64 KB of LDS, and with at most 128 registers per lane two workgroups share a CU, four waves per SIMD: a single wave
// issues a vector instruction only every 5 to 6 cycles, so a SIMD needs more than two resident waves to stay busy
// while some of them wait at a barrier.  (fp32 with 16-row blocks in four planes and one workgroup a CU took
// 40.5 us on 4096 x 4096, r = 512, d = 8, now 29; with two planes of one chunk the sums and the rows in flight
// did not fit 128 registers.)
template <typename D> constexpr int kRowsGQ = 16 / D::size;           // rows of a block
template <typename D> __device__ __forceinline__ void widen2(uint32_t w, float& lo, float& hi);
template <> __device__ __forceinline__ void widen2<BF16>(uint32_t w, float& lo, float& hi) {
    lo = __uint_as_float(w << 16); hi = __uint_as_float(w & 0xFFFF0000u);
}
template <> __device__ __forceinline__ void widen2<F16>(uint32_t w, float& lo, float& hi) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    h2 h; __builtin_memcpy(&h, &w, 4);
    lo = (float)h.x; hi = (float)h.y;
}

// Rows 2k and 2k+1 of two adjacent columns sit in the dwords a (row 2k) and b (row 2k+1); the unit
// of the even column takes their low halves, that of the odd column their high halves (one byte permute).
__device__ __forceinline__ uint32_t pair_rows(uint32_t a, uint32_t b, bool odd_column) {
    return __builtin_amdgcn_perm(b, a, odd_column ? 0x07060302u : 0x05040100u);
}

// Fetches and stages a chunk of the block's rows, 4 columns a thread: 512 threads cover the 2048 columns.  Rows past the matrix
// are read from its last row and columns past it from its first ones or from the next row (always a valid address): what
// they hold is never used, as the plan has no entry for such a column and the sums of such a row are not stored.
// WHOLE: n % 4 == 0.  Otherwise a piece that would end behind the matrix's last element is read from where it ends with
// it and put right when it is staged.
template <typename D, bool WHOLE> struct ChunkStager {
    static constexpr int R = kRowsGQ<D>;
    static constexpr int kPieceDwords = D::size;                      // 4 elements
    typedef uint32_t Piece __attribute__((ext_vector_type(kPieceDwords)));
    typedef Piece Loose __attribute__((aligned(WHOLE ? 4 * D::size : D::size)));
    Piece pre[R];
    int late, late_from;                                              // rows from late_from on were read `late` elements early

    __device__ __forceinline__ void fetch(const typename D::elem* __restrict__ G, int64_t i0, int m, int n, int c, int tid) {
        typedef typename D::elem E;
        const uint32_t col0 = (uint32_t)c * kChunk + (uint32_t)tid * 4;
        const uint32_t byte0 = (col0 < (uint32_t)n ? col0 : 0u) * (uint32_t)sizeof(E);
        const int last = (int)(m - 1 - i0 < R - 1 ? m - 1 - i0 : R - 1);   // rows of the block inside the matrix, less one (i0 < m)
        const char* base = reinterpret_cast<const char*>(G + i0 * (int64_t)n) + byte0;
        const uint64_t stride = (uint64_t)n * sizeof(E);
        if constexpr (WHOLE) {
#pragma unroll
            for (int t = 0; t < R; ++t) {
                pre[t] = __builtin_nontemporal_load(reinterpret_cast<const Loose*>(base));
                base += t < last ? stride : 0;
            }
        } else {
            late = 0; late_from = R;
            if (n < 4) {                                              // element by element
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    E x[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) x[q] = G[(i0 + (t < last ? t : last)) * n + (q < n ? q : n - 1)];
                    __builtin_memcpy(&pre[t], x, sizeof(x));
                }
                return;
            }
            if (i0 + last == m - 1) {
                late_from = last;
                if (col0 < (uint32_t)n && col0 + 4 > (uint32_t)n) late = (int)(col0 + 4 - (uint32_t)n);
            }
#pragma unroll
            for (int t = 0; t < R; ++t) {
                pre[t] = __builtin_nontemporal_load(reinterpret_cast<const Loose*>(base - (t >= late_from ? late : 0) * (int)sizeof(E)));
                base += t < last ? stride : 0;
            }
        }
    }
    // transposes the block and writes its 4 units (column q: all rows) into buffer `buf`
    __device__ __forceinline__ void stage(uint8_t* smem, int buf, int tid) {
        if constexpr (!WHOLE)
            if (late != 0) {
#pragma unroll
                for (int t = 0; t < R; ++t)
                    if (t >= late_from) pre[t] = drop_elements(pre[t], late);
            }
        // local column j = 4 tid + q sits at unit (j & 7) * (kChunk / 8) + (j >> 3)
        uint8_t* base = smem + buf * kPlaneStride + ((4 * (tid & 1)) * (kChunk / 8) + (tid >> 1)) * 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4 unit;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (D::size == 2) unit[k] = pair_rows(pre[2 * k][q >> 1], pre[2 * k + 1][q >> 1], q & 1);
                else unit[k] = pre[k][q];
            }
            *reinterpret_cast<u32x4*>(base + q * (kChunk / 8) * 16) = unit;
        }
    }
    // the piece without its first `by` (1 to 3) elements
    static __device__ __forceinline__ Piece drop_elements(const Piece& x, int by) {
        Piece o;
        if constexpr (D::size == 2) {
            const uint64_t v = (((uint64_t)x[1] << 32) | x[0]) >> (16 * by);
            o[0] = (uint32_t)v; o[1] = (uint32_t)(v >> 32);
        } else {
            o[0] = by == 1 ? x[1] : by == 2 ? x[2] : x[3];
            o[1] = by == 1 ? x[2] : x[3];
            o[2] = o[3] = x[3];
        }
        return o;
    }
};

__device__ __forceinline__ void gather_pair(const uint8_t* buf, const u32x4 e, u32x4 (&x)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) x[h] = *reinterpret_cast<const u32x4*>(buf + (h ? e.z : e.x));
}
template <typename D>
__device__ __forceinline__ void fma_pair(const u32x4 e, const u32x4 (&x)[2], float (&acc)[kRowsGQ<D>]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float v = __uint_as_float(h ? e.w : e.y);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (D::size == 2) {
                float lo, hi;
                widen2<D>(x[h][k], lo, hi);
                acc[2 * k]     = fmaf(v, lo, acc[2 * k]);
                acc[2 * k + 1] = fmaf(v, hi, acc[2 * k + 1]);
            } else {
                acc[k] = fmaf(v, __uint_as_float(x[h][k]), acc[k]);
            }
        }
    }
}

// One workgroup walks `nblk` consecutive row blocks (several when the grid is big: the first
// chunk of the next block is fetched and staged while the last chunk of the current one is
// consumed, and the stores of T go out under the next block's work, so that the set-up and the
// tail of a block cost nothing but for the first and the last one).
template <typename D, bool WHOLE>
__device__ __forceinline__ void gq_one_slot(ChunkStager<D, WHOLE>& stg, uint8_t* smem, const typename D::elem* __restrict__ G,
                                              const uint8_t* __restrict__ plan, const LoadedHeader& H,
                                              float* __restrict__ T, int64_t i0, int nblk, int m, int n, int r,
                                              int tid, int lane, int wave) {
    constexpr int R = kRowsGQ<D>;
    const int nchunks = H->nchunks;
    const auto* seg = as_const<uint32_t>(plan + H->off_q_seg) + wave;
    const u32x4* rp0 = reinterpret_cast<const u32x4*>(plan + H->off_q_rows) + (size_t)(as_const<PlanHeader>(plan)->q_stream_row[wave] >> 1) * kWave + lane;
    const u32x4* rp = rp0;
    const uint32_t mycol = as_const<uint16_t>(plan + H->off_q_vcol)[tid];
    const bool shared = H->q_any_shared != 0;
    const uint16_t* __restrict__ perm = reinterpret_cast<const uint16_t*>(plan + H->off_q_perm) + tid;
    const uint32_t first = perm[0];
    uint32_t walked = first;                                          // virtual column whose list this thread walks

    // ring of kPrefetch batches of plan rows in fixed register slots: a slot is consumed, then refilled with the batch four
    // further on (shifting the ring's registers would make every batch wait for its newest load)
    u32x4 ring[kPrefetch][kBatchLoads];
    auto ring_restart = [&]() {
        rp = rp0;
#pragma unroll
        for (int k = 0; k < kPrefetch; ++k)
#pragma unroll
            for (int q = 0; q < kBatchLoads; ++q) ring[k][q] = rp[(size_t)(k * kBatchLoads + q) * kWave];
        rp += (size_t)kPrefetch * kBatchLoads * kWave;
    };
    ring_restart();

    float acc[1][R];
#pragma unroll
    for (int t = 0; t < R; ++t) acc[0][t] = 0.0f;

    const uint8_t* buf = smem;
    auto step = [&](u32x4 (&slot)[kBatchLoads]) {
        u32x4 x[2][2];
        gather_pair(buf, slot[0], x[0]);
#pragma unroll
        for (int q = 0; q < kBatchLoads; ++q) {
            if (q + 1 < kBatchLoads) gather_pair(buf, slot[q + 1], x[(q + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            fma_pair<D>(slot[q], x[q & 1], acc[0]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < kBatchLoads; ++q) slot[q] = rp[(size_t)q * kWave];
        rp += (size_t)kBatchLoads * kWave;
    };

    stg.stage(smem, 0, tid);                                          // chunk 0 of the first block (fetched by the caller)
    __syncthreads();
    // Batch k of a chunk sits in ring slot (rot + k) % kPrefetch, where rot is what the chunks before left over:
    // the walk enters the unrolled slot sequence at slot rot instead of moving the ring's registers.
    static_assert(kPrefetch == 4, "the slot walk below is written for four slots");
    int rot = 0, c = 0, blk = 0;
    const int units = nblk * nchunks;                                 // (row block, chunk) pairs, in order
    int nb_next = (int)(seg[0] / kSegBatch);                          // batches of this wave in the coming chunk
    for (int u = 0; u < units; ++u) {
        const bool last_chunk = c + 1 == nchunks;
        const uint32_t next = last_chunk ? (uint32_t)tid : (uint32_t)perm[(size_t)(c + 1) * kThreadsGQ];
        const int nb = nb_next;
        nb_next = (int)(seg[(last_chunk ? 0 : c + 1) * kWavesGQ] / kSegBatch);   // arrives while this chunk is walked
        if (u + 1 < units)                                            // next chunk, maybe of the next block: lands while this one is consumed
            stg.fetch(G, i0 + (int64_t)(last_chunk ? blk + 1 : blk) * R, m, n, last_chunk ? 0 : c + 1, tid);
        buf = smem + (u & 1) * kPlaneStride;
        const bool more = u + 1 < units;
        // The next chunk is staged (into the buffer nobody reads now) in the middle of this one's
        // work rather than at its end, where every wave would wait for it; only a block's last
        // chunk with shared columns stages later, behind the merge that uses the same LDS.
        const bool stage_early = more && !(last_chunk && shared);
        int left = nb;
        switch (rot) {                                                // up to the ring's slot 0
            case 1: if (left > 0) { step(ring[1]); --left; } [[fallthrough]];
            case 2: if (left > 0) { step(ring[2]); --left; } [[fallthrough]];
            case 3: if (left > 0) { step(ring[3]); --left; } [[fallthrough]];
            default: break;
        }
        const int groups = left / kPrefetch, before = groups < 2 ? groups : 2;
        for (int g = before; g > 0; --g) {
            step(ring[0]); step(ring[1]); step(ring[2]); step(ring[3]);
        }
        if (stage_early) stg.stage(smem, (u + 1) & 1, tid);
        for (int g = groups - before; g > 0; --g) {
            step(ring[0]); step(ring[1]); step(ring[2]); step(ring[3]);
        }
        left -= groups * kPrefetch;
        if (left > 0) step(ring[0]);
        if (left > 1) step(ring[1]);
        if (left > 2) step(ring[2]);
        rot = (rot + nb) % kPrefetch;
        // The sums move to the lanes that walk the columns in the next chunk; after the last chunk
        // of a block they go home (thread t: virtual column t) and out to T.
        if (last_chunk && more) { ring_restart(); rot = 0; }          // the stream starts over; in flight during the stores
        swap_owner<R>(smem + (u & 1) * kPlaneStride, acc[0], walked, next);
        if (last_chunk) {
            const int64_t ib = i0 + (int64_t)blk * R;
            if (shared) {
                write_tile_shared<1, R>(smem, plan, H, T, acc, 1, ib, m, r, tid);   // uses the LDS of the first chunk buffer
                if (more) {
                    __syncthreads();                                  // before that LDS is staged into again
                    stg.stage(smem, (u + 1) & 1, tid);
                    __syncthreads();
                }
            } else if (mycol != kNoColumn) {
#pragma unroll
                for (int t = 0; t < R; ++t)
                    if (ib + t < m) T[(ib + t) * (int64_t)r + mycol] = acc[0][t];
            }
        }
        if (last_chunk) {                                             // the block's sums are out
#pragma unroll
            for (int t = 0; t < R; ++t) acc[0][t] = 0.0f;
            c = 0; ++blk;
            walked = first;
        } else {
            ++c;
            walked = next;
        }
    }
}

// Several columns per lane (r > 512, or columns used so unevenly that they were split): the same staging,
// plan ring and block walk as gq_one_slot, the lane's columns taken slot by slot inside each chunk.  A lane keeps its columns for all chunks (no dealing by length:
// the sums of NS columns per lane would not fit through LDS cheaply).
template <typename D, int NS, bool WHOLE>
__device__ __forceinline__ void gq_multi_slot(ChunkStager<D, WHOLE>& stg, uint8_t* smem, const typename D::elem* __restrict__ G,
                                                const uint8_t* __restrict__ plan, const LoadedHeader& H,
                                                float* __restrict__ T, int64_t i0, int nblk, int m, int n, int r,
                                                int tid, int lane, int wave) {
    constexpr int R = kRowsGQ<D>;
    const int nchunks = H->nchunks, nslots = H->nslots;
    const auto* seg = as_const<uint32_t>(plan + H->off_q_seg) + wave;
    const u32x4* rp0 = reinterpret_cast<const u32x4*>(plan + H->off_q_rows) + (size_t)(as_const<PlanHeader>(plan)->q_stream_row[wave] >> 1) * kWave + lane;
    const u32x4* rp = rp0;
    const auto* vcol = as_const<uint16_t>(plan + H->off_q_vcol);
    const bool shared = H->q_any_shared != 0;

    u32x4 ring[kPrefetch][kBatchLoads];                               // fixed register slots (see gq_one_slot)
    auto ring_restart = [&]() {
        rp = rp0;
#pragma unroll
        for (int k = 0; k < kPrefetch; ++k)
#pragma unroll
            for (int q = 0; q < kBatchLoads; ++q) ring[k][q] = rp[(size_t)(k * kBatchLoads + q) * kWave];
        rp += (size_t)kPrefetch * kBatchLoads * kWave;
    };
    ring_restart();

    float acc[NS][R];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < R; ++t) acc[s][t] = 0.0f;

    const uint8_t* buf = smem;
    auto step = [&](u32x4 (&slot)[kBatchLoads], float (&a)[R]) {
        u32x4 x[2][2];
        gather_pair(buf, slot[0], x[0]);
#pragma unroll
        for (int q = 0; q < kBatchLoads; ++q) {
            if (q + 1 < kBatchLoads) gather_pair(buf, slot[q + 1], x[(q + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            fma_pair<D>(slot[q], x[q & 1], a);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < kBatchLoads; ++q) slot[q] = rp[(size_t)q * kWave];
        rp += (size_t)kBatchLoads * kWave;
    };
    static_assert(kPrefetch == 4, "the rotation below is written for four slots");
    auto unrotate = [&](int rot) {                                    // slot 0 holds the oldest batch again
        if (rot != 0) {
            u32x4 t[kPrefetch][kBatchLoads];
#pragma unroll
            for (int k = 0; k < kPrefetch; ++k)
#pragma unroll
                for (int q = 0; q < kBatchLoads; ++q) {
                    t[k][q] = ring[(k + 1) % kPrefetch][q];
                    if (rot == 2) t[k][q] = ring[(k + 2) % kPrefetch][q];
                    if (rot == 3) t[k][q] = ring[(k + 3) % kPrefetch][q];
                }
#pragma unroll
            for (int k = 0; k < kPrefetch; ++k)
#pragma unroll
                for (int q = 0; q < kBatchLoads; ++q) ring[k][q] = t[k][q];
        }
    };

    stg.stage(smem, 0, tid);                                          // chunk 0 of the first block (fetched by the caller)
    __syncthreads();
    int rot = 0, c = 0, blk = 0;
    const int units = nblk * nchunks;
    for (int u = 0; u < units; ++u) {
        const bool last_chunk = c + 1 == nchunks;
        const bool more = u + 1 < units;
        if (more)
            stg.fetch(G, i0 + (int64_t)(last_chunk ? blk + 1 : blk) * R, m, n, last_chunk ? 0 : c + 1, tid);
        buf = smem + (u & 1) * kPlaneStride;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (s < nslots) {
                unrotate(rot);
                const int nb = (int)(seg[(c * nslots + s) * kWavesGQ] / kSegBatch);
                for (int g = nb / kPrefetch; g > 0; --g) {
                    step(ring[0], acc[s]); step(ring[1], acc[s]); step(ring[2], acc[s]); step(ring[3], acc[s]);
                }
                rot = nb % kPrefetch;
                if (rot > 0) step(ring[0], acc[s]);
                if (rot > 1) step(ring[1], acc[s]);
                if (rot > 2) step(ring[2], acc[s]);
            }
        }
        if (last_chunk) {                                             // the block's sums are complete
            const int64_t ib = i0 + (int64_t)blk * R;
            if (more) { ring_restart(); rot = 0; }                    // the stream starts over; in flight during the stores
            if (shared) {
                write_tile_shared<NS, R>(smem, plan, H, T, acc, nslots, ib, m, r, tid);   // uses the LDS of both chunk buffers
                if (more) {
                    __syncthreads();                                  // before that LDS is staged into again
                    if (tid < 2) *reinterpret_cast<f32x4*>(smem + tid * kPlaneStride + kChunk * 16) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                }
            } else {
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const uint32_t col = s < nslots ? (uint32_t)vcol[s * kThreadsGQ + tid] : kNoColumn;
                    if (col != kNoColumn) {
#pragma unroll
                        for (int t = 0; t < R; ++t)
                            if (ib + t < m) T[(ib + t) * (int64_t)r + col] = acc[s][t];
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int t = 0; t < R; ++t) acc[s][t] = 0.0f;
            c = 0; ++blk;
        } else {
            ++c;
        }
        if (more) stg.stage(smem, (u + 1) & 1, tid);               // the other buffer: nobody reads it now
        __syncthreads();                                              // the next chunk is staged; this one is no longer read
    }
}

struct NoRawCall {};
// RAW: for a call on raw ELL arrays.  (With the scatter form in the one kernel for all, the planned calls lost 1 %.)
template <typename D, bool WHOLE, bool RAW>
__global__ __launch_bounds__(kThreadsGQ, 4) void k_compress_gq(const CompressGroup, const std::conditional_t<RAW, RawCall, NoRawCall> raw) {
    constexpr int R = kRowsGQ<D>;
    extern __shared__ __align__(16) uint8_t smem[];
    const auto* grp = group_args<CompressGroup>();
    const auto pick = pick_problem(grp, grp->first_gq, (int)blockIdx.x);
    const CompressProblem& pr = pick.p;
    const int r = pick.r, d = pick.d;
    const typename D::elem* __restrict__ G = static_cast<const typename D::elem*>(pr.G);
    const uint8_t* __restrict__ plan = pr.plan;
    float* __restrict__ T = pr.T;
    float* __restrict__ S = pr.S;
    const int m = pr.m, n = pr.n;
    const int block = (int)blockIdx.x - pr.first_gq, nblocks = pr.wgs_gq, blocks_per_wg = pr.blocks_gq;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t i0 = (int64_t)block * blocks_per_wg * R;
    const int nblk = min(blocks_per_wg, (int)((m - i0 + R - 1) / R));   // row blocks of this workgroup

    ChunkStager<D, WHOLE> stg;
    stg.fetch(G, i0, m, n, 0, tid);                             // in flight while the plan's header arrives
    asm volatile("" ::: "memory");                                    // (or they would be asked for behind the comparisons below)
    const LoadedHeader H = load_header(plan);
    if (!plan_matches(H, m, n, r, d, false)) {                               // not a plan for this problem
        if constexpr (RAW) scatter_blocks<D>(G, raw, S, reinterpret_cast<float*>(smem), m, n, r, d, block, nblocks, tid, kThreadsGQ);
        else fill_s(S, __builtin_nanf(""), r, block, nblocks, tid, kThreadsGQ);
        return;
    }
    if (H->p_any_split) {
        const int64_t total = (int64_t)r * r;
        for (int64_t k = (int64_t)block * kThreadsGQ + tid; k < total; k += (int64_t)nblocks * kThreadsGQ) S[k] = 0.0f;
    }
    if (tid < 2) *reinterpret_cast<f32x4*>(smem + tid * kPlaneStride + kChunk * 16) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if (H->nslots == 1)      gq_one_slot<D, WHOLE>(stg, smem, G, plan, H, T, i0, nblk, m, n, r, tid, lane, wave);
    else if (H->nslots == 2) gq_multi_slot<D, 2, WHOLE>(stg, smem, G, plan, H, T, i0, nblk, m, n, r, tid, lane, wave);
    else                     gq_multi_slot<D, kMaxSlots, WHOLE>(stg, smem, G, plan, H, T, i0, nblk, m, n, r, tid, lane, wave);
}

// How many row blocks a workgroup takes.  A workgroup's next block is fetched while it walks the last chunk of the one
// before, so only its first block waits for memory and for the plan.  If equal shares of chunks (row blocks times chunks of
// a row) can be had from no more workgroups than the chip holds at a time, one share each: every CU is busy from start to
// end, and nothing is set up twice (kernels A and B: 2048 x 8192 and 8192 x 2048 together 45.0 -> 40.7 us, 11008 x 4096
// 66.0 -> 61.7).  Shares of more than eight chunks are halved and so on, because the two workgroups of a CU do not
// advance at the same speed.  Otherwise the workgroups are taken up as CUs fall free, and small ones even out the end:
// two blocks each on big grids, else one.
// Returns the number of workgroups.
template <int R> static unsigned share_blocks(CompressGroup& g) {
    constexpr int64_t kResident = 512;                                // two on each of 256 CUs
    int64_t work = 0, rows = 0, grid = 0;
    for (int p = 0; p < g.count; ++p) {
        work += (int64_t)((g.p[p].m + R - 1) / R) * ((g.p[p].n + kChunk - 1) / kChunk);
        rows += g.p[p].m;
    }
    auto fill = [&](auto&& blocks_of) {
        int64_t longest = 0;
        grid = 0;
        for (int p = 0; p < kMaxGroup; ++p) {
            CompressProblem& x = g.p[p];
            g.first_gq[p] = INT32_MAX;
            if (p >= g.count) continue;
            const int64_t chunks = (x.n + kChunk - 1) / kChunk, blocks = (x.m + R - 1) / R;
            const int64_t each = blocks_of(chunks);
            x.blocks_gq = (int32_t)each;
            x.wgs_gq = (int32_t)((blocks + each - 1) / each);
            g.first_gq[p] = x.first_gq = (int32_t)grid;
            grid += x.wgs_gq;
            longest = std::max(longest, each * chunks);
        }
        return longest;
    };
    for (int64_t rounds = 1; rounds <= 4; ++rounds) {
        const int64_t share = (work + rounds * kResident - 1) / (rounds * kResident);
        if (share > 8) continue;
        const int64_t longest = fill([&](int64_t chunks) { return (share + chunks - 1) / chunks; });
        if (grid <= rounds * kResident && longest * 8 <= share * 9) return (unsigned)grid;
    }
    fill([&](int64_t) { return (int64_t)(rows >= 16384 ? 2 : 1); });
    return (unsigned)grid;
}

template <typename D, bool WHOLE, bool RAW>
static hipError_t launch_gq(const CompressGroup& g, unsigned grid, const RawCall& raw, hipStream_t st) {
    constexpr size_t lds = (size_t)2 * kPlaneStride;                  // two chunk buffers
    static_assert(lds >= (size_t)kScatterRows * LSP_MAX_R * sizeof(float), "room for scatter_blocks");
    std::conditional_t<RAW, RawCall, NoRawCall> args{};
    if constexpr (RAW) args = raw;
    hipError_t e;
    if ((e = allow_dynamic_lds<k_compress_gq<D, WHOLE, RAW>, lds>()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_compress_gq<D, WHOLE, RAW>), dim3(grid), dim3(kThreadsGQ), lds, st, g, args);
    return hipGetLastError();
}

template <typename D>
static hipError_t launch_gq(CompressGroup& g, const RawCall& raw, hipStream_t st) {
    bool whole = true;
    const unsigned grid = share_blocks<kRowsGQ<D>>(g);
    for (int p = 0; p < g.count; ++p) whole = whole && g.p[p].n % 4 == 0;
    if constexpr (!std::is_same_v<D, BF16>)                           // bf16 with a kept plan: compress_mm.hip
        if (!raw.status) return whole ? launch_gq<D, true, false>(g, grid, raw, st) : launch_gq<D, false, false>(g, grid, raw, st);
    return whole ? launch_gq<D, true, true>(g, grid, raw, st) : launch_gq<D, false, true>(g, grid, raw, st);
}
}  // namespace lsp
