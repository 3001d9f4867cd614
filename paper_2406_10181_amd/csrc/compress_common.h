// Pieces shared by the translation units of the compress path (kernel A, instantiated once per storage
// type, kernel B and the launchers).
#pragma once

#include <utility>

#include "lsp_internal.h"

namespace lsp {

constexpr int kPlaneStride = kChunk * 16 + 16;   // bytes; last 16 bytes of a plane stay zero
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A plan is only followed when its header names this very problem: the offsets and counts in it
// index S and T with the call's r and m, so a plan built for other sizes (or a buffer that holds no
// plan at all) must not be walked.  Kernel A then fills S with NaN, which is how the caller sees
// the mistake (or takes the scatter form, raw calls), and kernel B does nothing; all kernels exit normally.
// tiles: kernel A of this call walks the tiles, so there must be some; kernel B asks for the same, or it would put what lies in T in the place of the NaN.
__device__ __forceinline__ bool plan_matches(const LoadedHeader& H, int m, int n, int r, int d, bool tiles) {
    const uint32_t steps = tiles ? H->m_total_steps : 1u;
    return same_problem(H->magic, H->m, H->n, H->r, H->d, m, n, r, d) && steps != 0;
}
__device__ __forceinline__ void fill_s(float* __restrict__ S, float x, int r, int block, int nblocks, int tid, int nthreads) {
    const int64_t total = (int64_t)r * r;
    for (int64_t k = (int64_t)block * nthreads + tid; k < total; k += (int64_t)nblocks * nthreads) S[k] = x;
}

// Scatter form of the raw calls, for projectors whose columns are too skewed for a plan: the same mathematics.  With a tile of T in
// LDS, every (row, column j, entry k) adds G[i][j] * Q_val[j][k] to T[i][Q_idx[j][k]]; then S[P_idx[i][k]][:] += P_val[i][k] * T[i][:]
// with global atomics.  Nearly always there is nothing to do, so it has no launch of its own (4 us of some 50 on 4096 x 4096): kernel A does
// it where it finds no plan.  Called by all threads of the workgroup; lds: kScatterRows * r floats.
constexpr int kScatterRows = 8;
template <typename D>
__device__ __forceinline__ void scatter_blocks(const typename D::elem* __restrict__ G, const RawCall& raw, float* __restrict__ S, float* Tl, int m, int n, int r, int d,
                                               int block, int nblocks, int tid, int nthreads) {
    if (*raw.status != LSP_ERR_SKEW) {                                // an index outside [0, r)
        fill_s(S, __builtin_nanf(""), r, block, nblocks, tid, nthreads);
        return;
    }
    for (int64_t i0 = (int64_t)block * kScatterRows; i0 < m; i0 += (int64_t)nblocks * kScatterRows) {
        __syncthreads();
        for (int k = tid; k < kScatterRows * r; k += nthreads) Tl[k] = 0.0f;
        __syncthreads();
        for (int64_t j = tid; j < n; j += nthreads) {
            float g[kScatterRows];
#pragma unroll
            for (int t = 0; t < kScatterRows; ++t) g[t] = (i0 + t < m) ? widen<D>(G[(i0 + t) * (int64_t)n + j]) : 0.0f;
            for (int k = 0; k < d; ++k) {
                const int b = raw.Q_idx[j * d + k];
                const float v = raw.Q_val[j * d + k];
#pragma unroll
                for (int t = 0; t < kScatterRows; ++t) atomicAdd(&Tl[t * r + b], g[t] * v);
            }
        }
        __syncthreads();
        for (int t = 0; t < kScatterRows && i0 + t < m; ++t)
            for (int k = 0; k < d; ++k) {
                const int a = raw.P_idx[(i0 + t) * d + k];
                const float v = raw.P_val[(i0 + t) * d + k];
                for (int b = tid; b < r; b += nthreads) atomicAdd(&S[(int64_t)a * r + b], v * Tl[t * r + b]);
            }
    }
}

constexpr int kBatchLoads = kSegBatch / 2;                    // 128-bit loads per batch of plan rows

// Partial sums of several owners of one column meet in LDS: every lane parks its R sums at its
// virtual column, [R][nslots * 512] floats; the first owner of a column then adds the owners'
// sums in owner order (they sit side by side) and stores the column of T.  No atomics, so the
// result does not depend on timing.  Called by all threads of the workgroup.
template <int NS, int R>
__device__ __forceinline__ void write_tile_shared(uint8_t* smem, const uint8_t* plan, const LoadedHeader& H, float* __restrict__ T,
                                                  const float (&acc)[NS][R], int nslots, int64_t i0, int m, int r, int tid) {
    __syncthreads();                                                  // the staged chunk is no longer read
    float* Tl = reinterpret_cast<float*>(smem);
    const int V = nslots * kThreadsGQ;
    const auto* vcol = as_const<uint16_t>(plan + H->off_q_vcol);
    const auto* vcnt = as_const<uint16_t>(plan + H->off_q_vcnt);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s < nslots) {
#pragma unroll
            for (int t = 0; t < R; ++t) Tl[t * V + s * kThreadsGQ + tid] = acc[s][t];
        }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s < nslots) {
            const int v = s * kThreadsGQ + tid;
            const int owners = vcnt[v];
            if (owners > 0) {
                const uint32_t bb = vcol[v] & 0x7FFFu;
                for (int t = 0; t < R; ++t) {
                    float sum = Tl[t * V + v];
                    for (int o = 1; o < owners; ++o) sum += Tl[t * V + v + o];
                    if (i0 + t < m) T[(i0 + t) * (int64_t)r + bb] = sum;
                }
            }
        }
    }
}

// Hands the R partial sums of every virtual column from the lane that walked its list in one
// chunk to the lane that walks it in the next (`from`, `to`: virtual columns of this thread; the
// plan deals the lists of each chunk to the waves by length).  They pass through the first 2 R KB
// of `area`, the LDS of the chunk consumed last: the first barrier makes sure nobody reads that
// chunk any more (and publishes whatever was written to other LDS before the call), the last one
// that the area may be staged into again.  Called by all threads.
template <int R>
__device__ __forceinline__ void swap_owner(uint8_t* area, float (&acc)[R], uint32_t from, uint32_t to) {
    f32x4* X = reinterpret_cast<f32x4*>(area);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R / 4; ++q)
        X[q * kThreadsGQ + from] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};   // lanes spread over all banks
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R / 4; ++q) {
        const f32x4 a = X[q * kThreadsGQ + to];
        acc[4 * q] = a[0]; acc[4 * q + 1] = a[1]; acc[4 * q + 2] = a[2]; acc[4 * q + 3] = a[3];
    }
    __syncthreads();
}

// Launchers of kernel A (they fill in first_gq, wgs_gq and blocks_gq; r and d are set): one workgroup = a block of rows of G at a time, 512 threads, one lane
// per (virtual) column of T.
hipError_t launch_gq_bf16(CompressGroup& g, const RawCall& raw, hipStream_t st);
hipError_t launch_gq_f16(CompressGroup& g, const RawCall& raw, hipStream_t st);
hipError_t launch_gq_f32(CompressGroup& g, const RawCall& raw, hipStream_t st);
hipError_t launch_mm_bf16(CompressGroup& g, hipStream_t st);   // kept plans (compress_mm.hip)

}  // namespace lsp
