// Optimiser-state re-projection (MaybeUpdate in Alg. 1, its last two assignments): when the
// projectors of a matrix are replaced, the subspace moments follow,
//     M <- (P^T P_prev) M (Q_prev^T Q),      V <- (P^T P_prev)^2 V (Q_prev^T Q)^2,
// the squares taken element by element.  Two steps:
//   1. A = P^T P_prev and B = Q_prev^T Q, r x r: products of two ELL matrices with the same rows;
//      row i adds its d x d products val * val' at (idx, idx'), with fp64 atomics in LDS on a block
//      of rows of the result that a workgroup owns.
//   2. four dense r x r products in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32): X = A M,
//      X2 = (A o A) V, then M = X B, V = X2 (B o B); the squares are taken while the tiles are staged,
//      and the two independent products of each stage share a launch.
// Runs once per change of projectors; nothing here is on the per-step path.
#include <algorithm>
#include <type_traits>

#include "products.h"

namespace lsp {


// C = L^T R for two ELL matrices with the same rows: C[L_idx[i][k]][R_idx[i][k']] += L_val[i][k] * R_val[i][k'].
// Global fp32 atomics are slow here (they go past the per-XCD L2), so a workgroup owns a block of rows of C
// in LDS.  It scans the column index of every entry (i, k) of L; a wave queues those that fall in its
// block, in LDS; then a lane per (queued entry, k') adds the product with an LDS atomic; then the block is
// written (C needs no clearing).  Scanning and adding are separate so that neither is a chain of dependent
// loads.  An entry that finds the wave's queue full is added by the lane that found it (correct, slow: only
// heavily skewed projectors get there).  Two independent pairs may share a launch; each has about one workgroup in 256 for its share of all entries.
// Entries with an index outside [0, r) are skipped.  The order of the LDS additions varies: results can differ in the last
// bits from run to run.
// What bounds it: the scan, which every workgroup makes of all entries (issue, and 64 bytes a cycle from L2), and trips to memory.  The next 32 entries a thread are on their way while
// 32 are looked at, no load has a condition (the compiler waits for one that has), and nothing is divided by d.
// The sums are taken in 64 bits, because ds_add_f32 serves one lane in 3 cycles, wherever the lanes' addresses lie (192 cycles a wave), and ds_add_f64 a wave in 20: 4096 and 11008 rows,
// r = 512, d = 8 18.9 -> 16.5 us, 4096 and 4096 11.4 -> 10.1; with the loads as they are now 18.2 -> 13.8 and 10.2 -> 9.7.
constexpr int kGramThreads = 1024, kGramSums = 12288, kGramQueue = 256, kGramInFlight = 8;   // (a wave's queue)
constexpr size_t kGramLds = (size_t)kGramThreads / kWave * kGramQueue * sizeof(int);               // ... and the sums
struct GramArgs {
    int32_t r, d;
    uint32_t d_inverse;                                             // ceil(2^32 / d); 0: d = 1
    int32_t block_rows[2], first[2];                                // rows of C a workgroup has of each pair; the pair's first workgroup
    int32_t pad[9];
    GramPair p[2];
    GramClear clear;
};
static_assert(sizeof(GramPair) == 64 && offsetof(GramArgs, p) == 64, "records of 64 bytes, loaded whole");
__device__ __forceinline__ uint32_t divided(uint32_t x, uint32_t d, uint32_t d_inverse) {
    if (d_inverse == 0) return x;
    const uint32_t q = __umulhi(x, d_inverse);                      // or one more
    return q * d > x ? q - 1 : q;
}
__global__ __launch_bounds__(kGramThreads) void k_gram(const GramArgs) {
    extern __shared__ __align__(16) uint8_t smem[];
    double* const acc = reinterpret_cast<double*>(smem + kGramLds);
    const auto* args = group_args<GramArgs>();
    words8 head = scalar_load<words8>(args);
    words16 pair0 = scalar_load<words16>(&args->p[0]), pair1 = scalar_load<words16>(&args->p[1]);
    arrived(head, pair0, pair1);
    const int r = (int)head[0], d = (int)head[1];
    const uint32_t d_inverse = head[2];
    const bool second = (int)blockIdx.x >= (int)head[6];
    const int block_rows = (int)(second ? head[4] : head[3]), block = (int)blockIdx.x - (second ? (int)head[6] : 0);
    GramPair P;
    const words16 pair = second ? pair1 : pair0;
    __builtin_memcpy(&P, &pair, 64);
    P.L_idx = global_pointer(P.L_idx); P.L_val = global_pointer(P.L_val); P.R_idx = global_pointer(P.R_idx); P.R_val = global_pointer(P.R_val); P.C = global_pointer(P.C);
    const int a0 = block * block_rows, a1 = min(r, a0 + block_rows);
    const int mine = (a1 - a0) * r;
    const int lane = threadIdx.x & 63;
    const int total = (int)(P.rows * d);                            // < 2^31, checked by the host
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    typedef i32x4 loose __attribute__((aligned(4)));
    static_assert(4 * kGramInFlight == 32, "one bit for every entry of a batch");
    // Entries 4 q .. 4 q + 3; the last ones begin at total - 4 at the latest, what they have twice counts once (fewer than 4 entries: one by one).
    const int quads = (int)(((int64_t)total + 3) / 4);
    auto fetch = [&](i32x4 (&a)[kGramInFlight], int t0) {
        if (total < 4) {
#pragma unroll
            for (int u = 0; u < kGramInFlight; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) a[u][q] = P.L_idx[q < total ? q : 0];
            return;
        }
#pragma unroll
        for (int u = 0; u < kGramInFlight; ++u) {
            const int t = t0 + u * kGramThreads + (int)threadIdx.x, at = t < quads ? 4 * t : 0;
            a[u] = *reinterpret_cast<const loose*>(P.L_idx + (at < total - 4 ? at : total - 4));
        }
    };
    auto entry_of = [&](int quad, int q) { return (total >= 4 && 4 * quad > total - 4 ? total - 4 : 4 * quad) + q; };
    i32x4 now[kGramInFlight], next[kGramInFlight];
    fetch(now, 0);
    for (int q = threadIdx.x; q < mine; q += kGramThreads) acc[q] = 0.0;
    __syncthreads();
    int* const queue = reinterpret_cast<int*>(smem) + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave) * kGramQueue;
    int queued = 0;                                                 // (uniform over the wave)
    auto add_entry = [&](int t, int a, int k2) {
        const float v = P.L_val[t];
        const int row = (int)divided((uint32_t)t, (uint32_t)d, d_inverse) * d;
        const int b = P.R_idx[row + k2];
        const float x = P.R_val[row + k2];
        if (v != 0.0f && (unsigned)b < (unsigned)r) unsafeAtomicAdd(&acc[(a - a0) * r + b], (double)v * (double)x);
    };
    for (int t0 = 0; t0 < quads; t0 += kGramThreads * kGramInFlight) {       // uniform trip count: the exchanges need whole waves
        const bool more = t0 + kGramThreads * kGramInFlight < quads;
        if (more) fetch(next, t0 + kGramThreads * kGramInFlight);
        if (t0 + kGramThreads * kGramInFlight >= quads) {           // the last entries are among these: none of the block's rows for what is not one, or was the quad's before
            const int extra = 4 * quads - total;
#pragma unroll
            for (int u = 0; u < kGramInFlight; ++u) {
                const int t = t0 + u * kGramThreads + (int)threadIdx.x;
                const int from = t >= quads ? 4 : t == quads - 1 && total >= 4 ? extra : 0, to = t == quads - 1 && total < 4 ? total : 4;
#pragma unroll
                for (int q = 0; q < 4; ++q) now[u][q] = q >= from && q < to ? now[u][q] : -1;
            }
        }
        uint32_t late = 0;                                          // entries that found the queue full
#pragma unroll
        for (int u = 0; u < kGramInFlight; ++u) {
            const int quad = t0 + u * kGramThreads + (int)threadIdx.x;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool hit = (unsigned)(now[u][q] - a0) < (unsigned)(a1 - a0);
                const uint64_t hits = __ballot(hit);
                if (hits == 0) continue;
                const int place = queued + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
                if (hit) {
                    if (place < kGramQueue) queue[place] = entry_of(quad, q);
                    else late |= 1u << (4 * u + q);
                }
                queued += __builtin_popcountll(hits);
            }
        }
        while (late) {
            const int k = __ffs((int)late) - 1;
            late &= late - 1;
            const int t = entry_of(t0 + (k >> 2) * kGramThreads + (int)threadIdx.x, k & 3), row = P.L_idx[t];
            for (int k2 = 0; k2 < d; ++k2) add_entry(t, row, k2);
        }
        queued = min(queued, kGramQueue);
        if (queued > kGramQueue / 2 || !more) {                     // what is queued joins the sums
            __builtin_amdgcn_wave_barrier();
            const int work = queued * d;
            for (int w0 = lane; w0 < work; w0 += kWave * kGramInFlight) {
                // every load of a batch is issued before the first addition: otherwise each item waits for its own
                int a[kGramInFlight], b[kGramInFlight];
                float v[kGramInFlight], x[kGramInFlight];
#pragma unroll
                for (int u = 0; u < kGramInFlight; ++u) {
                    const uint32_t w = (uint32_t)min(w0 + u * kWave, work - 1), e = divided(w, (uint32_t)d, d_inverse);
                    const int t = queue[e];
                    const int other = (int)(divided((uint32_t)t, (uint32_t)d, d_inverse) * (uint32_t)d + w - e * (uint32_t)d);
                    a[u] = P.L_idx[t];
                    v[u] = P.L_val[t];
                    b[u] = P.R_idx[other];
                    x[u] = P.R_val[other];
                }
#pragma unroll
                for (int u = 0; u < kGramInFlight; ++u)
                    if (w0 + u * kWave < work && v[u] != 0.0f && (unsigned)b[u] < (unsigned)r) unsafeAtomicAdd(&acc[(a[u] - a0) * r + b[u]], (double)v[u] * (double)x[u]);
            }
            queued = 0;
            __builtin_amdgcn_wave_barrier();
        }
        if (more)
#pragma unroll
            for (int u = 0; u < kGramInFlight; ++u) now[u] = next[u];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < mine; q += kGramThreads) P.C[(int64_t)a0 * r + q] = (float)acc[q];
    if (args->clear.p) {
        const auto* H = as_const<PlanHeader>(args->clear.plan);
        if (H->magic == kPlanMagic && H->p_any_split) {
            float* const p = global_pointer(args->clear.p);
            const int64_t count = args->clear.count;
            for (int64_t k = (int64_t)blockIdx.x * kGramThreads + threadIdx.x; k < count; k += (int64_t)gridDim.x * kGramThreads) p[k] = 0.0f;
        }
    }
}

// C = op(A) op(B) + beta E, all r x r row-major fp32; op squares every element (sqa, sqb) or transposes the
// operand (ta, tb) while its tiles are staged.  A launch takes up to kMaxGemmBatch independent products of
// one size (blockIdx.z picks one): a product alone is 256 small workgroups at r = 512, one per CU and each a
// chain of load latencies, so independent products share the chip.
template <int MN, int VEC>
__global__ __launch_bounds__(256) void k_gemm_rr(const GemmBatch) {
    __shared__ __align__(16) float lds[kTileFloats<MN, 32>];
    const auto* args = group_args<GemmBatch>();
    words2 head = scalar_load<words2>(args);
    words16 record = scalar_load<words16>(&args->p[blockIdx.z]);
    arrived(head, record);
    product_tile<MN, 32, VEC>(gemm_problem(record), (int)head[0], blockIdx.y * MN, blockIdx.x * MN, lds);
}

hipError_t launch_gram(const GramBatch& batch, int count, int32_t d, int32_t r, const GramClear* clear, hipStream_t st) {
    if (count < 1 || count > 2 || r > kGramSums) return hipErrorInvalidValue;
    int64_t entries = 0;
    for (int z = 0; z < count; ++z) {
        if (batch.p[z].rows * d > INT32_MAX) return hipErrorInvalidValue;
        entries += batch.p[z].rows * d;
    }
    // The rows of C are spread over about one workgroup
    // per CU rather than packed into as few as LDS allows (each workgroup scans all of L_idx either way); the pair with more entries has more of the workgroups.
    GramArgs args{};
    args.r = r; args.d = d;
    args.d_inverse = d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d);
    args.first[1] = INT32_MAX;
    int grid = 0;
    for (int z = 0; z < count; ++z) {
        const int share = (int)std::max<int64_t>(1, std::min<int64_t>(224, 256 * batch.p[z].rows * d / entries));
        args.p[z] = batch.p[z];
        args.block_rows[z] = std::max(1, std::min(kGramSums / (int)r, ((int)r + share - 1) / share));
        args.first[z] = grid;
        grid += ((int)r + args.block_rows[z] - 1) / args.block_rows[z];
    }
    if (clear) args.clear = *clear;
    hipError_t e;
    if ((e = allow_dynamic_lds<k_gram, kGramLds + kGramSums * sizeof(double)>()) != hipSuccess) return e;
    const size_t lds = kGramLds + (size_t)std::max(args.block_rows[0], args.block_rows[1]) * r * sizeof(double);
    hipLaunchKernelGGL(k_gram, dim3((unsigned)grid), dim3(kGramThreads), lds, st, args);
    return hipGetLastError();
}

hipError_t launch_gemm_rr_batch(const GemmBatch& batch, int count, int32_t r, hipStream_t st) {
    if (count < 1 || count > kMaxGemmBatch) return hipErrorInvalidValue;
    for (int z = 0; z < count; ++z)
        if ((batch.p[z].flags & kGemmTA) && (batch.p[z].flags & kGemmTB)) return hipErrorInvalidValue;   // not needed anywhere
    bool by16 = r % 4 == 0;                                          // groups of 16 bytes: whole ones, aligned operands
    for (int z = 0; z < count; ++z)
        by16 = by16 && reinterpret_cast<uintptr_t>(batch.p[z].A) % 16 == 0 && reinterpret_cast<uintptr_t>(batch.p[z].B) % 16 == 0;
    GemmBatch args = batch;
    args.r = r;
    auto go = [&](auto kernel, int tile) {
        const unsigned side = (unsigned)((r + tile - 1) / tile);
        hipLaunchKernelGGL(kernel, dim3(side, side, (unsigned)count), dim3(256), 0, st, args);
    };
    if (!by16)                 go(k_gemm_rr<32, 1>, 32);
    else if (wide_products(r)) go(k_gemm_rr<64, 4>, 64);
    else                       go(k_gemm_rr<32, 4>, 32);
    return hipGetLastError();
}

hipError_t launch_reproject(const int32_t* P_idx, const float* P_val, const int32_t* Pp_idx, const float* Pp_val,
                            const int32_t* Q_idx, const float* Q_val, const int32_t* Qp_idx, const float* Qp_val,
                            int64_t m, int64_t n, int32_t r, int32_t d, float* M, float* V, float* workspace,
                            hipStream_t st) {
    const int64_t rr = (int64_t)r * r;
    float* A = workspace;
    float* B = workspace + rr;
    float* X = workspace + 2 * rr;
    GramBatch grams{};
    grams.p[0] = GramPair{P_idx, P_val, Pp_idx, Pp_val, m, A, {}};
    grams.p[1] = GramPair{Qp_idx, Qp_val, Q_idx, Q_val, n, B, {}};
    hipError_t e = launch_gram(grams, 2, d, r, nullptr, st);
    if (e != hipSuccess) return e;
    // X = A M and X2 = (A o A) V in one launch, then M = X B and V = X2 (B o B) in another
    float* X2 = workspace + 3 * rr;
    GemmBatch left{}, right{};
    left.p[0] = GemmProblem{A, M, X, nullptr, 0.0f, 0, nullptr, {}};
    left.p[1] = GemmProblem{A, V, X2, nullptr, 0.0f, kGemmSqA, nullptr, {}};
    right.p[0] = GemmProblem{X, B, M, nullptr, 0.0f, 0, nullptr, {}};
    right.p[1] = GemmProblem{X2, B, V, nullptr, 0.0f, kGemmSqB, nullptr, {}};
    if ((e = launch_gemm_rr_batch(left, V ? 2 : 1, r, st)) != hipSuccess) return e;
    return launch_gemm_rr_batch(right, V ? 2 : 1, r, st);
}

}  // namespace lsp
