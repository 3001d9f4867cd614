// What the launches of r x r products share: a tile of a product, in a kernel of its own (reproject.hip) and beside the gather of the fitting gradient (fitgrad.hip).
#pragma once
#include <algorithm>
#include <type_traits>

#include "compress_common.h"

namespace lsp {

__device__ __forceinline__ GemmProblem gemm_problem(const words16& record) {
    GemmProblem P;
    __builtin_memcpy(&P, &record, 64);
    P.A = global_pointer(P.A); P.B = global_pointer(P.B); P.C = global_pointer(P.C); P.E = global_pointer(P.E); P.Ct = global_pointer(P.Ct);
    return P;
}
typedef float f32x16 __attribute__((ext_vector_type(16)));

// An MN x MN tile of a product by 256 threads.  K goes by in tiles of K.  Everything moves in groups of VEC floats: four where r is a multiple of 4 and the operands are aligned, as in the
// training configurations, otherwise one.  Both tiles lie in LDS with k running along the rows (As[i][k], Bs[j][k], rows padded by 16
// bytes); a group is four consecutive k of one row where the operand
// has k contiguous in memory (A as it is, B transposed: one 16-byte LDS store), else four consecutive rows of
// one k (four 4-byte LDS stores).  The matrix instruction is v_mfma_f32_32x32x2_f32: lane l supplies A[i = l % 32][k = l / 32] and B[k = l / 32][j = l % 32] and holds
// C[8 (v / 4) + 4 (l / 32) + v % 4][l % 32] in register v.  Within 8 consecutive k the lanes of half h = l / 32 take k = 4 h .. 4 h + 3
// with one 16-byte LDS load per operand, and the instruction number s of the group multiplies element s of
// both: it sums over k = s and k = 4 + s, and the four of them over all eight.
// MN = 32: the four waves share each tile's k, and their four sums meet in LDS.  MN = 64: a wave has a quadrant, all k of it in four sums one after the other (the rounding of four short
// sums and not of one long), which takes half as much from L2 for a result and a chain of latencies four times as long.
// Short tiles are faster, as more of them are in flight on a CU: 512 x 512, d = 8, two launches of two products each, the whole re-projection of a 4096 x 11008 matrix 109.0 us with K = 128 and 108.2 with 32;
// r = 768 131.9 and 121.9, r = 1024 (MN = 32) 197 with K = 128, 187 with 64.  Two buffers in LDS, one barrier a tile: no better (r = 1024 193).
// (VEC = 1 had K = 128 and loads with conditions: fitting 3001 x 2999, r = 250, d = 5 80.2 us, now 61.0; 1262 x 2000, r = 527, d = 3 108.4 and 76.2.)
template <int K> constexpr int kTileRow = K + 4;                     // floats per LDS row
template <int MN, int K> constexpr int kTileFloats = std::max(2 * MN * kTileRow<K>, MN == 32 ? 4 * 16 * 64 : 0);   // of LDS: both tiles, afterwards the waves' sums
// 64 x 64 tiles where 256 CUs have one each of a product, and less from L2 is worth more than many short chains (us, 4096 x 4096, d = 8, 32 and 64: r = 512 fitting 93 and 101, r = 768 refresh 132 and 150,
// fitting 183 and 182, r = 1024 refresh 197 and 184, fitting 213 and 200; all with K = 64 for 32 x 32).
inline bool wide_products(int r) { return r >= 1024; }
template <int MN, int K, int VEC>
__device__ __forceinline__ void product_tile(const GemmProblem& P, int r, int row0, int col0, float* lds) {
    constexpr int kTileRow = lsp::kTileRow<K>, kTileGroups = MN * K / VEC / 256;   // groups of VEC floats of each tile a thread stages
    constexpr int kAlong = K / VEC, kDown = 256 / kAlong;             // where k is contiguous: groups of a row, rows of 256 groups
    constexpr int kStepK = VEC == 1 ? 256 / MN : MN == 32 ? 32 : 16; // where rows are: k of 256 groups
    static_assert((MN == 32 || MN == 64) && (VEC == 1 || VEC == 4) && kTileGroups * 256 * VEC == MN * K, "whole groups for every thread");
    typedef float group __attribute__((ext_vector_type(VEC)));
    float* const As = lds;
    float* const Bs = lds + MN * kTileRow;
    const float* __restrict__ A = P.A;
    const float* __restrict__ B = P.B;
    const bool ta = P.flags & kGemmTA, tb = P.flags & kGemmTB, sqa = P.flags & kGemmSqA, sqb = P.flags & kGemmSqB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    // Group q = tid + 256 e of a tile.  k contiguous in memory: row q / (K / 4), k = 4 (q % (K / 4)) .. + 3 (rows step
    // with e).  Rows contiguous in memory: a wave takes 16 rows (four groups) of 16 k, so that it reads 64-byte pieces and
    // its 4-byte stores meet no bank twice (with 32 rows of 8 k: four lanes to a bank); k steps by 32 with e.
    const bool a_kc = !ta, b_kc = tb;
    const int t_mn = VEC == 1 ? tid % MN : 4 * ((lane & 3) + 4 * (MN == 32 ? wave & 1 : wave)), t_k = VEC == 1 ? tid / MN : (lane >> 2) + (MN == 32 ? 16 * (wave >> 1) : 0);
    const int a_mn = a_kc ? tid / kAlong : t_mn, a_k = a_kc ? VEC * (tid % kAlong) : t_k;
    const int b_mn = b_kc ? tid / kAlong : t_mn, b_k = b_kc ? VEC * (tid % kAlong) : t_k;
    float* const as0 = As + a_mn * kTileRow + a_k;
    float* const bs0 = Bs + b_mn * kTileRow + b_k;
    const int as_step = a_kc ? kDown * kTileRow : kStepK, bs_step = b_kc ? kDown * kTileRow : kStepK;
    group an[2][kTileGroups], bn[2][kTileGroups];                   // the next two tiles
    // Every lane loads, past the last row and k the last ones once more: loads that some lanes leave out would be waited for one by one.  (r * r < 2^31)
    int a_row[kTileGroups], b_row[kTileGroups];
#pragma unroll
    for (int e = 0; e < kTileGroups; ++e) {
        a_row[e] = a_kc ? min(row0 + a_mn + kDown * e, r - 1) * r : min(row0 + a_mn, r - VEC);
        b_row[e] = b_kc ? min(col0 + b_mn + kDown * e, r - 1) * r : min(col0 + b_mn, r - VEC);
    }
    const int a_last = r - (a_kc ? VEC : 1), b_last = r - (b_kc ? VEC : 1), a_kstep = a_kc ? 1 : r, b_kstep = b_kc ? 1 : r;
    auto fetch = [&](auto set, int k0) {
        constexpr int Z = decltype(set)::value;
#pragma unroll
        for (int e = 0; e < kTileGroups; ++e) {
            an[Z][e] = *reinterpret_cast<const group*>(A + a_row[e] + min(k0 + a_k + (a_kc ? 0 : kStepK * e), a_last) * a_kstep);
            bn[Z][e] = *reinterpret_cast<const group*>(B + b_row[e] + min(k0 + b_k + (b_kc ? 0 : kStepK * e), b_last) * b_kstep);
        }
    };
    const int wave_row = MN == 32 ? 0 : 32 * (wave >> 1), wave_col = MN == 32 ? 0 : 32 * (wave & 1), wave_k = MN == 32 ? wave * (K / 4) : 0;
    constexpr int kWaveK = MN == 32 ? K / 4 : K;
    const float* ap = As + (wave_row + (lane & 31)) * kTileRow + wave_k + 4 * (lane >> 5);
    const float* bp = Bs + (wave_col + (lane & 31)) * kTileRow + wave_k + 4 * (lane >> 5);
    f32x16 total;                                                   // MN = 64: the quarters of K that are done
#pragma unroll
    for (int v = 0; v < 16; ++v) total[v] = 0.0f;
    const int quarter = ((r + K - 1) / K + 3) / 4;
    int left = quarter;
    auto tile = [&](auto set, auto ahead, int k0) {
        constexpr int Z = decltype(set)::value;
#pragma unroll
        for (int e = 0; e < kTileGroups; ++e) {
            group a = an[Z][e], b = bn[Z][e];
            if (k0 + a_k + (a_kc ? 0 : kStepK * e) >= r) a = 0.0f;
            if (k0 + b_k + (b_kc ? 0 : kStepK * e) >= r) b = 0.0f;
            if (sqa) a *= a;
            if (sqb) b *= b;
            if (a_kc) *reinterpret_cast<group*>(as0 + e * as_step) = a;
            else {
#pragma unroll
                for (int s = 0; s < VEC; ++s) as0[e * as_step + s * kTileRow] = a[s];
            }
            if (b_kc) *reinterpret_cast<group*>(bs0 + e * bs_step) = b;
            else {
#pragma unroll
                for (int s = 0; s < VEC; ++s) bs0[e * bs_step + s * kTileRow] = b[s];
            }
        }
        __syncthreads();
        if constexpr (decltype(ahead)::value) fetch(set, k0 + 2 * K);
#pragma unroll
        for (int g = 0; g < kWaveK / 8; ++g) {                      // a wave's part of the tile, 8 k at a time
            const f32x4 a = *reinterpret_cast<const f32x4*>(ap + 8 * g);
            const f32x4 b = *reinterpret_cast<const f32x4*>(bp + 8 * g);
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], b[s], acc, 0, 0, 0);
        }
        if (MN == 64 && --left == 0) {
            left = quarter;
#pragma unroll
            for (int v = 0; v < 16; ++v) { total[v] += acc[v]; acc[v] = 0.0f; }
        }
        __syncthreads();
    };
    constexpr std::integral_constant<int, 0> kEven{};
    constexpr std::integral_constant<int, 1> kOdd{};
    constexpr std::true_type kAhead{};
    constexpr std::false_type kLast{};
    fetch(kEven, 0);
    fetch(kOdd, K);
    int k0 = 0;
    for (; k0 + 3 * K < r; k0 += 2 * K) {
        tile(kEven, kAhead, k0);
        tile(kOdd, kAhead, k0 + K);
    }
    if (k0 + 2 * K < r) {                                           // three tiles are left, two, or one
        tile(kEven, kAhead, k0);
        tile(kOdd, kLast, k0 + K);
        tile(kEven, kLast, k0 + 2 * K);
    } else {
        tile(kEven, kLast, k0);
        if (k0 + K < r) tile(kOdd, kLast, k0 + K);
    }
    if constexpr (MN == 64) {
        typedef f32x4 loose __attribute__((aligned(4)));
        const int j = col0 + wave_col + (lane & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = row0 + wave_row + 8 * q + 4 * (lane >> 5);
            if (i >= r || j >= r) continue;                         // (four rows or none: r % 4 == 0)
            f32x4 sum;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                sum[s] = total[4 * q + s] + acc[4 * q + s];
                if (P.E) sum[s] = fmaf(P.beta, P.E[(int64_t)(i + s) * r + j], sum[s]);
                P.C[(int64_t)(i + s) * r + j] = sum[s];
            }
            if (P.Ct) *reinterpret_cast<loose*>(P.Ct + (int64_t)j * r + i) = sum;
        }
        return;
    }
    float* const Cs = lds;                                          // (every wave is done with the tiles)
#pragma unroll
    for (int v = 0; v < 16; ++v) Cs[(wave * 16 + v) * 64 + lane] = acc[v];
    __syncthreads();
    const int j = col0 + (lane & 31);
#pragma unroll
    for (int q = 0; q < 4; ++q) {                                   // a wave adds up a quarter of the tile
        const int v = 4 * wave + q, i = row0 + 8 * wave + 4 * (lane >> 5) + q;
        float sum = ((Cs[v * 64 + lane] + Cs[(16 + v) * 64 + lane]) + Cs[(32 + v) * 64 + lane]) + Cs[(48 + v) * 64 + lane];
        if (i < r && j < r) {
            if (P.E) sum = fmaf(P.beta, P.E[(int64_t)i * r + j], sum);
            P.C[(int64_t)i * r + j] = sum;
            if (P.Ct) P.Ct[(int64_t)j * r + i] = sum;
        }
    }
}

}  // namespace lsp
