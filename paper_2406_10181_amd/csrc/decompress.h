// Decompress and apply:  W <- rn(W - P S Q^T)  (Alg. 1, apply step; Alg. 3, last step of the
// layer loop).  One launch, one fused read-modify-write pass over W:
//   phase 1  U = P S for the workgroup's R rows of W (gathers d rows of S per row, S stays in
//            L2), stored in LDS in fp32, the rows of a column in units of 4 rows (k_decompress and k_decompress_any), 8 or 16 (k_decompress_wide);
//   phase 2  every thread has the d (column, value) pairs of its columns' rows of Q in registers
//            and gathers U with one 128-bit LDS read per pair and 4 rows; W is read, updated in fp32 and rounded once.
// The bytes that have to move are the read and the write of W; no matrix cores (sparse gather + fp32 FMA).
// What bounds it: no single thing.  In the launch of the seven matrices of a 6.7B-style layer (bf16, r = 512, d = 8, k_decompress_wide in blocks of 32 rows;
// 199 us, 207 with k_decompress) HBM moves 921 MB (4.6 TB/s, 70 % of a plain read-modify-write pass), the LDS works 48 % of the cycles
// (half of that for bank conflicts), the vector ALUs 47 %, L2 hands out 1.41 GB (rows of W, Q and S); 2.9 waves a
// SIMD are resident on average (4 fit), and they wait for data 29 % of their time and for their turn to issue 50 %.
//
// The same kernels, built with NORMS, serve the estimation bias of Def. 2 (the test MaybeUpdate
// makes in Alg. 1): with S = P^T G Q they rebuild P S Q^T tile by tile in registers, read G where
// the apply step reads W, and instead of storing anything add up (P S Q^T - G)^2 and G^2; every
// workgroup leaves its two sums in a list that k_bias_finish adds in a fixed order.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "lsp_internal.h"

namespace lsp {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename D> struct Pair { uint32_t x; };                 // two neighbouring elements of W
template <> struct Pair<F32> { float x, y; };

template <typename D> __device__ __forceinline__ void pair_widen(uint32_t p, float& lo, float& hi);
template <> __device__ __forceinline__ void pair_widen<F16>(uint32_t p, float& lo, float& hi) {
    lo = widen<F16>((uint16_t)(p & 0xFFFFu)); hi = widen<F16>((uint16_t)(p >> 16));
}
template <> __device__ __forceinline__ void pair_widen<BF16>(uint32_t p, float& lo, float& hi) {
    lo = __uint_as_float(p << 16); hi = __uint_as_float(p & 0xFFFF0000u);
}
template <typename D> __device__ __forceinline__ uint32_t pair_narrow(float lo, float hi) {
    return (uint32_t)narrow<D>(lo) | ((uint32_t)narrow<D>(hi) << 16);
}

template <typename D> __device__ __forceinline__ void widen_pair(const Pair<D>& p, float* out) {
    if constexpr (D::size == 4) { out[0] = p.x; out[1] = p.y; }
    else pair_widen<D>(p.x, out[0], out[1]);
}
template <typename D> __device__ __forceinline__ Pair<D> narrow_pair(const float* in) {
    if constexpr (D::size == 4) return Pair<D>{in[0], in[1]};
    else return Pair<D>{pair_narrow<D>(in[0], in[1])};
}

// Sums x and y over the workgroup (NT threads) and lets thread 0 store them; `red` is LDS nobody
// else uses any more.  Fixed order: the result does not depend on timing.
template <int NT>
__device__ __forceinline__ void block_sum2(float x, float y, float2* red, float2* dst) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        x += __shfl_down(x, off);
        y += __shfl_down(y, off);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_float2(x, y);
    __syncthreads();
    if (threadIdx.x == 0) {
        float2 t = red[0];
        for (int w = 1; w < NT / 64; ++w) { t.x += red[w].x; t.y += red[w].y; }
        *dst = t;
    }
}

// Phase 1, for d = DD (or, with DD = 0, any d), AHEAD loads in flight: the R * d (row of S, value) pairs of the tile go to LDS first, then every
// work item (row of the tile, 4 consecutive columns b) issues its 128-bit loads of S back to back, so the whole gather
// costs few memory round trips.  A row's last quad is read from r - 4 on when r is no multiple of 4: some columns are then
// made twice, with the same result; or, where the tile's columns lie in whole quads (Place::kQuads), it is turned into its place, with
// whatever behind the last column.  place(row, b, c): where element (row, b + c) of the tile lives (c < 4).
// The pairs are asked for first of all (tile_entry: a thread's first one; nearly always it has no other): loads return in order, and behind those of W the build would wait for HBM
// once more.  At d = 16 the rows of Q before them are as much as W, and they wait for their turn (2048 x 2048, r = 256, d = 16 12.0 us first of all, 11.7 in turn; 4096 x 16384, r = 1024 103.1 and 102.5).
// Rows past m: value 0, row 0 of S.
__device__ __forceinline__ int2 tile_entry(const int32_t* __restrict__ P_idx, const float* __restrict__ P_val, int64_t i0, int m, int d, int q) {
    const int64_t at = i0 * d + q, count = (int64_t)m * d, there = at < count ? at : count - 1;
    const int idx = P_idx[there];
    const float val = P_val[there];
    return at < count ? make_int2(idx, __float_as_int(val)) : make_int2(0, 0);
}
template <int R, int DD, int AHEAD, bool STRIPES, int NT, typename Place>
__device__ __forceinline__ void build_u_tile(const Place& place, int2* pent, const int2 first_entry, const float* __restrict__ S,
                                             const int32_t* __restrict__ P_idx, const float* __restrict__ P_val,
                                             int64_t i0, int m, int r, int dim) {
    typedef f32x4 loose __attribute__((aligned(4)));
    const int d = DD > 0 ? DD : dim;
    constexpr bool kAsked = DD != 16;
    if (kAsked && (int)threadIdx.x < R * d) pent[threadIdx.x] = first_entry;
    for (int q = threadIdx.x + (kAsked ? NT : 0); q < R * d; q += NT) pent[q] = tile_entry(P_idx, P_val, i0, m, d, q);
    __syncthreads();
    if (r < 4) {
        for (int q = threadIdx.x; q < R * r; q += NT) {
            const int row = q / r, b = q - row * r;
            float u = 0.0f;
            for (int k = 0; k < d; ++k) u = fmaf(__int_as_float(pent[row * d + k].y), S[pent[row * d + k].x * r + b], u);
            *place(row, 0, b) = u;
        }
        return;
    }
    const int quads = (r + 3) >> 2;
    // Row of the tile and column quad of this thread's next item (a division for each item would take as long as its sums).
    // Beyond r = 1024 S does not fit the L2 of an XCD (4 MB), and row by row most of its rows come from further away each time: then the waves
    // take one stripe of 64 quads of all rows after the other, as all workgroups do at about the same time, so that a stripe (2 MB at r = 2048) is
    // shared in L2 (4096 x 4096, r = 2048, d = 8, bf16: 47.7 -> 44.9 us; r = 1536, d = 16, fp16, 1000 x 2048: 24.5 -> 24.0).  Not where the
    // last stripe would leave more than an eighth of the lanes idle (r = 1100: 32.4, with stripes 32.7); at r = 1024 and below it is even.
    constexpr int WAVES = NT / kWave;
    static_assert(!STRIPES || R % WAVES == 0, "every wave has the same number of rows of a stripe");
    // (STRIPES: so the rest has no code for it)
    const bool stripes = STRIPES && r > 1024 && (quads + kWave - 1) / kWave * kWave * 8 <= quads * 9;
    const int row0 = stripes ? (int)threadIdx.x / kWave : (int)threadIdx.x / quads;
    int row = row0, b4 = stripes ? (int)threadIdx.x % kWave : (int)threadIdx.x - row0 * quads;
    int row_step = stripes ? WAVES : R, b4_step = 0;                 // (one item a thread: no second division)
    if (!stripes && quads * R > NT) { row_step = NT / quads; b4_step = NT - row_step * quads; }
    auto advance = [&]() {
        row += row_step; b4 += b4_step;
        if (stripes) {
            if (row >= R) {
                row = row0; b4 += kWave;
                if (b4 >= quads) { row = R; b4 = quads; }
            }
        } else if (b4 >= quads) { b4 -= quads; ++row; }
    };
    auto store = [&](int at_row, int b, f32x4 u) {
        if constexpr (Place::kQuads) {
            if ((r & 3) != 0) {                                     // b = r - 4 instead of the quad's own column
                const int turn = -b & 3;
                u = turn == 0 ? u : turn == 1 ? f32x4{u.y, u.z, u.w, u.w} : turn == 2 ? f32x4{u.z, u.w, u.w, u.w} : f32x4{u.w, u.w, u.w, u.w};
                b += turn;
            }
        }
        *place(at_row, b, 0) = u.x; *place(at_row, b, 1) = u.y; *place(at_row, b, 2) = u.z; *place(at_row, b, 3) = u.w;
    };
    // d < AHEAD: several items at a time, while there are more than one for every thread (the step of the MLP pair, fp16, d = 4: 75.7 us one by
    // one, now 75.0; where a thread has one item only it would be work for nothing: the attention matrices 22.1, with two items 22.6)
    if constexpr (DD > 0 && AHEAD / (DD > 0 ? DD : 1) >= 2) {
        constexpr int ITEMS = AHEAD / DD;
        for (int left = quads * R; left > NT; left -= ITEMS * NT) {
            f32x4 x[ITEMS][DD];
            float v[ITEMS][DD];
            int at[ITEMS], b[ITEMS];
#pragma unroll
            for (int u = 0; u < ITEMS; ++u) {
                at[u] = min(row, R - 1);                             // past the last item: some of the last row once more
                b[u] = min(b4 * 4, r - 4);
                advance();
#pragma unroll
                for (int k = 0; k < DD; ++k) {
                    const int2 e = pent[at[u] * DD + k];
                    v[u][k] = __int_as_float(e.y);
                    x[u][k] = *reinterpret_cast<const loose*>(S + (int64_t)e.x * r + b[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < ITEMS; ++u) {
                f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < DD; ++k) {
                    sum.x = fmaf(v[u][k], x[u][k].x, sum.x); sum.y = fmaf(v[u][k], x[u][k].y, sum.y);
                    sum.z = fmaf(v[u][k], x[u][k].z, sum.z); sum.w = fmaf(v[u][k], x[u][k].w, sum.w);
                }
                store(at[u], b[u], sum);
            }
        }
    }
    for (; row < R; advance()) {
        const int b = min(b4 * 4, r - 4);
        f32x4 u = {0.0f, 0.0f, 0.0f, 0.0f};
        auto add = [&](int k0, auto count) {
            constexpr int N = decltype(count)::value;
            f32x4 x[N];
#pragma unroll
            for (int k = 0; k < N; ++k) x[k] = *reinterpret_cast<const loose*>(S + (int64_t)pent[row * d + k0 + k].x * r + b);
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const float v = __int_as_float(pent[row * d + k0 + k].y);
                u.x = fmaf(v, x[k].x, u.x); u.y = fmaf(v, x[k].y, u.y);
                u.z = fmaf(v, x[k].z, u.z); u.w = fmaf(v, x[k].w, u.w);
            }
        };
        if constexpr (DD > 0) {
            constexpr int A = DD < AHEAD ? DD : AHEAD, WHOLE = DD / A * A;
#pragma unroll
            for (int k = 0; k < WHOLE; k += A) add(k, std::integral_constant<int, A>{});
            if constexpr (WHOLE < DD) add(WHOLE, std::integral_constant<int, DD - WHOLE>{});
        } else {
            int k = 0;
            for (; k + 8 <= d; k += 8) add(k, std::integral_constant<int, 8>{});
            for (; k + 4 <= d; k += 4) add(k, std::integral_constant<int, 4>{});
            for (; k < d; ++k) add(k, std::integral_constant<int, 1>{});
        }
        store(row, b, u);
    }
}

// Planes of 4 rows, PS bytes apart: element (row, b) is number row % 4 of the b-th float4 of its plane.
template <int PS> struct PlanePlace {
    static constexpr bool kQuads = false;
    uint8_t* smem;
    __device__ __forceinline__ float* operator()(int row, int b, int c) const { return reinterpret_cast<float*>(smem + (row >> 2) * PS) + (b + c) * 4 + (row & 3); }
};

// The rows of a block of W (or G) as buffers of their own: lanes past a row's end load zero and store nothing, and so does
// a whole row past the matrix, without a branch.  Branches around loads and stores are what the kernel below must not have: the
// compiler counts the memory operations in flight over every path to a use, and an operation that one path skips makes
// the use wait for younger ones as well.
typedef __amdgpu_buffer_rsrc_t RowBuffer;
template <typename D> struct RowBlock {
    char* base;                                                     // first row of the block
    int64_t stride;                                                 // bytes from row to row
    int rows;                                                       // rows of the block inside the matrix
    int n;
    // row t from column col on (a pass: at most a few thousand columns)
    __device__ __forceinline__ RowBuffer from(int t, int col) const {
        const int left = n - col < 65536 ? n - col : 65536;
        return __builtin_amdgcn_make_buffer_rsrc(base + t * stride + (int64_t)col * D::size, 0, t < rows ? left * D::size : 0, 0x00027000);
    }
};
constexpr int kNonTemporal = 2;                                     // cache policy of the streaming accesses
template <typename V> __device__ __forceinline__ V row_load(RowBuffer b, uint32_t offset) {
    V out;
    if constexpr (sizeof(V) == 2) { const uint16_t t = __builtin_amdgcn_raw_buffer_load_b16(b, (int)offset, 0, kNonTemporal); __builtin_memcpy(&out, &t, 2); }
    else if constexpr (sizeof(V) == 4) { const uint32_t t = __builtin_amdgcn_raw_buffer_load_b32(b, (int)offset, 0, kNonTemporal); __builtin_memcpy(&out, &t, 4); }
    else { const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(b, (int)offset, 0, kNonTemporal); __builtin_memcpy(&out, &t, 8); }
    return out;
}
template <typename V> __device__ __forceinline__ void row_store(RowBuffer b, uint32_t offset, const V& v) {
    if constexpr (sizeof(V) == 2) { uint16_t t; __builtin_memcpy(&t, &v, 2); __builtin_amdgcn_raw_buffer_store_b16(t, b, (int)offset, 0, kNonTemporal); }
    else if constexpr (sizeof(V) == 4) { uint32_t t; __builtin_memcpy(&t, &v, 4); __builtin_amdgcn_raw_buffer_store_b32(t, b, (int)offset, 0, kNonTemporal); }
    else { u32x2 t; __builtin_memcpy(&t, &v, 8); __builtin_amdgcn_raw_buffer_store_b64(t, b, (int)offset, 0, kNonTemporal); }
}

// The passes of a workgroup: `count` of the row block's, from `first` on, in an order rotated by the workgroup's position
// inside its XCD (workgroups are dealt to the 8 XCDs round-robin): all workgroups read the same Q arrays, and without
// the rotation they would all ask the same few L2 channels for the same lines at once.  (The divisions, which the first
// loads wait for, are left out where there is nothing to divide.)
struct Passes {
    int all, first, count, rot;
    __device__ __forceinline__ Passes(int n, int step, int block, int part, int parts) {
        all = n / step + (n % step != 0);                           // step is a power of two
        first = 0; count = all; rot = 0;
        if (parts > 1) {
            const int each = all / parts, more = all - each * parts;
            first = part * each + min(part, more);
            count = each + (part < more ? 1 : 0);
        }
        if (all > 1) rot = (int)((unsigned)(block / 8) % (unsigned)all);
    }
    __device__ __forceinline__ int at(int p) const {
        int q = first + p + rot;
        if (q >= all) q -= all;
        return q;
    }
};

// Fast kernel: DD = compile-time d, two columns per thread, n even.  PS = bytes between the 4-row planes of U in
// LDS, a compile-time constant >= 16 r so that the plane offset folds into the immediate offset of the LDS read and a
// gather costs no address arithmetic.
// A thread's patch of W (R rows x 2 columns) for the next pass is loaded plane by plane into the registers that the
// plane just finished has left, so a whole pass is in flight at any time at the cost of one patch; the rows of Q follow
// at the end of the pass.
template <typename D, int RG, int DD, int PS, int NT, bool NORMS>
__global__ __launch_bounds__(NT, (DD == 16 ? 2 : 4)) void k_decompress(const ApplyGroup) {
    extern __shared__ __align__(16) uint8_t smem[];
    constexpr int CPT = 2;
    constexpr int R = 4 * RG;
    constexpr int NE = CPT * DD;                                    // entries owned by a thread in one pass
    static_assert(NE % 4 == 0, "entries are loaded 4 at a time");
    typedef Pair<D> Patch;
    // a row block is shared by `parts` workgroups, each with its share of the passes (all build the tile of U)
    const auto* grp = group_args<ApplyGroup>();
    const auto pick = pick_problem(grp, grp->first, (int)blockIdx.x);
    const ApplyProblem& pr = pick.p;
    const int r = pick.r;
    const int unit = (int)blockIdx.x - pr.first, parts = pr.parts;
    const int block = parts > 1 ? unit / parts : unit, part = unit - block * parts;
    const float* __restrict__ S = pr.S;
    const int32_t* __restrict__ P_idx = pr.P_idx;
    const float* __restrict__ P_val = pr.P_val;
    const int32_t* __restrict__ Q_idx = pr.Q_idx;
    const float* __restrict__ Q_val = pr.Q_val;
    const int m = pr.m, n = pr.n;
    const int64_t i0 = (int64_t)block * R;
    int2* pent = reinterpret_cast<int2*>(smem + RG * PS);
    const f32x4* Us4 = reinterpret_cast<const f32x4*>(smem);

    constexpr int step = NT * CPT;
    const Passes passes(n, step, block, part, parts);
    const int npass = passes.count;
    auto pass_col = [&](int p) -> int { return passes.at(p) * step; };   // the pass's first column
    const int lane_col = (int)threadIdx.x * CPT;                    // of the pass; past n: nothing there for this thread
    const RowBlock<D> rows{static_cast<char*>(pr.W) + i0 * n * D::size, (int64_t)n * D::size, m - i0 < R ? (int)(m - i0) : R, n};

    Patch w[R];
    int4 qi[NE / 4];
    f32x4 qv[NE / 4];
    auto load_w = [&](int t, int col) { w[t] = row_load<Patch>(rows.from(t, col), (uint32_t)lane_col * D::size); };
    auto load_q = [&](int col) {
        const int jq = col < n - lane_col ? col + lane_col : n - CPT;
        const int4* qip = reinterpret_cast<const int4*>(Q_idx + (int64_t)jq * DD);
        const f32x4* qvp = reinterpret_cast<const f32x4*>(Q_val + (int64_t)jq * DD);
#pragma unroll
        for (int k = 0; k < NE / 4; ++k) { qi[k] = qip[k]; qv[k] = qvp[k]; }
    };
    auto idx_of = [&](int e) -> uint32_t {
        const int4 q = qi[e >> 2];
        return (uint32_t)((e & 3) == 0 ? q.x : (e & 3) == 1 ? q.y : (e & 3) == 2 ? q.z : q.w);
    };
    float num = 0.0f, den = 0.0f;                                   // NORMS: this thread's sums of squares
    // the pass at column col; more: the patch of the pass at column next is loaded behind it
    auto pass = [&](int col, int next, auto more) {
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            float acc[4][CPT];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int c = 0; c < CPT; ++c) acc[t][c] = 0.0f;
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
#pragma unroll
                for (int k = 0; k < DD; ++k) {
                    const f32x4 u = Us4[idx_of(c * DD + k) + g * (PS / 16)];
                    const float v = qv[(c * DD + k) >> 2][(c * DD + k) & 3];
                    acc[0][c] = fmaf(v, u.x, acc[0][c]);
                    acc[1][c] = fmaf(v, u.y, acc[1][c]);
                    acc[2][c] = fmaf(v, u.z, acc[2][c]);
                    acc[3][c] = fmaf(v, u.w, acc[3][c]);
                    if constexpr (DD >= 8) if (k % 8 == 7) __builtin_amdgcn_sched_barrier(0);   // eight gathers in flight: more would not fit the registers
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float x[CPT];
                widen_pair<D>(w[g * 4 + t], x);
                if constexpr (NORMS) {
                    const bool on = col < n - lane_col && g * 4 + t < rows.rows;
#pragma unroll
                    for (int c = 0; c < CPT; ++c) {
                        const float diff = acc[t][c] - x[c];
                        num = on ? fmaf(diff, diff, num) : num;
                        den = on ? fmaf(x[c], x[c], den) : den;
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < CPT; ++c) x[c] -= acc[t][c];
                    row_store(rows.from(g * 4 + t, col), (uint32_t)lane_col * D::size, narrow_pair<D>(x));
                }
                if constexpr (decltype(more)::value) load_w(g * 4 + t, next);
            }
        }
        if constexpr (decltype(more)::value) load_q(next);
    };

    int col = pass_col(0);
    int2 first_entry = make_int2(0, 0);
    if constexpr (DD != 16) {
        first_entry = tile_entry(P_idx, P_val, i0, m, DD, (int)threadIdx.x);
        asm volatile("" ::: "memory");                                // (in this order)
    }
#pragma unroll
    for (int t = 0; t < R; ++t) load_w(t, col);                     // in flight while the U tile is built
    load_q(col);
    build_u_tile<R, DD, (D::size == 4 && (RG > 2 || DD == 8) ? 4 : 8), (PS > 16384), NT>(PlanePlace<PS>{smem}, pent, first_entry, S, P_idx, P_val, i0, m, r, DD);
    __syncthreads();
    for (int p = 1; p < npass; ++p) {
        const int next = pass_col(p);
        pass(col, next, std::true_type{});
        col = next;
    }
    if (npass > 0) pass(col, col, std::false_type{});
    if constexpr (NORMS) block_sum2<NT>(num, den, reinterpret_cast<float2*>(smem), reinterpret_cast<float2*>(grp->partial) + blockIdx.x);
}

#define LSP_LDS_AS __attribute__((address_space(3)))
// Wide kernel: n % 8 == 0, r % 4 == 0.  LP neighbouring lanes (4; 2 in blocks of 8 rows) work on the same columns, each on four rows of a plane of 4 LP: a column of U
// is a unit of 16 LP bytes in LDS, and a gather of theirs reads one whole.  The 16 lanes that an LDS read serves at a time then ask for 4 units instead of 16, so fewer
// meet on a bank, whatever the order of Q's entries (k_decompress on columns in random order: 186 us for four matrices 4096 x 11008, r = 512, d = 8, bf16, 176 with Q
// reordered; here 167 and 166).  A thread holds the entries of 2 columns of Q (1 for d = 16 and in fp32) and gets those of the others from its neighbours by
// DPP moves; its patch of W is 4 rows x 8 (4) columns of each plane, moved in 16 bytes a row (pieces of 8 bytes, with the patch reloaded in halves: 202 us).  Each entry
// gives an address for all planes, and half or a quarter of the entries leave d = 16 at 128 registers, so that two workgroups share a CU.
// Three forms, by what is asked for ahead (loads return in order, so within a pass what is needed first goes first):
//   kDeep, on grids of one workgroup a CU, which may have 256 registers: the next pass's entries and patch when a pass begins (4096 x 16384, r = 512, d = 8 72.4 -> 64.2 us);
//   kTwo: the next patch when a pass begins, the entries with it if a thread has at most 8, at its end otherwise (bf16, beside kPlain: 8192 x 4096, r = 512, d = 4 32.7 -> 30.7 us,
//     d = 8 39.0 -> 38.7; 16384 x 2048, r = 256, d = 4 31.4 -> 30.2; bias pass 11008 x 4096, r = 512, d = 8 46.0 -> 44.4);
//   kPlain: both at the end of a pass; for 32 rows, whose second patch would not fit 128 registers, and where two passes or fewer on at most two workgroups a CU leave little to
//     fetch ahead for (5120 x 2048, r = 512, d = 8 21.7, kTwo 22.8; 5120 x 768, r = 256, d = 2 8.2 and 8.8).
// What bounds it, 4096 x 11008 four times (166 us): HBM at 4.3 TB/s of the 5.3 to 5.8 that its pattern allows; the LDS reads take some 85 us of it.

// Units of U in LDS: the 16-byte pieces of a unit and the units of a block of 256 bytes trade places by the block's number, so that the stores of the build, where a
// wave has one row of 256 neighbouring columns, fall on all banks.
template <int LP> __device__ __forceinline__ uint32_t unit_of(uint32_t b) {
    if constexpr (LP == 4) return (b << 6) ^ ((b << 2) & 0xF0u);
    else return (b << 5) ^ ((b << 1) & 0x70u);
}
template <int LP, int PLANE> struct UnitPlace {
    static constexpr bool kQuads = true;
    uint8_t* smem;
    // b a multiple of 4
    __device__ __forceinline__ float* operator()(int row, int b, int c) const {
        const uint32_t at = (unit_of<LP>((uint32_t)b) ^ (((uint32_t)row >> 2 & (LP - 1)) << 4)) + ((uint32_t)row & 3) * 4;
        return reinterpret_cast<float*>(smem + (row / (4 * LP)) * PLANE + (at ^ ((uint32_t)c * (16 * LP))));
    }
};
// x of lane S of the LP neighbouring lanes that share a unit
template <int LP, int S> __device__ __forceinline__ uint32_t of_lane(uint32_t x) {
    constexpr int ctrl = LP == 4 ? S * 0x55 : S == 0 ? 0xA0 : 0xF5;   // quad_perm
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, ctrl, 0xF, 0xF, true);
}

// f(0), f(1), ... of constants
template <typename F, int... k> __device__ __forceinline__ void every_of(F& f, std::integer_sequence<int, k...>) { (f(std::integral_constant<int, k>{}), ...); }
template <int N, typename F> __device__ __forceinline__ void every(F&& f) { every_of(f, std::make_integer_sequence<int, N>{}); }

enum WideForm { kPlain, kTwo, kDeep };
// LOOSE: any n, r and d.  What lies in whole patches of a row is done as above, from wherever the row begins in memory; the columns behind the last one (fewer than a patch is
// wide) are left to the last two waves, an element each: they have least to do in a row's last pass.
template <typename D, int G, int LP, int DD, bool BIG, int NT, bool NORMS, WideForm FORM, bool LOOSE>
__device__ __forceinline__ void decompress_wide() {
    extern __shared__ __align__(16) uint8_t smem[];
    static_assert(!LOOSE || G == 1, "one plane");
    constexpr int CPT = DD == 16 || D::size == 4 ? 1 : 2;                           // columns whose entries of Q a thread holds
    constexpr int PR = 4 * LP;                                      // rows of a plane of units
    constexpr int R = G * PR, PLANE = G > 1 ? 32768 : 0;
    constexpr int COLS = CPT * LP;                                  // columns of a thread's patch, LP threads have the same
    constexpr int NE = CPT * DD;
    constexpr int DW = COLS * D::size / 4;                          // dwords of a row of it
    constexpr int VW = DW < 4 ? DW : 4, NV = DW / VW;               // in loads of VW
    constexpr bool DEEP = FORM == kDeep, TWO = FORM != kPlain, TWO_Q = DEEP || (TWO && NE <= 8);   // two sets of registers, which passes take in turn, for the patch of W and the entries
    // Units of U are asked for 8 (4) ahead of the FMAs: with two waves a SIMD the compiler's own order, one or two ahead, left the reads' latency bare (us before and with it;
    // 4096 x 4096, r = 512, d = 8, bf16, Q reordered or not: 22.5 and 21.7, bias pass 22.0 and 21.1; 4096 x 11008 50.1 and 48.3, 40.9 and 39.1; 4096 x 4096, r = 1024, d = 16, fp32
    // 44.3 and 42.5; bias pass 4096 x 16384, r = 1024, d = 16, bf16 95 and 87).  16 bits at d = 16 are bound by the reads themselves: 4096 x 16384 103 and 104.5.
    constexpr bool AHEAD = TWO && !(LP == 4 && DD == 16 && D::size == 2 && !NORMS);
    typedef uint32_t Vec __attribute__((ext_vector_type(VW)));
    const auto* grp = group_args<ApplyGroup>();
    const auto pick = pick_problem(grp, grp->first, (int)blockIdx.x);
    const ApplyProblem& pr = pick.p;
    const int r = pick.r;
    const int unit = (int)blockIdx.x - pr.first, parts = pr.parts;
    const int block = parts > 1 ? unit / parts : unit, part = unit - block * parts;
    const float* __restrict__ S = pr.S;
    const int32_t* __restrict__ P_idx = pr.P_idx;
    const float* __restrict__ P_val = pr.P_val;
    const int32_t* __restrict__ Q_idx = pr.Q_idx;
    const float* __restrict__ Q_val = pr.Q_val;
    const int m = pr.m, n = pr.n;
    const int64_t i0 = (int64_t)block * R;
    int2* pent = reinterpret_cast<int2*>(smem + (G > 1 ? G * PLANE : (LOOSE ? (r + 3) / 4 * 4 : r) * (16 * LP)));

    constexpr int step = NT * CPT;
    const Passes passes(n, step, block, part, parts);
    const int npass = passes.count;
    auto pass_col = [&](int p) -> int { return passes.at(p) * step; };
    const int patched = LOOSE ? n / COLS * COLS : n;                // columns in whole patches
    const int own_col = (int)threadIdx.x * CPT;                     // of the pass: the first column whose entries this thread holds
    const int lane_col = (int)threadIdx.x / LP * COLS;              // and the first of its patch
    const uint32_t p4 = threadIdx.x & (LP - 1);                     // rows 4 p4 .. of a plane are this thread's
    const uint32_t piece = p4 << 4;
    const int rows = m - i0 < R ? (int)(m - i0) : R;
    char* const base = static_cast<char*>(pr.W) + i0 * n * D::size;
    const uint32_t stride = (uint32_t)n * D::size;                  // (host: 16 rows are less than 2^31 bytes)
    const uint32_t lane_off = p4 * 4 * stride + (uint32_t)lane_col * D::size;
    // row t of the thread's four in plane g: what lies behind the matrix's last row is past the buffer's end, and a thread past the last column goes there too
    auto buffer = [&](int g, int t, int col) {
        const int row = g * PR + t;
        const uint32_t left = rows > row ? (uint32_t)min(rows - row, PR) * stride - (uint32_t)col * D::size : 0u;
        return __builtin_amdgcn_make_buffer_rsrc(base + (int64_t)row * stride + (int64_t)col * D::size, 0, left, 0x00027000);
    };
    auto offset = [&](int col) { return lane_col < patched - col ? lane_off : 0x80000000u; };

    uint32_t w_[TWO ? 2 : 1][G][4][DW];
    uint32_t at_[TWO_Q ? 2 : 1][NE];                                // units of the entries
    float qv_[TWO_Q ? 2 : 1][NE];
    auto load_w = [&](int s, int g, int t, int col, uint32_t off) {
        auto& w = w_[s];
        const RowBuffer b = buffer(g, t, col);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            Vec x;
            if constexpr (VW == 4) x = __builtin_amdgcn_raw_buffer_load_b128(b, (int)off + v * 16, 0, kNonTemporal);
            else if constexpr (VW == 2) x = __builtin_amdgcn_raw_buffer_load_b64(b, (int)off + v * 8, 0, kNonTemporal);
            else x[0] = __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, kNonTemporal);
#pragma unroll
            for (int k = 0; k < VW; ++k) w[g][t][v * VW + k] = x[k];
        }
    };
    // Rows that begin anywhere leave lines of W half written, which are whole in L2 a pass or a neighbour later: temporal stores, but for the deep form in 16 bits (us, non-temporal and temporal: fp32 3001 x 2999 24.9
    // and 23.7, 4501 x 1601 25.0 and 23.7, 16001 x 2047 71.7 and 67.8, 9000 x 4100 97.4 and 100.1; 16 bits on more workgroups 8001 x 8190 75.2 and 73.8; the deep form 3001 x 2999, d = 5 17.6 and 19.1, 4096 x 4098
    // 25.2 and 26.4).  Rows of whole pieces: non-temporal.
    constexpr int kStorePolicy = LOOSE && !(DEEP && D::size == 2) ? 0 : kNonTemporal;
    auto store_w = [&](int s, int g, int t, int col, uint32_t off) {
        auto& w = w_[s];
        const RowBuffer b = buffer(g, t, col);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            Vec x;
#pragma unroll
            for (int k = 0; k < VW; ++k) x[k] = w[g][t][v * VW + k];
            if constexpr (VW == 4) __builtin_amdgcn_raw_buffer_store_b128(x, b, (int)off + v * 16, 0, kStorePolicy);
            else if constexpr (VW == 2) __builtin_amdgcn_raw_buffer_store_b64(x, b, (int)off + v * 8, 0, kStorePolicy);
            else __builtin_amdgcn_raw_buffer_store_b32(x[0], b, (int)off, 0, kStorePolicy);
        }
    };
    // Past the last column, and past the last pass, a buffer's end keeps entries from being read (4096 x 1536, r = 256, d = 2, bf16 9.65 -> 9.1 us; 11008 x 4096, r = 512, d = 8
    // 54.9 -> 53.6), but for long rows of few blocks at d = 8 in 16 bits addresses are the faster way (3000 x 11008, r = 256 45.8 and 45.1; 4096 x 4096, r = 512 even).
    auto load_q = [&](int s, int col, bool go_on) {
        auto &at = at_[s]; auto &qv = qv_[s];
        constexpr bool BOUNDED = LOOSE || !(DEEP && DD >= 8 && D::size == 2);
        constexpr int E = NE % 4 == 0 ? 4 : NE % 2 == 0 ? 2 : 1;
        typedef uint32_t Words __attribute__((ext_vector_type(E)));
        const int j = BOUNDED || col < n - own_col ? col + own_col : n - CPT;
        const int bytes = go_on ? n * (DD * 4) : 0;
        const RowBuffer ib = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(Q_idx), 0, bytes, 0x00027000);
        const RowBuffer vb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Q_val), 0, bytes, 0x00027000);
        auto load = [&](RowBuffer buf, const void* base, int k) {
            if constexpr (!BOUNDED) return reinterpret_cast<const Words*>(static_cast<const uint32_t*>(base) + (int64_t)j * DD)[k];
            else if constexpr (E == 4) return __builtin_amdgcn_raw_buffer_load_b128(buf, j * (DD * 4) + k * 16, 0, 0);
            else if constexpr (E == 2) return __builtin_amdgcn_raw_buffer_load_b64(buf, j * (DD * 4) + k * 8, 0, 0);
            else return Words{__builtin_amdgcn_raw_buffer_load_b32(buf, j * (DD * 4) + k * 4, 0, 0)};
        };
#pragma unroll
        for (int k = 0; k < NE / E; ++k) {
            const Words i = load(ib, Q_idx, k), v = load(vb, Q_val, k);
#pragma unroll
            for (int e = 0; e < E; ++e) { at[k * E + e] = i[e]; qv[k * E + e] = __uint_as_float(v[e]); }
        }
    };
    float num = 0.0f, den = 0.0f;
    auto pass = [&](auto set, int col, int next, bool go_on, auto more) {
        constexpr int s = decltype(set)::value;
        auto& w = w_[s];
        auto& at = at_[TWO_Q ? s : 0];
        auto& qv = qv_[TWO_Q ? s : 0];
        const uint32_t off = offset(col), next_off = go_on ? offset(next) : 0x80000000u;
        if constexpr (TWO_Q) load_q(1 - s, next, go_on);
        if constexpr (TWO) {
#pragma unroll
            for (int t = 0; t < 4; ++t) load_w(1 - s, 0, t, next, next_off);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) at[e] = unit_of<LP>(at[e]);
        // (deep: sums of a pass and row, so that what lies outside the matrix is left out once a pass and not element by element)
        float pass_num[4] = {0.0f, 0.0f, 0.0f, 0.0f}, pass_den[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        // columns 2 C and 2 C + 1 of the patch take their sums
        auto combine = [&](auto which, const float (&acc)[G][4][2]) {
            constexpr int C = decltype(which)::value;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    float x[2];
                    if constexpr (D::size == 4) { x[0] = __uint_as_float(w[g][t][2 * C]); x[1] = __uint_as_float(w[g][t][2 * C + 1]); }
                    else {
                        uint32_t both = w[g][t][C];
                        asm volatile("" : "+v"(both));                // (or it is widened long before, fp16)
                        pair_widen<D>(both, x[0], x[1]);
                    }
                    if constexpr (NORMS && AHEAD) {
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const float diff = acc[g][t][c] - x[c];
                            pass_num[t] = fmaf(diff, diff, pass_num[t]);
                            pass_den[t] = fmaf(x[c], x[c], pass_den[t]);
                        }
                    } else if constexpr (NORMS) {
                        const bool on = lane_col < patched - col && g * PR + (int)p4 * 4 + t < rows;
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const float diff = acc[g][t][c] - x[c];
                            num = on ? fmaf(diff, diff, num) : num;
                            den = on ? fmaf(x[c], x[c], den) : den;
                        }
                    } else {
                        x[0] -= acc[g][t][0]; x[1] -= acc[g][t][1];
                        if constexpr (D::size == 4) { w[g][t][2 * C] = __float_as_uint(x[0]); w[g][t][2 * C + 1] = __float_as_uint(x[1]); }
                        else w[g][t][C] = pair_narrow<D>(x[0], x[1]);
                    }
                }
        };
        auto zero = [](float (&acc)[G][4][2]) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[g][t][0] = acc[g][t][1] = 0.0f;
        };
        // entry k of column c of pair C, of the lane that holds it
        auto unit = [&](auto C, auto c, int k) { return of_lane<LP, (CPT == 2 ? C() : 2 * C() + c())>(at[(CPT == 2 ? c() * DD : 0) + k]) ^ piece; };
        auto value = [&](auto C, auto c, int k) { return __uint_as_float(of_lane<LP, (CPT == 2 ? C() : 2 * C() + c())>(__float_as_uint(qv[(CPT == 2 ? c() * DD : 0) + k]))); };
        auto add = [](float (&acc)[G][4][2], int g, int c, float v, f32x4 u) {
            acc[g][0][c] = fmaf(v, u.x, acc[g][0][c]);
            acc[g][1][c] = fmaf(v, u.y, acc[g][1][c]);
            acc[g][2][c] = fmaf(v, u.z, acc[g][2][c]);
            acc[g][3][c] = fmaf(v, u.w, acc[g][3][c]);
        };
        if constexpr (AHEAD) {
            // A units ahead: one is asked for when one has been used.
            constexpr int N = COLS * DD, MOST = !DEEP || (DD == 16 && D::size == 2) ? 4 : 8, A = MOST < N ? MOST : N;
            f32x4 u[A];
            float acc[G][4][2];
            auto ask = [&](auto entry) {
                constexpr int e = decltype(entry)::value, column = e / DD;
                u[e % A] = *(const f32x4 LSP_LDS_AS*)(uintptr_t)unit(std::integral_constant<int, column / 2>{}, std::integral_constant<int, column & 1>{}, e % DD);
            };
            every<A>(ask);
            every<N>([&](auto entry) {
                constexpr int e = decltype(entry)::value, column = e / DD, k = e % DD;
                constexpr std::integral_constant<int, column / 2> C{};
                constexpr std::integral_constant<int, column & 1> c{};
                if constexpr (c() == 0 && k == 0) zero(acc);
                add(acc, 0, c(), value(C, c, k), u[e % A]);
                if constexpr (e + A < N) ask(std::integral_constant<int, e + A>{});
                if constexpr (c() == 1 && k == DD - 1) combine(C, acc);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (NORMS)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const bool on = lane_col < patched - col && (int)p4 * 4 + t < rows;
                    num += on ? pass_num[t] : 0.0f;
                    den += on ? pass_den[t] : 0.0f;
                }
        } else {
            every<COLS / 2>([&](auto C) {
                float acc[G][4][2];
                zero(acc);
                every<2>([&](auto c) {
#pragma unroll
                    for (int k = 0; k < DD; ++k) {
                        const uint32_t here = unit(C, c, k);
                        const float v = value(C, c, k);
#pragma unroll
                        for (int g = 0; g < G; ++g) add(acc, g, c(), v, *(const f32x4 LSP_LDS_AS*)(uintptr_t)(here + g * PLANE));
                        if constexpr (DD * G >= 8) if (k % (8 / G) == 8 / G - 1) __builtin_amdgcn_sched_barrier(0);
                    }
                });
                combine(C, acc);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
        if constexpr (!NORMS) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t) store_w(s, g, t, col, off);
        }
        if constexpr (!TWO_Q && decltype(more)::value) load_q(0, next, go_on);   // (loads return in order: what is needed first)
        if constexpr (!TWO && decltype(more)::value) {
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int t = 0; t < 4; ++t) load_w(s, g, t, next, next_off);
        }
    };

    int col = pass_col(0);
    int2 first_entry = make_int2(0, 0);
    if constexpr (DD != 16) {
        first_entry = tile_entry(P_idx, P_val, i0, m, DD, (int)threadIdx.x);
        asm volatile("" ::: "memory");                                // (in this order)
    }
    load_q(0, col, true);
    if constexpr (DD != 16) __builtin_amdgcn_sched_barrier(0);        // (the same order as at the end of a pass, or every pass would wait for W where it wants the last entries)
    {
        const uint32_t off = offset(col);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int t = 0; t < 4; ++t) load_w(0, g, t, col, off);     // in flight while the U tile is built
    }
    // Plain form, where one or two passes are all there is: with more of S than of the patch to come, its rows would stand in line behind all of W, so W arrives first.
    // (us without and with the wait, bf16, from HBM; 16 rows a block: 5120 x 1024, r = 512, d = 2 10.0 and 8.8, d = 4 11.5 and 10.4, d = 8 16.3 and 14.5; 5120 x 2048, d = 4 17.3 and 16.6; but r = 128, d = 8
    // 11.0 and 11.6.  32 rows, one pass: 28160 x 1024, r = 352, d = 4 35.2 and 31.9, d = 8 45.5 and 43.5; 16384 x 640, r = 352, d = 4 16.0 and 14.9; d = 2 is even, 20000 x 640, r = 288 16.6 and 17.6.)
    if constexpr (FORM == kPlain && (G == 1 || DD != 2)) {
        if (G == 1 ? r >= 256 : npass <= 1) {
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0x0F70);                       // vmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    build_u_tile<R, DD, (D::size == 4 && (R > 8 || DD == 8) ? 4 : 8), BIG, NT>(UnitPlace<LP, PLANE>{smem}, pent, first_entry, S, P_idx, P_val, i0, m, r, DD);
    __syncthreads();
    if constexpr (LOOSE) {                                          // the columns behind the last whole patch
        constexpr int kRest = COLS - 1;
        static_assert(kRest * R <= 2 * kWave, "two waves");
        const int e = (int)threadIdx.x - (NT - 2 * kWave), at_row = e / COLS, c = e % COLS;
        if (part == 0 && e >= 0 && at_row < rows && patched + c < n) {
            const int64_t j = patched + c;
            typename D::elem* const w = reinterpret_cast<typename D::elem*>(base + at_row * (int64_t)stride) + j;
            uint32_t b[DD];
            float v[DD];
            const typename D::elem stored = *w;
#pragma unroll
            for (int k = 0; k < DD; ++k) { b[k] = (uint32_t)Q_idx[j * DD + k]; v[k] = Q_val[j * DD + k]; }
            float sum = 0.0f;
#pragma unroll
            for (int k = 0; k < DD; ++k) {
                const uint32_t at = (unit_of<LP>(b[k]) ^ ((uint32_t)at_row >> 2 << 4)) + ((uint32_t)at_row & 3) * 4;
                sum = fmaf(v[k], *reinterpret_cast<const float*>(smem + at), sum);
            }
            const float x = widen<D>(stored);
            if constexpr (NORMS) {
                const float diff = sum - x;
                num = fmaf(diff, diff, num);
                den = fmaf(x, x, den);
            } else *w = narrow<D>(x - sum);
        }
    }
    constexpr std::integral_constant<int, 0> even{};
    if constexpr (TWO) {
        constexpr std::integral_constant<int, 1> odd{};
        for (int p = 0; p < npass;) {
            int next = pass_col(min(p + 1, npass - 1));
            pass(even, col, next, p + 1 < npass, std::true_type{});
            if (++p >= npass) break;
            col = next; next = pass_col(min(p + 1, npass - 1));
            pass(odd, col, next, p + 1 < npass, std::true_type{});
            ++p; col = next;
        }
    } else {
        for (int p = 1; p < npass; ++p) {
            const int next = pass_col(p);
            pass(even, col, next, true, std::true_type{});
            col = next;
        }
        if (npass > 0) pass(even, col, col, true, std::false_type{});
    }
    if constexpr (NORMS) block_sum2<NT>(num, den, reinterpret_cast<float2*>(smem), reinterpret_cast<float2*>(grp->partial) + blockIdx.x);
}

template <typename D, int G, int LP, int DD, bool BIG, int NT, bool NORMS, WideForm FORM>
__global__ __launch_bounds__(NT, FORM == kDeep ? 2 : 4) void k_decompress_wide(const ApplyGroup) { decompress_wide<D, G, LP, DD, BIG, NT, NORMS, FORM, false>(); }
template <typename D, int LP, int DD, bool NORMS, WideForm FORM>
__global__ __launch_bounds__(512, FORM == kDeep ? 2 : 4) void k_expand_loose(const ApplyGroup) { decompress_wide<D, 1, LP, DD, false, 512, NORMS, FORM, true>(); }

// General kernel: any n and d.  A thread has two columns of a pass: neighbours (PAIR, n even), or columns 64 apart, each
// loaded and stored by itself.  The entries of Q are taken four at a time for the whole patch (R x 2 sums in registers),
// the next four in flight; the next pass's first four are asked for before its patch of W, because loads return in order.
template <typename D, int RG, int PS, int NT, bool PAIR, bool NORMS>
__global__ __launch_bounds__(NT, (NORMS ? 3 : 4)) void k_decompress_any(const ApplyGroup) {
    extern __shared__ __align__(16) uint8_t smem[];
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    typedef i32x4 loose_i __attribute__((aligned(4)));
    typedef f32x4 loose_f __attribute__((aligned(4)));
    constexpr int R = 4 * RG;
    const auto* grp = group_args<ApplyGroup>();
    const auto pick = pick_problem(grp, grp->first, (int)blockIdx.x);
    const ApplyProblem& pr = pick.p;
    const int r = pick.r, d = pick.d;
    const int unit = (int)blockIdx.x - pr.first, parts = pr.parts;
    const int block = parts > 1 ? unit / parts : unit, part = unit - block * parts;
    const int32_t* __restrict__ Q_idx = pr.Q_idx;
    const float* __restrict__ Q_val = pr.Q_val;
    const int m = pr.m, n = pr.n;
    const int64_t i0 = (int64_t)block * R;
    const f32x4* Us4 = reinterpret_cast<const f32x4*>(smem);
    constexpr int step = NT * 2;
    const Passes passes(n, step, block, part, parts);
    const int npass = passes.count;
    auto pass_col = [&](int p) -> int { return passes.at(p) * step; };   // the pass's first column
    const int lane_col = PAIR ? (int)threadIdx.x * 2 : ((int)threadIdx.x >> 6) * 128 + ((int)threadIdx.x & 63);
    constexpr int kApart = PAIR ? 1 : kWave;                        // from the first column to the second
    const RowBlock<D> rows{static_cast<char*>(pr.W) + i0 * n * D::size, (int64_t)n * D::size, m - i0 < R ? (int)(m - i0) : R, n};

    typedef typename std::conditional<PAIR, Pair<D>, typename D::elem>::type Piece;
    constexpr int NP = PAIR ? 1 : 2;
    Piece w[R][NP];
    i32x4 qi[2][2];                                                 // [buffer][column]
    f32x4 qv[2][2];
    auto load_w = [&](int col) {
#pragma unroll
        for (int t = 0; t < R; ++t)
#pragma unroll
            for (int c = 0; c < NP; ++c) w[t][c] = row_load<Piece>(rows.from(t, col), (uint32_t)(lane_col + c * kApart) * D::size);
    };
    auto load_q = [&](int buf, int col, int k0) {                     // entries k0 .. of both columns; past d: not touched
        const int count = d - k0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int jc = col < n - lane_col - c * kApart ? col + lane_col + c * kApart : n - 1;
            const int64_t at = (int64_t)jc * d + k0;
            if (count >= 4) {
                qi[buf][c] = *reinterpret_cast<const loose_i*>(Q_idx + at);
                qv[buf][c] = *reinterpret_cast<const loose_f*>(Q_val + at);
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (k < count) { qi[buf][c][k] = Q_idx[at + k]; qv[buf][c][k] = Q_val[at + k]; }
            }
        }
    };
    float num = 0.0f, den = 0.0f;                                   // NORMS: this thread's sums of squares
    float acc[R][2];
    auto take = [&](int buf, int count) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (k > 0 && k >= count) break;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int g = 0; g < RG; ++g) {
                    const f32x4 u = Us4[(uint32_t)qi[buf][c][k] + g * (PS / 16)];
                    const float v = qv[buf][c][k];
                    acc[g * 4 + 0][c] = fmaf(v, u.x, acc[g * 4 + 0][c]);
                    acc[g * 4 + 1][c] = fmaf(v, u.y, acc[g * 4 + 1][c]);
                    acc[g * 4 + 2][c] = fmaf(v, u.z, acc[g * 4 + 2][c]);
                    acc[g * 4 + 3][c] = fmaf(v, u.w, acc[g * 4 + 3][c]);
                }
        }
    };
    int col = pass_col(0);
    const int2 first_entry = tile_entry(pr.P_idx, pr.P_val, i0, m, d, (int)threadIdx.x);
    asm volatile("" ::: "memory");                                    // (in this order)
    load_q(0, col, 0);
    load_w(col);
    build_u_tile<R, 0, 0, (PS > 16384), NT>(PlanePlace<PS>{smem}, reinterpret_cast<int2*>(smem + RG * PS), first_entry, pr.S, pr.P_idx, pr.P_val, i0, m, r, d);
    __syncthreads();
    for (int p = 0; p < npass; ++p) {
#pragma unroll
        for (int t = 0; t < R; ++t) acc[t][0] = acc[t][1] = 0.0f;
        for (int k0 = 0;; k0 += 8) {                                // buffers 0 and 1 in turn
            if (k0 + 4 < d) load_q(1, col, k0 + 4);
            take(0, d - k0);
            if (k0 + 4 >= d) break;
            if (k0 + 8 < d) load_q(0, col, k0 + 8);
            take(1, d - k0 - 4);
            if (k0 + 8 >= d) break;
        }
        const int next = p + 1 < npass ? pass_col(p + 1) : col;
        if (p + 1 < npass) load_q(0, next, 0);
#pragma unroll
        for (int t = 0; t < R; ++t) {
            float x[2];
            if constexpr (PAIR) widen_pair<D>(w[t][0], x);
            else { x[0] = widen<D>(w[t][0]); x[1] = widen<D>(w[t][1]); }
            if constexpr (NORMS) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const bool on = col < n - lane_col - c * kApart && t < rows.rows;
                    const float diff = acc[t][c] - x[c];
                    num = on ? fmaf(diff, diff, num) : num;
                    den = on ? fmaf(x[c], x[c], den) : den;
                }
            } else {
                x[0] -= acc[t][0]; x[1] -= acc[t][1];
                if constexpr (PAIR) {
                    row_store(rows.from(t, col), (uint32_t)lane_col * D::size, narrow_pair<D>(x));
                } else {
                    row_store(rows.from(t, col), (uint32_t)lane_col * D::size, narrow<D>(x[0]));
                    row_store(rows.from(t, col), (uint32_t)(lane_col + kApart) * D::size, narrow<D>(x[1]));
                }
            }
        }
        if (p + 1 < npass) load_w(next);
        col = next;
    }
    if constexpr (NORMS) block_sum2<NT>(num, den, reinterpret_cast<float2*>(smem), reinterpret_cast<float2*>(grp->partial) + blockIdx.x);
}

// k_expand_loose, one instantiation file a storage type (decompress_loose.h): d from 2 to kLooseEntries, rows of up to 2^24 columns; grid: workgroups of 8 rows (eight) or 16.
// (On more than one workgroup a CU d = 11 and 12 spill 12 to 52 bytes a lane in 16 bits, and beside k_decompress_any they are 1.13 to 1.54 times as fast, in fp32 1.08 to 1.8.)
constexpr int kLooseEntries = 12;
template <typename D> hipError_t launch_loose(const ApplyGroup& g, unsigned grid, bool eight, bool norms, hipStream_t st);

// The fast kernel needs an even n and d in {2, 4, 8, 16}; a group takes it only if all of its problems qualify.
inline bool fast_shape(int32_t n, int32_t d) { return (n % 2) == 0 && (d == 2 || d == 4 || d == 8 || d == 16); }

// k_decompress_wide (us; k_decompress and it; apply of one matrix unless said otherwise; uniform columns, Q not reordered).  It takes whole pieces of 8 columns and
// whole units of 4, every matrix of the group, or the group goes to k_expand_loose or k_decompress (loose_call), with the same result.  Where it and k_decompress can, it is used
//   for d = 16, where two columns' entries of Q in a thread leave k_decompress 192 registers: 4096 x 16384, r = 1024, bf16, zipf 129 and 101; 4096 x 4096, r = 1024, fp32 53.0 and
//     43.6; 2048 x 2048, r = 256, bf16 (8 rows) 15.3 and 12.4; bias pass 4096 x 4096, r = 512, bf16 77 and 67, with the compress call before it;
//   for 16 bits in blocks of 16 and 32 rows: four matrices 4096 x 11008, r = 512, d = 8 187 and 167 (176 and 166 with Q reordered); 4096 x 16384, r = 512, d = 8 75.7 and 66.8;
//     4096 x 8192, r = 256, d = 2 31.6 and 28.9; 16384 x 4096, d = 4 57.8 and 56.2; 4096 x 4096, r = 512, d = 8 22.2 and 21.6 (21.7 and 21.6 reordered); bias pass, r = 512, d = 8, 4096
//     x 4096 22.2 and 21.3 (20.6 and 21.0 reordered), 4096 x 11008 44.5 and 39.6 (40.4 and 38.9), 11008 x 4096 51.7 and 44.3 (46.1 and 43.8);
//   for fp32 where the grid fits the chip at once (deep) and in the bias pass: 4096 x 4096, r = 512, d = 8 32.9 and 30.6; 4096 x 2048, r = 256, d = 4 25.1 and 16.7; bias pass
//     8192 x 2048, r = 256, d = 4 27.6 and 18.4, 8192 x 4096, r = 512, d = 8 43.0 and 38.2.
// Elsewhere k_decompress is ahead: fp32 on larger grids (8192 x 4096, r = 512, d = 8 58.4 and 66.5; with 16 rows a thread has half as many registers in flight), and d <= 8 in
// blocks of 8 rows, whose pieces are 8 bytes (2048 x 2048, r = 512, d = 8, bf16 8.8 and 9.5; 4096 x 4096, r = 2048, d = 8 44.5 and 46.8).
constexpr unsigned kResidentDeep = 256;                              // workgroups of the deep form, one a CU
inline bool wide_shape(int64_t n, int32_t r) { return r >= 4 && r % 4 == 0 && n % 8 == 0 && n <= 1 << 24; }   // (32-bit offsets inside a plane of rows)
inline bool loose_group(const ApplyGroup& g, int32_t d) {
    bool loose = d >= 2 && d <= kLooseEntries;
    for (int p = 0; p < g.count; ++p) loose = loose && g.p[p].n <= 1 << 24;
    return loose;
}
// Where k_decompress_wide cannot be used, k_expand_loose or the two kernels with units of 4 rows (k_decompress for n even and d = 2, 4, 8, 16: fast; else k_decompress_any, which has two
// neighbouring columns a thread where n is even: pair).  lines: every row of W is whole lines of 128 bytes (fp32: n % 32 == 0).  grid: workgroups of 512 threads, n: the widest matrix, eight: 8 rows a workgroup.  (us, k_decompress(_any) and k_expand_loose; one matrix after
// another, W and G from HBM.  "1.05 times": k_expand_loose is so many times as fast.)
//   16 bits, fast: 4002 x 4098, r = 500, d = 8 26.3 and 24.9, 9000 x 4098, r = 600 69.2 and 61.0, 6002 x 2502, r = 333, d = 2 21.2 and 20.5; not in 8 rows (1500 x 2302, d = 8 0.95 times), nor where rows
//     are one pass, or one and a bit in more workgroups than the chip holds.
//   16 bits, not fast: even rows 5002 x 1602 and longer 1.07 to 2 times; odd ones, one workgroup a CU, 3001 x 2999, r = 250, d = 5 18.2 and 17.4, 4001 x 4095, r = 500, d = 12 38.3 and 30.8, in 8 rows
//     2001 x 4095, r = 300, d = 9 21.7 and 16.9.  With 257 to 447 workgroups some CUs have two and others one, which short lists do not cover: 5000 x 1601, r = 300, d = 2 15.8 and 19.0, d = 8 21.8 and
//     24.4, d = 10 27.2 and 25.5; 6001 x 2501, r = 333, d = 4 25.5 and 28.1, d = 7 33.8 and 31.0; 4500 to 6001 x 3071 0.81 to 1.02 times with d <= 5 and 8, x 3501 0.92 to 1.06 but for d = 4, where the
//     entries of k_decompress_any come in one piece (4500 x 4099, r = 1000 40.2 and 42.4).  On more workgroups the line is a second pass that is mostly empty: 16001 x 1535, d = 5 0.95 times, x 1801 1.03.
//   fp32, where k_decompress(_any) reaches 4.2 TB/s of HBM and k_expand_loose 3.3: there the shorter the lists, and the more there is to move, the worse it does (4001 x 8191, r = 500, d = 4 62.1 and
//     79.9, d = 8 67.4 and 81.4).  An odd d costs k_decompress_any more than d + 1, and so do even rows: list_weight; the longest rows for each weight, at about 0.95 times: in 8 rows 2040 x 5001 0.94 to
//     1.10 times, x 8191 0.84 to 1.02; one workgroup a CU, d <= 4 4001 x 2301 0.98 to 1.03, x 3071 0.90 to 0.96, d = 5 to 8 3001 x 6001 0.98 to 1.09, 4001 x 8191 0.82 to 0.89; more of them, d <= 4 16001 x
//     1535 0.95 to 0.97, x 2047 0.91 to 0.95, d = 5 7500 x 2301 1.03, x 3071 0.98, d = 6 and 8 x 3501 1.03, x 6001 0.95, d = 7 x 6001 0.99, x 8191 0.93; 9000 x 4099, r = 600, d = 12 123 and 113.
//     Rows of whole lines cost k_expand_loose no line twice, and it is ahead at any length: 2048 x 16384, r = 224, d = 5 71.0 and 61.4, 5120 x 4096, r = 1024, d = 5 54.9 and 50.8, 6464 x 14400, r = 976, d = 6
//     217 and 178; 2040 to 16001 rows of 8192 and 8224, d = 3 0.93 to 1.02 times, of 16384 1.22.  (Whole halves of a line are not enough: x 4104 and x 12004 0.78 to 1.05 times.)
//     (W in the cache behind L2: 3001 x 2999, r = 250, d = 6 24.9 and 22.0, 4001 x 8191, r = 500, d = 4 1.07 times.)  Fast, only in 8 rows just beyond 4096 columns, a stride that 8 rows of k_decompress
//     fare badly with (1500 x 4098 1.07 to 1.11 times; x 6002 0.95; 4002 x 8194, r = 500, d = 2 61 and 79).
//     Up to 512 columns half of the threads of the others have none: one workgroup a CU (3001 x 401 1.01 to 1.16 times), and elsewhere where the tile is large as well (9000 x 301, r = 1024, d = 4 23.7
//     and 18.5; 16001 x 301, r = 16 0.86 to 0.96 times).
//   Bias pass, where nothing is written: 9000 x 4099, r = 600, d = 5, bf16 65.1 and 43.3, fp32 69.5 and 47.6; 5000 x 1601, r = 300, d = 2, bf16 19.8 and 14.6; fast fp32 from 4096 columns on (4002 x 8194,
//     d = 8 39.5 and 36.3, d = 2 28.0 and 28.9; 3002 x 2998, d = 2 13.3 and 15.0).
//   d = 1, 4501 x 1101 10.6 and 12.5, so there is no kernel for it.
inline int list_weight(int32_t d, bool pair) {
    const int weight = d <= 4 ? 0 : d == 5 ? 1 : d == 7 ? 3 : d <= 8 ? 2 : 4;
    return pair && weight > 0 && weight < 4 ? weight + 1 : weight;
}
inline bool loose_call(unsigned grid, int32_t n, int32_t r, int32_t d, int elem_size, bool fast, bool pair, bool lines, bool eight, bool norms) {
    const bool deep = grid <= kResidentDeep;
    if (elem_size == 2) {
        if (fast) return !eight && n > (deep ? 1024 : 1536);
        if (norms || deep || pair || d >= 9) return n > (deep ? 1024 : 1536);
        if (grid >= 448) return n > 1664;
        return d != 4 && n > (d == 6 || d == 7 ? 2176 : 3328);
    }
    if (fast) return norms ? n >= 4096 : eight && n >= 4096 && n < 5120;
    if (n <= 1024) return n <= 512 && (deep || (r > 512 && !norms));
    constexpr int kAny = 1 << 30;
    constexpr int kLongest[3][5] = {{7168, 7168, 7168, kAny, kAny}, {2560, 7168, 7168, kAny, kAny}, {1536, 2560, 3840, 7168, kAny}};
    return norms || lines || n <= kLongest[!deep ? 2 : eight ? 0 : 1][list_weight(d, pair)];
}
inline bool wide_group(const ApplyGroup& g, int32_t r) {
    bool wide = true;
    for (int p = 0; p < g.count; ++p) wide = wide && wide_shape(g.p[p].n, r);
    return wide;
}
// Small work where k_decompress is ahead all the same (blocks of 16 rows of 512 threads, d <= 8; grid: workgroups, n: the widest matrix).  In a call of one pass nothing covers
// the lane moves, two of the six VALU instructions of an entry, and k_decompress makes the tile faster where a thread has one item of it (r <= 128).  (us, k_decompress and k_decompress_wide.)
//   One workgroup a CU, n <= 1024, bf16: 4096 x 768, r = 128, d = 2 5.8 and 6.5; r = 256 7.2 and 7.0; d = 4 7.0 and 7.3; 4096 x 512, r = 256, d = 8 7.7 and 8.3; 4096 x 1024, r = 512,
//     d = 4 8.7 and 8.4; from 1280 columns on it is ahead (4096 x 1280, r = 128, d = 4 9.5 and 8.5).  fp32: 4096 x 1024, r = 256, d = 2 9.6 and 10.5, d = 4 10.3 and 10.8, d = 8 12.2
//     and 11.9; in its bias pass it is ahead (d = 4 12.1 and 10.7).
//   257 to 511 blocks, r <= 128: 5120 x 1280, d = 2 10.5 and 11.4, d = 4 12.1 and 13.0, d = 8 16.0 and 15.8; r = 256 13.0 and 12.2, 13.7 and 13.1; bias pass 5120 x 4096, r = 128, d = 2
//     16.8 and 17.3, d = 4 22.0 and 21.0.
inline bool narrow_call(unsigned grid, int32_t n, int32_t r, int32_t d, int elem_size, bool norms) {
    if (grid <= kResidentDeep) {
        if (n > 1024) return false;
        return elem_size == 2 ? r <= 64 * d : !norms && d <= 4;
    }
    if (grid >= 512) return false;
    return r <= 128 && d <= (norms ? 2 : 4);
}

template <typename D, int RG, int PS, int NT, bool NORMS = false>
static hipError_t launch_d(ApplyGroup& g, int32_t r, int32_t d, int passes, hipStream_t st, float* partial = nullptr) {
    // widest matrices first: workgroups are started in index order as CUs fall free, and a workgroup's
    // run time grows with n, so the long ones should not be the last to start
    for (int a = 1; a < g.count; ++a)
        for (int b = a; b > 0 && g.p[b].n > g.p[b - 1].n; --b) std::swap(g.p[b], g.p[b - 1]);
    bool fast = true, pair = true, lines = true;
    g.r = r; g.d = d; g.partial = partial;
    unsigned grid = 0;
    for (int p = 0; p < kMaxGroup; ++p) {                           // about `passes` passes for every workgroup
        ApplyProblem& x = g.p[p];
        g.first[p] = INT32_MAX;
        if (p >= g.count) continue;
        fast = fast && fast_shape(x.n, d);
        pair = pair && x.n % 2 == 0;
        lines = lines && x.n % 32 == 0;
        x.parts = (int32_t)((((int64_t)x.n + 2 * NT - 1) / (2 * NT) + passes - 1) / passes);
        g.first[p] = x.first = (int32_t)grid;
        grid += (unsigned)((x.m + RG * 4 - 1) / (RG * 4) * x.parts);
    }
    hipError_t e;
    const bool narrow = RG == 4 && NT == 512 && d <= 8 && narrow_call(grid, g.p[0].n, r, d, D::size, NORMS);   // (the matrices are in the order of their widths)
    if (RG > 1 && fast && !narrow && wide_group(g, r)) {
        constexpr int LP = RG <= 2 ? 2 : 4, G = RG <= 2 ? 1 : RG / 4;
#define LSP_LAUNCH_WIDE(DDV, FORM)                                                                             \
    do {                                                                                                       \
        constexpr auto kern = k_decompress_wide<D, G, LP, DDV, (PS > 16384), NT, NORMS, FORM>;                 \
        constexpr size_t ents = (size_t)RG * 4 * DDV * sizeof(int2);                                           \
        constexpr size_t units = G > 1 ? (size_t)RG * PS : (size_t)(PS > 16384 ? 2048 : 1024) * 16 * LP;       \
        if ((e = allow_dynamic_lds<kern, units + ents>()) != hipSuccess) return e;                             \
        const size_t lds = (G > 1 ? units : (size_t)r * 16 * LP) + ents;                                       \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, st, g);                           \
        return hipGetLastError();                                                                              \
    } while (0)
// (8 rows at d = 16 and r <= 1024: at most 128 blocks of 16 rows, so the grid is never beyond that of the deep form)
#define LSP_WIDE(DDV)                                                                                          \
    do {                                                                                                       \
        if constexpr (G == 1 && NT == 512)                                                                     \
            if (grid <= kResidentDeep) LSP_LAUNCH_WIDE(DDV, kDeep);                                            \
        if constexpr (G == 1 && NT == 512 && DDV <= 8 && D::size == 2 && !NORMS)                               \
            if (grid < 512 && g.p[0].n <= 2048) LSP_LAUNCH_WIDE(DDV, kPlain);                                    \
        if constexpr ((D::size == 2 || DDV == 16 || NORMS) && (LP == 4 || PS > 16384)) LSP_LAUNCH_WIDE(DDV, (G == 1 ? kTwo : kPlain));   \
    } while (0)
        if constexpr (LP == 4) {
            if (d == 2) LSP_WIDE(2);
            if (d == 4) LSP_WIDE(4);
            if (d == 8) LSP_WIDE(8);
        }
        if constexpr (NT == 512 && RG > 1)
            if (d == 16) LSP_WIDE(16);
#undef LSP_WIDE
#undef LSP_LAUNCH_WIDE
    }
    if constexpr (RG <= 4 && RG > 1 && NT == 512 && PS <= 16384) {
        if (!(fast && wide_group(g, r)) && loose_group(g, d) && loose_call(grid, g.p[0].n, r, d, D::size, fast, pair, lines, RG == 2, NORMS)) return launch_loose<D>(g, grid, RG == 2, NORMS, st);
    }
#define LSP_LAUNCH_FAST(DDV)                                                                                   \
    do {                                                                                                       \
        constexpr auto kern = k_decompress<D, RG, DDV, PS, NT, NORMS>;                                         \
        constexpr size_t lds = (size_t)RG * PS + (size_t)RG * 4 * DDV * sizeof(int2);                          \
        if ((e = allow_dynamic_lds<kern, lds>()) != hipSuccess) return e;                                        \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, st, g);                            \
        return hipGetLastError();                                                                              \
    } while (0)
    if (fast && d == 2) LSP_LAUNCH_FAST(2);
    if (fast && d == 4) LSP_LAUNCH_FAST(4);
    if (fast && d == 8) LSP_LAUNCH_FAST(8);
    if constexpr (RG <= 4 && NT == 512) {                           // the others are for the fast kernel at d <= 8
        if constexpr (RG > 1)                                       // (4 rows: d <= 8)
            if (fast && d == 16) LSP_LAUNCH_FAST(16);
#define LSP_LAUNCH_ANY(PAIRV)                                                                                  \
    do {                                                                                                       \
        constexpr auto kern = k_decompress_any<D, RG, PS, NT, PAIRV, NORMS>;                                   \
        if ((e = allow_dynamic_lds<kern, (size_t)RG * PS + (size_t)RG * 4 * LSP_MAX_D * sizeof(int2)>()) != hipSuccess) return e; \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), (size_t)RG * PS + (size_t)RG * 4 * d * sizeof(int2), st, g); \
        return hipGetLastError();                                                                              \
    } while (0)
        if (pair) LSP_LAUNCH_ANY(true);
        LSP_LAUNCH_ANY(false);
#undef LSP_LAUNCH_ANY
    }
#undef LSP_LAUNCH_FAST
    return hipErrorInvalidValue;
}

// Workgroups of 8 rows instead of 16, given the number of blocks of 16 rows (n: the widest matrix; wide: k_decompress_wide's shapes).  With 8 rows there are
// twice as many workgroups, but each reads all of Q, and d <= 8 goes to k_decompress.  (us, 8 rows | 16 rows, apply and bias pass, W and G from HBM.)
//   * At most 128 blocks, half of the CUs idle otherwise: 8 rows.
//       1000 x 2048, r = 128, d = 2, bf16     6.2 |  8.0     8.3 |  9.4        2048 x 2048, r = 512, d = 8, bf16    11.5 | 13.6    13.7 | 15.7
//       2048 x 16384, r = 256, d = 4, bf16   31.3 | 46.3    27.3 | 32.9        2048 x 8192, r = 256, d = 16, fp32   42.9 | 60.1    36.9 | 45.4
//       2048 x 2048, r = 256, d = 16, bf16   13.4 | 19.5    15.8 | 20.0        1000 x 4096, r = 512, d = 16, bf16   21.3 | 32.8    22.8 | 30.7
//       2048 x 2047, r = 250, d = 5, bf16     8.6 | 12.2    10.7 | 12.8        2040 x 8191, r = 900, d = 7, bf16    26.7 | 39.8    23.2 | 29.9
//       2048 x 2047, r = 250, d = 5, fp32    11.7 | 14.6                       2040 x 8191, r = 900, d = 7, fp32    42.7 | 53.9
//     (Rows of 16 KB are the exception: 2048 x 4096, r = 512, d = 8, fp32     29.5 | 26.6    23.3 | 21.5.)
//   * 129 to 255 blocks: some CUs have two workgroups of 8 rows and others one.  16 rows, the more so the larger d is:
//       2064 x 4096, r = 512, d = 8, bf16    23.3 | 19.9    23.8 | 21.0        3072 x 16384, r = 512, d = 8, bf16   76.0 | 63.1    62.5 | 50.6
//       4080 x 4096, r = 512, d = 8, fp32    45.9 | 31.4    34.7 | 24.5        4080 x 8192, r = 256, d = 16, bf16   90.7 | 58.3    95.8 | 49.6
//       3072 x 2048, r = 512, d = 8, fp32    20.7 | 18.1    20.5 | 16.3        3072 x 2048, r = 256, d = 4, fp32    16.1 | 15.1    14.5 | 12.7
//       4080 x 4096, r = 256, d = 4, bf16       (bias)      18.3 | 16.2        4073 x 8191, r = 250, d = 7, bf16    46.7 | 44.1    35.7 | 29.0
//     but 8 rows in fp32 below 4096 columns where the lists are short and the tile small (r <= 64 d), in the apply step up to 1024 columns whatever d is:
//       4080 x 1024, r = 256, d = 4, fp32     9.8 | 11.0    11.7 | 11.0        3072 x 1024, r = 512, d = 2, fp32    10.7 |  9.4    13.1 | 10.7
//       2064 x 3072, r = 128, d = 2, fp32    17.0 | 17.3    12.8 | 14.8        4080 x 2048, r = 128, d = 2, fp32    16.2 | 15.9    12.7 | 12.5
//     and in the bias pass of long rows in 16 bits at d = 2 and r <= 256: 2064 x 8192, r = 128 16.4 | 17.9; 4080 x 16384, r = 256 30.7 | 31.1; r = 512 33.8 | 31.3.  Where 16 rows
//     would be k_decompress as well they are even or behind at d <= 4: 2064 x 3074, r = 256, d = 4, fp32 20.7 | 22.1, bias 16.6 | 17.6 (3072 rows 19.2 | 18.4); 2064 x 8194, bf16 (bias) 24.2 | 25.7.
inline bool eight_rows(int64_t blocks, int64_t n, int32_t r, int32_t d, int elem_size, bool fast, bool wide, bool norms) {
    if (r > 1024 || blocks <= 128) return true;                     // (r > 1024: 16 rows of U would take the whole LDS)
    if (blocks > 255 || r > 512 || !fast || d > 8) return false;
    if (elem_size == 2) return norms && (wide ? n >= 8192 && d <= 2 && r <= 256 : n >= 4096 && d <= 4);
    if (n >= 4096) return false;
    return wide ? r <= 64 * d && (d <= 2 || (!norms && n <= 1024)) : d <= 4;
}

// The apply step with at most 64 blocks of 16 rows, where blocks of 8 would leave half of the CUs idle: blocks of 4 rows in k_decompress and k_decompress_any, or of 8 in the two kernels
// that share units between lanes, and a row block's passes shared by as many workgroups as there are CUs for (each makes the tile of U).  (us, 8 rows and with this; bf16 and fp32.)
//   4 rows: 1024 x 1024, r = 128, d = 4 4.9 and 3.6, 5.4 and 3.9; 1024 x 4096, r = 512, d = 8 13.6 and 10.6, 20.1 and 13.7; 768 x 3072, r = 384, d = 4 8.2 and 6.2, 10.5 and 7.7; 1024 x 2048,
//     r = 1000, d = 8 10.9 and 9.1, 13.2 and 10.3; n odd 1001 x 701, r = 100, d = 5 5.1 and 4.6, 5.2 and 4.7; fp32 1001 x 2999, r = 250, d = 5 12.6 and 10.6.
//   Passes shared: 512 x 2048, r = 128, d = 8 7.3 (4 rows 6.0) and 4.8, 8.7 (6.9) and 5.0.
//   8 rows: d = 16 (4 rows: 1024 x 4096, r = 512 19.7 and 23.4); 16 bits, n odd, more than 1024 columns (1001 x 2003, r = 120, d = 3 6.2 and 6.8).
//   More than 12 entries a row, which k_decompress_any reads from L2 for every block: 8 rows too (bf16, 8 rows, 4 and 8 with the passes shared: 1024 x 2048, r = 341, d = 32 1, 1.19 and 0.75 of the time, 513 x
//     4099, r = 171, d = 14 1, 0.82 and 0.55), unless there is half a pass at the most, with nothing to share (1024 x 131, d = 20 1, 0.89 and 0.98).
// fp32 with 113 to 128 blocks and r <= 512, two workgroups of 4 rows on nearly every CU, of which 4 rows read Q twice as often as 8: d <= 4 up to 6144 columns (8 rows and 4, times: 2048 x 2048, r = 512 1.23 with
// d = 2 and 1.10 with d = 4, 2048 x 6144 1.09 and 1.00, 8192 columns 0.86 and 0.81), and rows of 16 KB, 8 of which fare badly together (2048 x 4096, r = 512, d = 8 29.2 and 23.1 us; 4000 columns 0.86 times,
// 4104 0.89, 12288 0.88); with fewer blocks some CUs have one (1500 x 3000, r = 256, d = 8 14.5 and 16.5 us), and in 16 bits 8 rows are the better ones (2048 x 4096 16.2 and 17.4).
inline bool few_blocks(int64_t blocks, int64_t n, int32_t r, int32_t d, int elem_size, bool fast) {
    if (r > 1024) return false;
    return blocks <= 64 || (elem_size == 4 && fast && r <= 512 && blocks > 112 && blocks <= 128 && ((d <= 4 && n <= 6144) || (d <= 8 && n == 4096)));
}

// Rows per workgroup: 16 (four planes of U in LDS) or 8 (above), and 512 threads, except
//   * 1024 or more blocks, 16-bit storage, 256 < r <= 512: 32 rows, so that the rows of Q are streamed from L2 half as
//     often (the seven matrices of a 6.7B-style layer, d = 8, one call: 202 us, with 16 rows 227; d = 16 325 and 335; 16384 x 4096, r = 512, d = 8 67.2 and 73.3); fp32 patches of 32
//     rows would not fit the registers.  Nor where k_expand_loose serves (16384 x 4098, d = 4), which has 16;
//     With few entries of Q in k_decompress_wide 16 rows are the faster ones, which ask ahead and end more evenly: d = 2, from 2048 columns on: the layer 161.5 and 148.7 us,
//     16384 x 4096 53.9 and 51.3, 20000 x 8192 156 and 118 (1024 columns 17.4 and 17.8); d = 4, 2048 to 8192 columns: 16384 x 4096 57.6 and 56.1, 20000 x 8192 162 and 130, but
//     four matrices 4096 x 11008 153.7 and 157.4;
//   * 512 or more blocks and r <= 512: 256 threads with at most eight passes each; four such workgroups share a CU and
//     cover each other's set-up.  It is even with 512 threads in 16 bits (11008 x 4096, r = 512, d = 8 55.9 | 54.7; 8192 x 4096
//     40.5 | 40.8; 16384 x 4096, r = 256, d = 4 53.8 | 54.3; 8192 x 2048, r = 512, d = 4 20.8 | 19.9) and ahead in fp32 (82.6 | 84.7; 16384 x 4096: 114 | 117.5).
template <typename D>
static hipError_t launch_d_shape(ApplyGroup& g, int32_t r, int32_t d, hipStream_t st) {
    constexpr int kAll = 1 << 30;                                   // no row block is shared
    int64_t blocks = 0, widest = 0;
    bool fast = true, pair = true, lines = true;
    for (int p = 0; p < g.count; ++p) {
        blocks += (g.p[p].m + 15) / 16;
        pair = pair && g.p[p].n % 2 == 0;
        lines = lines && g.p[p].n % 32 == 0;
        widest = g.p[p].n > widest ? g.p[p].n : widest;
        fast = fast && fast_shape(g.p[p].n, d);
    }
    if (r > 1024) return launch_d<D, 2, 32768, 512>(g, r, d, kAll, st);
    const bool wide = wide_group(g, r);
    const bool loose8 = !(fast && wide) && loose_group(g, d) && loose_call((unsigned)(2 * blocks), (int32_t)widest, r, d, D::size, fast, pair, lines, true, false);
    if (few_blocks(blocks, widest, r, d, D::size, fast)) {
        const bool eight = blocks <= 64 && (fast ? d > 8 : d > kLooseEntries ? widest > 512 : loose8 && D::size == 2);
        int64_t each = 0;                                           // row blocks
        for (int p = 0; p < g.count; ++p) each += eight ? (g.p[p].m + 7) / 8 : (g.p[p].m + 3) / 4;
        const int64_t passes = (widest + 1023) / 1024, share = std::max<int64_t>(1, kResidentDeep / each);
        const int most = (int)((passes + share - 1) / share);
        if (eight) return r <= 256 ? launch_d<D, 2, 4096, 512>(g, r, d, most, st) : r <= 512 ? launch_d<D, 2, 8192, 512>(g, r, d, most, st)
                                                                                            : launch_d<D, 2, 16384, 512>(g, r, d, most, st);
        return r <= 256 ? launch_d<D, 1, 4096, 512>(g, r, d, most, st) : r <= 512 ? launch_d<D, 1, 8192, 512>(g, r, d, most, st)
                                                                                  : launch_d<D, 1, 16384, 512>(g, r, d, most, st);
    }
    if (eight_rows(blocks, widest, r, d, D::size, fast, wide, false))
        return r <= 256 ? launch_d<D, 2, 4096, 512>(g, r, d, kAll, st) : r <= 512 ? launch_d<D, 2, 8192, 512>(g, r, d, kAll, st)
                                                                                 : launch_d<D, 2, 16384, 512>(g, r, d, kAll, st);
    const bool loose = !(fast && wide) && loose_group(g, d) && loose_call((unsigned)blocks, (int32_t)widest, r, d, D::size, fast, pair, lines, false, false);
    if constexpr (D::size == 2)
        if (fast && !loose && (d <= 8 || wide) && blocks >= 1024 && 256 < r && r <= 512 && !(wide && d <= 4 && widest >= 2048 && (d <= 2 || widest <= 8192)))
            return launch_d<D, 8, 8192, 512>(g, r, d, kAll, st);
    if (fast && !loose && d <= 8 && blocks >= 512 && r <= 512)
        return r <= 256 ? launch_d<D, 4, 4096, 256>(g, r, d, 8, st) : launch_d<D, 4, 8192, 256>(g, r, d, 8, st);
    return r <= 256 ? launch_d<D, 4, 4096, 512>(g, r, d, kAll, st) : r <= 512 ? launch_d<D, 4, 8192, 512>(g, r, d, kAll, st)
                                                                             : launch_d<D, 4, 16384, 512>(g, r, d, kAll, st);
}

// Estimation bias: one problem, one pair of sums per workgroup.
inline bool bias_eight_rows(int64_t m, int64_t n, int32_t r, int32_t d, int elem_size) {
    return eight_rows((m + 15) / 16, n, r, d, elem_size, fast_shape((int32_t)n, d), wide_shape(n, r), true);
}
template <typename D>
static hipError_t launch_bias_shape(ApplyGroup& g, int32_t r, int32_t d, float* partial, hipStream_t st) {
    constexpr int kAll = 1 << 30;
    const int64_t m = g.p[0].m;
    const bool eight = bias_eight_rows(m, g.p[0].n, r, d, D::size);
    if (r > 1024) return launch_d<D, 2, 32768, 512, true>(g, r, d, kAll, st, partial);
    if (eight)    return r <= 256 ? launch_d<D, 2, 4096, 512, true>(g, r, d, kAll, st, partial) : r <= 512 ? launch_d<D, 2, 8192, 512, true>(g, r, d, kAll, st, partial)
                                                                                                : launch_d<D, 2, 16384, 512, true>(g, r, d, kAll, st, partial);
    return r <= 256 ? launch_d<D, 4, 4096, 512, true>(g, r, d, kAll, st, partial) : r <= 512 ? launch_d<D, 4, 8192, 512, true>(g, r, d, kAll, st, partial)
                                                                                      : launch_d<D, 4, 16384, 512, true>(g, r, d, kAll, st, partial);
}

}  // namespace lsp
