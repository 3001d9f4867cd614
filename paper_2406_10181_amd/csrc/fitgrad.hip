// Gradient of the data term of projector fitting with respect to the stored projector values
// (the minimisation in MaybeUpdate, Alg. 1; Eq. 2):
//     F(P, Q) = 1/2 || P P^T G Q Q^T - G ||_F^2,    gP[i][k] = dF / dP_val[i][k],   gQ[j][k] = dF / dQ_val[j][k].
// With S = P^T G Q, R = P S Q^T - G, Z = P^T R Q the chain rule gives
//     dF/dPhat = (R Q) S^T + (G Q) Z^T,          dF/dQhat = (R^T P) S + (G^T P) Z,
// and everything that involves R collapses onto r x r matrices, because
//     R Q = P S (Q^T Q) - G Q,    R^T P = Q S^T (P^T P) - G^T P,    Z = (P^T P) S (Q^T Q) - S.
// So with C_P = P^T P, C_Q = Q^T Q, S1 = S C_Q, X = C_P S (all r x r):
//     dF/dPhat[i][a] = sum_k' P_val[i][k'] M1[P_idx[i][k']][a] + sum_b T[i][b] D[a][b],      M1 = S1 S^T,
//     dF/dQhat[j][b] = sum_k' Q_val[j][k'] M2[Q_idx[j][k']][b] + sum_a Y[j][a] D[a][b],      M2 = S^T X,
//     D = Z - S = C_P S1 - 2 S,     T = G Q (m x r),     Y = G^T P (n x r).
// G is streamed twice: once by the compress kernels (T and S, as in every training step) and once, row by
// row through the column-sorted copy of P in the plan, for Y.  The dense r x r products run in fp32 on the
// matrix cores; the rest is gathers and fp32 dot products (Y and a second copy of D are kept transposed, so that both
// sides' dot products run along rows).  No m x n temporary exists.
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <utility>

#include "products.h"

namespace lsp {

// Y[j][a] = sum over the entries (i, v) of row a of P^T of v * G[i][j]: a wave has one piece of a row of P^T and a tile of
// 256 columns; a lane loads 16 bytes of a row of G, and with 16-bit storage the two halves of the wave take every
// other entry and add up through lane exchanges.  The four waves of a workgroup take consecutive pieces, nearly always
// of consecutive a, so that they write 16 bytes of a row of Y together.  Rows cut into pieces (heavily skewed projectors)
// add up with atomics on a Y that was cleared.
// Every row of G is wanted by d rows of P^T, so G goes from L2 to the CUs d times: that traffic (268 MB at
// 4096 x 4096, d = 8, 16-bit) is what the kernel's time is made of.  HBM sees G once: an XCD takes every a for a column tile
// before its next tile, so a tile of G (m rows of 256 elements, 2 MB at m = 4096) stays in that XCD's L2 for its
// d visits.  With a workgroup a piece (four waves, a quarter of the entries each, 8 bytes a lane) it took 34 us there, 23 with a wave a piece (24 with the address of a row made anew for every load: BELOW_4G,
// a 32-bit offset), now 22.6, fp16 21.8: rows and values of the entries by DPP moves and not by exchanges through LDS.  L2 hands out 12 of the 17 TB/s that it can (64 bytes a cycle and channel);
// the products on the matrix cores instead of the vector ALUs took 22.0.
// A row's last piece starts at n - VEC when n is no multiple of VEC, up to VEC - 1 columns before its tile if the tile has
// fewer than VEC columns: the wave's sums have room for them in front.  n < VEC: one column a lane (VEC = 1).
constexpr int kThreadsY = 256, kWavesY = kThreadsY / kWave, kXcds = 8, kTileY = 256;
// The work is (tile of columns, four pieces), the pieces fastest, and each XCD has an eighth of it, one after the other (workgroup b runs on XCD b % 8), so that it has hardly more than one tile of G
// at a time, and all XCDs the same amount (a tile for an XCD at a time, 4096 x 4160, r = 512, d = 8, fp16 28.3 us, so 23.8).
__device__ __forceinline__ bool place_in_y(int block, bool later, int nitems, int tiles, int& item0, int& tile) {
    const int groups = (nitems + kWavesY - 1) / kWavesY;
    const uint32_t units = (uint32_t)groups * (uint32_t)tiles, each = (units + kXcds - 1) / kXcds, half = (each + 1) / 2, seq = (uint32_t)block / kXcds + (later ? half : 0);
    const uint32_t unit = (uint32_t)block % kXcds * each + seq;
    if (seq >= (later ? each : half) || unit >= units) return false;
    tile = (int)(unit / (uint32_t)groups);
    item0 = (int)(unit - (uint32_t)tile * (uint32_t)groups) * kWavesY;
    return true;
}

// The sums of a workgroup's four pieces go to Y: part[w * stride + c] for column tile0 + c, c < WIDTH.
template <int WIDTH>
__device__ __forceinline__ void store_y(const float* part, int stride, const uint8_t* plan, const LoadedHeader& H, float* __restrict__ Y, int item0, int nitems, int tile0, int n, int r) {
    __syncthreads();
    const int c = threadIdx.x, j = tile0 + c;
    if (j >= n || c >= WIDTH) return;
    float* out = Y + (int64_t)j * r;
    int a[kWavesY];
    bool plain = true;                                              // four whole rows of P^T in a row
#pragma unroll
    for (int w = 0; w < kWavesY; ++w) {
        const auto* p = as_const<int32_t>(plan + H->off_p_item) + 4 * min(item0 + w, nitems - 1);
        a[w] = item0 + w < nitems ? p[0] : -1;
        plain = plain && a[w] == a[0] + w && p[3] == 0;
    }
    if (plain && ((a[0] | r) & 3) == 0) {
        *reinterpret_cast<f32x4*>(out + a[0]) = f32x4{part[c], part[stride + c], part[2 * stride + c], part[3 * stride + c]};
        return;
    }
#pragma unroll
    for (int w = 0; w < kWavesY; ++w) {
        if (a[w] < 0) continue;
        const auto* p = as_const<int32_t>(plan + H->off_p_item) + 4 * (item0 + w);
        if (p[3]) atomicAdd(out + a[w], part[w * stride + c]);
        else out[a[w]] = part[w * stride + c];
    }
}

template <int K> __device__ __forceinline__ uint32_t row_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x150 + K, 0xF, 0xF, true); }   // of each 16 lanes (row_newbcast)
template <typename F, int... k> __device__ __forceinline__ void each_of(const F& f, std::integer_sequence<int, k...>) { (f(std::integral_constant<int, k>{}), ...); }
// The gather and the r x r products have nothing of each other: a product is a chain of latencies on a workgroup or two a CU, the gather a matter of L2's rate.  So each of the two launches
// of products has half of the gather behind it (4096 x 4096, r = 512, d = 8, bf16: products 10 and 12 us and the gather 22, now 18 and 21; the call 98 -> 87 us).  The products come first, so that no
// chain begins late; with registers for five or six waves a SIMD the 64 x 64 tiles spill (r = 1024: 193 us, 243 and 330).
struct GatherArgs { const void* G; const uint8_t* plan; float* Y; int32_t r, d, m, n, tiles, first, side, products, later, pad; GemmProblem p[kMaxGemmBatch]; };
static_assert(sizeof(GatherArgs) == 256 && kMaxGemmBatch == 3, "records of 64 bytes, loaded whole");
template <typename D, int VEC, bool BELOW_4G, int SIDE, int GROUP>
__global__ __launch_bounds__(kThreadsY, 4) void k_gather_rows(const GatherArgs) {
    constexpr int LG = VEC == 1 ? kWave : kTileY / VEC < kWave ? kTileY / VEC : kWave;   // lanes of an entry
    constexpr int NG = kWave / LG;                                  // entries a wave takes at a time
    constexpr int kLead = VEC;                                      // room in front of a tile (VEC - 1, rounded up to whole pieces)
    constexpr int kPart = kLead + kTileY;
    __shared__ __align__(16) float lds[std::max(kWavesY * kPart, kTileFloats<SIDE, 32>)];
    const auto* args = group_args<GatherArgs>();
    words16 head = scalar_load<words16>(args);
    arrived(head);
    struct { const typename D::elem* G; const uint8_t* plan; float* Y; int32_t r, d, m, n, tiles, first, side, products, later, pad; } a;
    __builtin_memcpy(&a, &head, 64);
    if ((int)blockIdx.x < a.first) {
        const int tile = (int)(blockIdx.x / (unsigned)a.side), z = tile / a.side;
        if (z >= a.products) return;
        words16 record = scalar_load<words16>(&args->p[z]);
        arrived(record);
        const GemmProblem P = gemm_problem(record);
        const int row = tile - z * a.side, col = (int)blockIdx.x - tile * a.side;
        product_tile<SIDE, 32, GROUP>(P, a.r, row * SIDE, col * SIDE, lds);
        return;
    }
    const typename D::elem* __restrict__ G = global_pointer(a.G);
    const uint8_t* __restrict__ plan = global_pointer(a.plan);
    float* __restrict__ Y = global_pointer(a.Y);
    const int m = a.m, n = a.n, r = a.r, d = a.d;
    float (*part)[kPart] = reinterpret_cast<float (*)[kPart]>(lds);
    typedef typename D::elem Piece __attribute__((ext_vector_type(VEC)));
    typedef Piece Loose __attribute__((aligned(D::size)));
    const LoadedHeader H = load_header(plan);
    if (!plan_matches(H, m, n, r, d, false)) return;
    const int nitems = H->p_nitems;
    int item0, tile;
    if (!place_in_y((int)blockIdx.x - a.first, a.later != 0, nitems, a.tiles, item0, tile)) return;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const auto* itp = as_const<int32_t>(plan + H->off_p_item) + 4 * min(item0 + wave, nitems - 1);
    const RowItem it{itp[0], itp[1], itp[2], itp[3]};
    const uint2* ent = reinterpret_cast<const uint2*>(plan + H->off_p_ent) + it.start;
    const int tile0 = tile * kTileY, grp = lane / LG, ql = lane % LG;
    const int j0 = tile0 + ql * VEC;                                // this lane's columns
    const bool live = j0 < n && ql * VEC < kTileY;
    const int at = live ? min(j0, n - VEC) : 0;                     // where its piece starts
    float acc[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) acc[q] = 0.0f;
    // Lanes 16 x + i hold entry NG i + (which of the NG this lane's part of the wave takes) of a batch, so that a lane has each entry's row and value by a DPP move.
    constexpr int kSteps = 16, kBatch = kSteps * NG, kInFlight = 8;
    const int mine_of_batch = NG * (lane & 15) + grp;
    uint2 next = ent[min(mine_of_batch, max(it.len - 1, 0))];
    for (int base = 0; base < it.len; base += kBatch) {
        uint2 mine = next;                                           // behind the last entry: its row again, times zero
        if (base + mine_of_batch >= it.len) mine.y = 0u;
        next = ent[min(base + kBatch + mine_of_batch, it.len - 1)];
        if constexpr (BELOW_4G) mine.x *= (uint32_t)n * D::size;     // the row's offset in G, once per entry and not per load
        const int steps = (min(it.len - base, kBatch) + NG - 1) / NG;
        auto take = [&](auto which) {
            constexpr int k0 = decltype(which)::value * kInFlight;
            if (k0 >= steps) return;                                  // (uniform)
            Piece x[kInFlight];
            auto load = [&](auto step) {
                constexpr int u = decltype(step)::value;
                const uint32_t row = row_lane<k0 + u>(mine.x);
                if constexpr (BELOW_4G) x[u] = *reinterpret_cast<const Loose*>(reinterpret_cast<const char*>(G) + (row + (uint32_t)at * D::size));
                else x[u] = *reinterpret_cast<const Loose*>(G + at + (int64_t)row * n);
            };
            each_of(load, std::make_integer_sequence<int, kInFlight>{});
            __builtin_amdgcn_sched_barrier(0);                        // all of them in flight before the first is used
            auto add = [&](auto step) {
                constexpr int u = decltype(step)::value;
                const float v = __uint_as_float(row_lane<k0 + u>(mine.y));
#pragma unroll
                for (int q = 0; q < VEC; ++q) acc[q] = fmaf(v, widen<D>(x[u][q]), acc[q]);
            };
            each_of(add, std::make_integer_sequence<int, kInFlight>{});
        };
        each_of(take, std::make_integer_sequence<int, kSteps / kInFlight>{});
    }
    if constexpr (NG > 1) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[q] += __shfl_xor(acc[q], LG);
    }
    if (grp == 0 && live) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) part[wave][kLead + at - tile0 + q] = acc[q];   // (the same sums where pieces overlap)
    }
    store_y<VEC == 1 ? kWave : kTileY>(&part[0][kLead], kLead + kTileY, plan, H, Y, item0, nitems, tile0, n, r);
}

// Both gradients: g[i][k] = sum_k' val[i][k'] M[idx[i][k']][a] + sum_b X[i][b] D[a][b],  a = idx[i][k] (left: X = T, D, M1; right:
// X = Y, D^T, M2).  One wave per row i; the dot products run over its lanes, four b at a time and eight entries k
// together, so that their loads overlap; lane k' < d also carries the k'-th term of the first sum (d <= 64).  The eight
// sums meet in ten lane exchanges: each of the first three steps also halves the number of sums a lane has.
// (4096 x 4096, r = 512, d = 8: 33 us with a kernel of its own for each side and a merge of partial lists, now 20.)
struct GradSide { const float* X; const float* D; const float* M; const int32_t* idx; const float* val; float* g; int32_t rows; int32_t pad[3]; };
struct GradArgs { int32_t left_blocks, r, d, pad[13]; GradSide left, right; };
static_assert(sizeof(GradSide) == 64 && sizeof(GradArgs) == 192, "records of 64 bytes, loaded whole");
__global__ __launch_bounds__(256) void k_grad(const GradArgs) {
    typedef f32x4 loose __attribute__((aligned(4)));
    constexpr int KC = 8;
    const auto* args = group_args<GradArgs>();
    words4 head = scalar_load<words4>(args);
    words16 left = scalar_load<words16>(&args->left), right = scalar_load<words16>(&args->right);
    arrived(head, left, right);
    const int left_blocks = (int)head[0], r = (int)head[1], d = (int)head[2];
    const bool is_left = (int)blockIdx.x < left_blocks;
    GradSide s;
    const words16 side = is_left ? left : right;
    __builtin_memcpy(&s, &side, 64);
    s.X = global_pointer(s.X); s.D = global_pointer(s.D); s.M = global_pointer(s.M); s.idx = global_pointer(s.idx); s.val = global_pointer(s.val); s.g = global_pointer(s.g);
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)__builtin_amdgcn_readfirstlane(((int)blockIdx.x - (is_left ? 0 : left_blocks)) * 4 + (int)(threadIdx.x >> 6));
    if (i >= s.rows) return;
    const float* __restrict__ X = s.X + i * r;
    const float* __restrict__ Dm = s.D;
    const bool mine = lane < d;
    const int64_t own = i * d + min(lane, d - 1);                   // (every lane reads: a load that some lanes leave out would be waited for where it stands)
    const float pv = s.val[own];
    const int own_idx = s.idx[own], my_idx = mine ? own_idx : 0;
    const float* __restrict__ Mrow = s.M + (int64_t)my_idx * r;
    const int quads = r >> 2;
    for (int k0 = 0; k0 < d; k0 += KC) {
        int64_t row[KC];
        float acc[KC];
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const int a = __builtin_amdgcn_readlane(my_idx, min(k0 + q, d - 1));
            row[q] = (int64_t)a * r;
            acc[q] = Mrow[a];
        }
#pragma unroll
        for (int q = 0; q < KC; ++q) acc[q] = mine ? pv * acc[q] : 0.0f;
#pragma unroll 2
        for (int b4 = lane; b4 < quads; b4 += 64) {
            const f32x4 x = *reinterpret_cast<const loose*>(X + b4 * 4);
            f32x4 y[KC];
#pragma unroll
            for (int q = 0; q < KC; ++q) y[q] = *reinterpret_cast<const loose*>(Dm + row[q] + b4 * 4);
#pragma unroll
            for (int q = 0; q < KC; ++q) acc[q] = fmaf(x.x, y[q].x, fmaf(x.y, y[q].y, fmaf(x.z, y[q].z, fmaf(x.w, y[q].w, acc[q]))));
        }
        if (4 * quads + lane < r) {                                 // the last one to three b
            const float x = X[4 * quads + lane];
#pragma unroll
            for (int q = 0; q < KC; ++q) acc[q] = fmaf(x, Dm[row[q] + 4 * quads + lane], acc[q]);
        }
#pragma unroll
        for (int half = KC / 2, off = 32; half > 0; half >>= 1, off >>= 1)
#pragma unroll
            for (int q = 0; q < half; ++q) {
                const bool high = (lane & off) != 0;
                const float keep = high ? acc[q + half] : acc[q], give = high ? acc[q] : acc[q + half];
                acc[q] = keep + __shfl_xor(give, off);
            }
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) acc[0] += __shfl_xor(acc[0], off);
        const int k = k0 + (lane >> 3);
        if ((lane & 7) == 0 && k < d) s.g[i * d + k] = acc[0];
    }
}

// floats of workspace: T (m r) | S, C_P, C_Q, S1, X, D, D^T, M1, M2 (9 r^2) | Y (n r)
size_t fitgrad_workspace_floats(int64_t m, int64_t n, int32_t r, int32_t d) {
    (void)d;
    const size_t rr = (size_t)r * (size_t)r;
    return align_up((size_t)m * r, 64) + 9 * align_up(rr, 64) + align_up((size_t)r * (size_t)n, 64);
}

// Y = G^T P, the first half of it or the later one, and beside it the products of `batch`.
template <typename D>
static hipError_t launch_gather(const void* G, const uint8_t* plan, float* Y, int64_t m, int64_t n, int32_t r, int32_t d, bool later, const GemmBatch& batch, int products, hipStream_t st) {
    GatherArgs args{G, plan, Y, r, d, (int32_t)m, (int32_t)n};
    args.tiles = (int)((n + kTileY - 1) / kTileY);                   // (one column a lane: one tile)
    bool by16 = r % 4 == 0;                                          // groups of 16 bytes: whole ones, aligned operands
    for (int z = 0; z < products; ++z) {
        args.p[z] = batch.p[z];
        by16 = by16 && reinterpret_cast<uintptr_t>(batch.p[z].A) % 16 == 0 && reinterpret_cast<uintptr_t>(batch.p[z].B) % 16 == 0;
    }
    const bool wide = by16 && wide_products(r);
    args.side = wide ? (r + 63) / 64 : (r + 31) / 32;
    args.later = later;
    args.products = products;
    args.first = (products * args.side * args.side + kXcds - 1) / kXcds * kXcds;
    const int64_t groups = ((int)plan_max_items(m, r, d) + kWavesY - 1) / kWavesY, each = (groups * args.tiles + kXcds - 1) / kXcds;
    const int64_t grid = args.first + (each + 1) / 2 * kXcds;
    if (grid > INT32_MAX) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kThreadsY), 0, st, args);
        return hipGetLastError();
    };
    const bool below = m * n * D::size <= (int64_t)UINT32_MAX;
    constexpr int kPiece = 16 / D::size;
    auto pick = [&](auto vec, auto below_4g) {
        constexpr int V = decltype(vec)::value;
        constexpr bool B = decltype(below_4g)::value;
        return !by16 ? go(k_gather_rows<D, V, B, 32, 1>) : wide ? go(k_gather_rows<D, V, B, 64, 4>) : go(k_gather_rows<D, V, B, 32, 4>);
    };
    if (n >= kPiece) return below ? pick(std::integral_constant<int, kPiece>{}, std::true_type{}) : pick(std::integral_constant<int, kPiece>{}, std::false_type{});
    return below ? pick(std::integral_constant<int, 1>{}, std::true_type{}) : pick(std::integral_constant<int, 1>{}, std::false_type{});
}

hipError_t launch_fitgrad(const void* G, const uint8_t* plan, const int32_t* P_idx, const float* P_val,
                          const int32_t* Q_idx, const float* Q_val, int64_t m, int64_t n, int32_t r, int32_t d,
                          float* gP, float* gQ, float* ws, lsp_dtype dtype, hipStream_t st) {
    const size_t rr = align_up((size_t)r * (size_t)r, 64);
    float* T = ws;
    float* S = T + align_up((size_t)m * r, 64);
    float* CP = S + rr; float* CQ = CP + rr; float* S1 = CQ + rr; float* X = S1 + rr;
    float* Dm = X + rr; float* Dt = Dm + rr; float* M1 = Dt + rr; float* M2 = M1 + rr;
    float* Y = M2 + rr;
    hipError_t e;
    // T = G Q and S = P^T T: the compress kernels (a plan of another problem leaves S full of NaN, which then
    // reaches every output)
    CompressGroup g;
    memset(&g, 0, sizeof(g));
    g.count = 1; g.p[0].G = G; g.p[0].plan = plan; g.p[0].T = T; g.p[0].S = S; g.p[0].m = (int32_t)m; g.p[0].n = (int32_t)n;
    if ((e = launch_compress_planned(g, r, d, dtype, st)) != hipSuccess) return e;
    // C_P = P^T P, C_Q = Q^T Q
    GramBatch grams{};
    grams.p[0] = GramPair{P_idx, P_val, P_idx, P_val, m, CP, {}};
    grams.p[1] = GramPair{Q_idx, Q_val, Q_idx, Q_val, n, CQ, {}};
    const GramClear clear{plan, Y, (int64_t)r * n};                  // (pieces of rows of P^T add up in Y)
    if ((e = launch_gram(grams, 2, d, r, &clear, st)) != hipSuccess) return e;
    // the r x r chain: two launches of independent products
    GemmBatch first{}, second{};
    first.p[0] = GemmProblem{S, CQ, S1, nullptr, 0.0f, 0, nullptr, {}};                                               // S1 = S C_Q
    first.p[1] = GemmProblem{CP, S, X, nullptr, 0.0f, 0, nullptr, {}};                                                // X  = C_P S
    second.p[0] = GemmProblem{CP, S1, Dm, S, -2.0f, 0, Dt, {}};                                                  // D  = C_P S1 - 2 S
    second.p[1] = GemmProblem{S1, S, M1, nullptr, 0.0f, kGemmTB, nullptr, {}};                                        // M1 = S1 S^T
    second.p[2] = GemmProblem{S, X, M2, nullptr, 0.0f, kGemmTA, nullptr, {}};                                         // M2 = S^T X
    // ... and beside them Y = G^T P
    auto beside = [&](bool later, const GemmBatch& batch, int products) {
        switch (dtype) {
            case LSP_F32:  return launch_gather<F32>(G, plan, Y, m, n, r, d, later, batch, products, st);
            case LSP_F16:  return launch_gather<F16>(G, plan, Y, m, n, r, d, later, batch, products, st);
            default:       return launch_gather<BF16>(G, plan, Y, m, n, r, d, later, batch, products, st);
        }
    };
    if ((e = beside(false, first, 2)) != hipSuccess) return e;
    if ((e = beside(true, second, 3)) != hipSuccess) return e;
    const int left_blocks = (int)((m + 3) / 4), right_blocks = (int)((n + 3) / 4);
    GradArgs grad{};
    grad.left_blocks = left_blocks; grad.r = r; grad.d = d;
    grad.left = GradSide{T, Dm, M1, P_idx, P_val, gP, (int32_t)m, {}};
    grad.right = GradSide{Y, Dt, M2, Q_idx, Q_val, gQ, (int32_t)n, {}};
    hipLaunchKernelGGL(k_grad, dim3((unsigned)(left_blocks + right_blocks)), dim3(256), 0, st, grad);
    return hipGetLastError();
}

}  // namespace lsp
