// Compress: S = P^T G Q  (Alg. 1, compress step; Alg. 3, projected gradient of a layer).
//
// Two kernels per call, both gather-form and free of global atomics in the common case:
//   A  T = G Q     (fp16, fp32 and raw calls; bf16 with a kept plan: compress_mm.hip)
//                  one workgroup per block of 8 rows of G (4 of fp32); G is streamed once from HBM in
//                  chunks of kChunk columns and staged in LDS transposed, as it is stored, one 16-byte
//                  unit per column, so one 128-bit LDS read serves all rows of the block; each
//                  lane owns one column b of T and walks the plan's list of (column of G, value)
//                  pairs of b, accumulating in registers.  With one column per lane the plan deals
//                  the lists of every chunk to the waves by length, and the partial sums change
//                  lanes between chunks (swap_owner).
//   B  S = P^T T   one wave per piece of a row of P^T and 1/8 of the columns; reads rows of T.
// The path streams G once.  Kernel A is nearest to the vector ALUs' issue rate (8 widenings and 8 FMAs per pair and 8 rows
// of 16-bit storage), not to HBM: the vector ALUs issue in 67 % of the cycles, the LDS works 45 %, and L2 hands out the plan once per
// block of 8 rows; the waves (3.3 a SIMD, 4 fit) wait for data 42 % of their time (bf16, the matrices of a 6.7B-style layer).  For bf16 with a
// kept plan the matrix cores take the sums over (compress_mm.hip).  For fp16 they do not yet: three fp16 parts of an fp32 value are exact only if each has
// a power of two of its own (in a column of its own that is possible) and the values lie within 2^29 of the largest.  fp32 has no such instruction.

#include <algorithm>

#include "compress_common.h"

namespace lsp {

// ----------------------------------------------------------------------------------------------
// Kernel B for r < 4: S[a][stripe] (+)= sum_e v_e T[i_e][stripe] for one piece of a
// row of P^T and one stripe of 256 columns, one column per thread.
constexpr int kThreadsB = 256;
constexpr int kStripeQuads = 64;                              // column quads (float4) per stripe
__global__ __launch_bounds__(kThreadsB) void k_compress_pt(const CompressGroup) {
    const auto* grp = group_args<CompressGroup>();
    const auto pick = pick_problem(grp, grp->first_pt, (int)blockIdx.x);
    const CompressProblem& pr = pick.p;
    const int r = pick.r, d = pick.d, nstripes = pick.quads;
    const bool tiles = pick.tiles != 0;
    const uint8_t* __restrict__ plan = pr.plan;
    const float* __restrict__ T = pr.T;
    float* __restrict__ S = pr.S;
    const int block = (int)blockIdx.x - pr.first_pt;
    const LoadedHeader H = load_header(plan);
    if (!plan_matches(H, pr.m, pr.n, r, d, tiles)) return;                   // kernel A has filled S with NaN
    const int stripe = block % nstripes, item = block / nstripes;
    if (item >= H->p_nitems) return;
    words4 fields = scalar_load<words4>(as_const<RowItem>(plan + H->off_p_item) + item);
    arrived(fields);
    const RowItem it{(int32_t)fields[0], (int32_t)fields[1], (int32_t)fields[2], (int32_t)fields[3]};
    const uint2* ent = reinterpret_cast<const uint2*>(plan + H->off_p_ent) + it.start;
    for (int b = stripe * kStripeQuads * 4 + threadIdx.x; b < min(r, (stripe + 1) * kStripeQuads * 4); b += kThreadsB) {
        float acc = 0.0f;
        for (int e = 0; e < it.len; ++e) {
            const uint2 en = ent[e];
            acc = fmaf(__uint_as_float(en.y), T[(int64_t)en.x * r + b], acc);
        }
        float* dst = S + (int64_t)it.a * r + b;
        if (it.atomic) atomicAdd(dst, acc); else *dst = acc;
    }
}

// Kernel B, the usual variant (r >= 4), XCD-aware.  The columns of T are cut into 8 stripes, one per XCD:
// workgroups are dealt to the 8 XCDs round-robin, so with stripe = blockIdx % 8 an XCD only ever
// touches its own m x r/8 slice of T, which fits its 4 MB L2 -- T comes from HBM once instead of
// once per use (each row of T is used by d rows of S).  Each of the 4 waves of a workgroup takes
// one piece of a row of P^T; its 64 lanes form 64/LG groups of LG lanes (LG = 8, 16, 32 or 64 >= quads
// per stripe), group g takes entries g, g + groups, ...; the groups' sums meet through lane
// exchanges in a fixed order.  Where a slice would be larger than the L2, each XCD may take its columns in two rounds (rounds_of).
// A row's last quad starts at r - 4 when r is no multiple of 4 and stores only what the
// quad before it has not (3001 rows, r = 250, d = 5: 26 us one column a thread, now 6).
// With r up to 256, eight lanes a group and not sixteen, half of them without a column, make one trip to L2 of 64 entries and not two (us, both kernels of compress, sixteen and
// eight: 4096 x 4096, r = 256, d = 8, bf16 23.8 and 22.5; 2048 x 2048, r = 128, d = 8, fp16 14.2 and 13.2; 320 x 1216, r = 16, d = 8 12.3 and 10.9).
template <int LG>
__global__ __launch_bounds__(kThreadsB) void k_compress_pt8(const CompressGroup) {
    constexpr int NG = kWave / LG;                            // entry groups per wave
    const auto* grp = group_args<CompressGroup>();
    const auto pick = pick_problem(grp, grp->first_pt, (int)blockIdx.x);
    const CompressProblem& pr = pick.p;
    const int r = pick.r, d = pick.d, sq = pick.quads;
    const bool tiles = pick.tiles != 0;
    const uint8_t* __restrict__ plan = pr.plan;
    const float* __restrict__ T = pr.T;
    float* __restrict__ S = pr.S;
    const int block = (int)blockIdx.x - pr.first_pt;
    const LoadedHeader H = load_header(plan);
    if (!plan_matches(H, pr.m, pr.n, r, d, tiles)) return;                   // kernel A has filled S with NaN
    const bool second = block >= pr.round_pt;
    const int at_block = second ? block - pr.round_pt : block;
    const int stripe = (at_block & 7) + (second ? 8 : 0);
    const int item = (at_block >> 3) * (kThreadsB / kWave) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (item >= H->p_nitems) return;
    words4 fields = scalar_load<words4>(as_const<RowItem>(plan + H->off_p_item) + item);
    arrived(fields);
    const RowItem it{(int32_t)fields[0], (int32_t)fields[1], (int32_t)fields[2], (int32_t)fields[3]};
    const uint2* ent = reinterpret_cast<const uint2*>(plan + H->off_p_ent) + it.start;
    const int lane = threadIdx.x & 63;
    const int grp_e = lane / LG, ql = lane % LG;
    const int b4 = stripe * sq + ql;
    const bool live = ql < sq && b4 * 4 < r;
    const int b = live ? min(b4 * 4, r - 4) : 0;                      // first column of this lane's quad
    typedef f32x4 loose __attribute__((aligned(4)));
    const float* Tcol = T + b;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    // The piece's entries are loaded once, 64 at a time (one per lane), and handed to the groups by
    // lane exchange, so that the loads of T do not each wait for a load of their entry and can
    // all be in flight together.  Groups without an entry in the last step load the last entry's row again and take zeros in its place (times
    // zero, an infinity there would be a NaN).
    // Eight loads of T in flight per lane: 57 to 71 registers, seven or eight waves a SIMD.  (Sixteen take 100 and more and leave four: the step over
    // seven matrices of a 6.7B-style layer 428 instead of 418 us; 4096 x 4096, r = 2048, d = 8, compress alone 60.9 -> 55.4.)
    constexpr int kSteps = kWave / NG, kAhead = 8;
    static_assert(kSteps % kAhead == 0, "a block of steps ends with the wave's entries");
    // Steps k0, k0 + 1, ... of the 64 entries, those below `last`, at most kAhead - 1; then, in a place of its own, number min(k0 + kAhead - 1, last): where that is the piece's last one, some groups may
    // have none of the `left` entries.  (Looked for in every step: attention matrices, both directions, 17.41 and 17.54 us.)
    auto take = [&](const uint2 mine, int k0, int last, int left) {
        f32x4 x[kAhead];
        float v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            x[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            v[k] = 0.0f;
            if (k == kAhead - 1 || k0 + k < last) {                             // uniform over the wave
                const int src = (k == kAhead - 1 ? min(k0 + k, last) : k0 + k) * NG + grp_e;   // lane holding entry base + step * NG + grp
                const uint32_t row = (uint32_t)__shfl((int)mine.x, src);
                v[k] = __uint_as_float((uint32_t)__shfl((int)mine.y, src));
                x[k] = *reinterpret_cast<const loose*>(Tcol + (int64_t)row * r);
            }
        }
        __builtin_amdgcn_sched_barrier(0);                                      // all of them in flight before the first is used
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (NG > 1 && k == kAhead - 1) {
                const bool has = min(k0 + k, last) * NG + grp_e < left;
                x[k].x = has ? x[k].x : 0.0f; x[k].y = has ? x[k].y : 0.0f; x[k].z = has ? x[k].z : 0.0f; x[k].w = has ? x[k].w : 0.0f;
            }
            acc.x = fmaf(v[k], x[k].x, acc.x); acc.y = fmaf(v[k], x[k].y, acc.y);
            acc.z = fmaf(v[k], x[k].z, acc.z); acc.w = fmaf(v[k], x[k].w, acc.w);
        }
    };
    int base = 0;
    uint2 next = ent[min(lane, max(it.len - 1, 0))];                            // the next 64 entries come with the rows of these
    for (; base + kWave <= it.len; base += kWave) {
        const uint2 mine = next;
        next = ent[min(base + kWave + lane, it.len - 1)];
        for (int k0 = 0; k0 < kSteps; k0 += kAhead) take(mine, k0, kSteps, kWave);
    }
    if (base < it.len) {
        uint2 mine = next;
        if (base + lane >= it.len) mine.y = 0u;
        const int left = it.len - base, last = (left - 1) / NG;
        for (int k0 = 0; k0 <= last; k0 += kAhead) take(mine, k0, last, left);
    }
#pragma unroll
    for (int step = LG; step < kWave; step *= 2) {            // group g adds group g ^ (step / LG)
        acc.x += __shfl_xor(acc.x, step); acc.y += __shfl_xor(acc.y, step);
        acc.z += __shfl_xor(acc.z, step); acc.w += __shfl_xor(acc.w, step);
    }
    if (lane < LG && live) {
        float* dst = S + (int64_t)it.a * r + b;
        const int have = b4 * 4 - b;                                  // elements that the quad before stores
        if (it.atomic) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k >= have) atomicAdd(dst + k, acc[k]);
        } else {
            *reinterpret_cast<loose*>(dst) = acc;                     // (the same sums where quads overlap)
        }
    }
}

// ----------------------------------------------------------------------------------------------
static bool walks_tiles(lsp_dtype dtype, const RawCall& raw) { return dtype == LSP_BF16 && !raw.status; }   // (plans of raw calls have no tiles)

static hipError_t launch_gq(CompressGroup& g, const RawCall& raw, lsp_dtype dtype, hipStream_t st) {
    switch (dtype) {
        case LSP_F32:  return launch_gq_f32(g, raw, st);
        case LSP_F16:  return launch_gq_f16(g, raw, st);
        default:       return walks_tiles(dtype, raw) ? launch_mm_bf16(g, st) : launch_gq_bf16(g, raw, st);
    }
}

// The hardware hands the workgroups of a launch to the CUs in index order as CUs fall free, so the
// order of the problems inside a group is the order of a greedy list schedule: the problems whose
// workgroups run longest (widest matrices: work per row block grows with n) go first, and the
// short ones fill in behind them.
static void longest_first(CompressGroup& g) {
    for (int a = 1; a < g.count; ++a)
        for (int b = a; b > 0 && g.p[b].n > g.p[b - 1].n; --b) std::swap(g.p[b], g.p[b - 1]);
}

constexpr int kMostRounds = 2;
// Rounds of kernel B: two where a slice of T, m rows of r / 8 columns, is larger than an XCD's L2 (4 MB) and half of it is made of whole lines of 128 bytes (r a multiple of 512; then no fewer of the lanes of a group
// have a column either); without whole lines only where half of it is not much larger than the L2, most lanes have a column all the same, and every row of T is wanted more than twice.  (us, with kernel A on 512
// columns, fp16, one round and two: r = 2048 8192 rows, d = 8 77.0 and 62.6, d = 2 52.0 and 51.0, 5120 rows 52.0 and 49.5, 28000 rows 326 and 294; r = 1536 8192 rows 67 and 61, 28000 rows 270 and 278; r = 1024 16384 rows
// 80 and 67, d = 2 52 and 50.  r = 1920 8192 rows, d = 8 85 and 80, d = 2 53 and 54, 16384 rows, d = 8 195 and 210; r = 1664 8192 rows 75 and 70, 12000 rows 119 and 121; r = 1040 16384 rows 120 and 132, r = 1280 128 and
// 139.  Four rounds: r = 2048 8192 rows, d = 8 67.  A slice of 4 MB: 4096 x 4096, r = 2048, bf16 44.9 and 45.6, r = 1536 37.9 and 38.6, 8192 x 4096, r = 1024 48.7 and 47.8.)
static int rounds_of(int64_t rows, int32_t r, int32_t d) {
    const int64_t slice = rows * r * 4 / 8;
    return slice > (4 << 20) && r >= 1024 && (r % 512 == 0 || (r > 1536 && d >= 4 && slice <= (9 << 20))) ? 2 : 1;
}

hipError_t launch_compress_planned(CompressGroup& g, int32_t r, int32_t d, lsp_dtype dtype, hipStream_t st, const RawCall& raw) {
    const int nstripes = (r + kStripeQuads * 4 - 1) / (kStripeQuads * 4);
    const bool striped = r >= 4, tiles = walks_tiles(dtype, raw);
    longest_first(g);
    g.r = r; g.d = d; g.tiles = tiles ? 1 : 0;
    hipError_t e = launch_gq(g, raw, dtype, st);
    if (e != hipSuccess) return e;
    // (a launch for each number of rounds that there is, nearly always one: the order of a sum depends on it, and is a matter of the matrix alone)
    for (int rounds = 1; rounds <= (striped ? kMostRounds : 1); rounds *= 2) {
        const int sq = ((r + 3) / 4 + 8 * rounds - 1) / (8 * rounds);
        g.quads = striped ? sq : nstripes;
        int32_t blocks = 0;
        for (int p = 0; p < kMaxGroup; ++p) {
            g.first_pt[p] = INT32_MAX;
            if (p >= g.count) continue;
            const int32_t items = (int32_t)plan_max_items(g.p[p].m, r, d);
            g.first_pt[p] = g.p[p].first_pt = blocks;
            g.p[p].round_pt = (items + 3) / 4 * 8;
            if (!striped) blocks += items * nstripes;
            else if (rounds_of(g.p[p].m, r, d) == rounds) blocks += g.p[p].round_pt * rounds;
        }
        if (blocks == 0) continue;
        if (!striped)      hipLaunchKernelGGL(k_compress_pt, dim3((unsigned)blocks), dim3(kThreadsB), 0, st, g);
        else if (sq <= 8) hipLaunchKernelGGL(k_compress_pt8<8>, dim3((unsigned)blocks), dim3(kThreadsB), 0, st, g);
        else if (sq <= 16) hipLaunchKernelGGL(k_compress_pt8<16>, dim3((unsigned)blocks), dim3(kThreadsB), 0, st, g);
        else if (sq <= 32) hipLaunchKernelGGL(k_compress_pt8<32>, dim3((unsigned)blocks), dim3(kThreadsB), 0, st, g);
        else               hipLaunchKernelGGL(k_compress_pt8<64>, dim3((unsigned)blocks), dim3(kThreadsB), 0, st, g);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lsp

