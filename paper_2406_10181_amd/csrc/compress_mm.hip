// Compress, kernel A for bf16: T = G Q on the matrix cores.  See compress.hip for the path as a whole.
//
// A column of T is a sum over a list of (column of G, value), and the lists share nothing, so this is no matrix product.  But
// v_mfma_f32_4x4x4_16b_bf16 is 16 independent products [4 x 4] [4 x 4], and each can serve a list: its A operand is four values from the list
// as three bf16 parts that add up, each times its power of two, to the fp32 value exactly (in three of its rows), its B operand their four columns
// of G (4 rows; gathered by transposing LDS reads, which hand a lane one row's four values).  So a product of 16 bits by 24 is taken exactly, and
// the three sums, which a lane has for its row side by side, are added at the end: the error against 64 bits is 0.3 to 0.6 of that of a chain of fp32 FMAs.  An instruction does
// 4 rows x 64 entries; the vector ALUs took 8 widenings and FMAs for 8 rows x 64 entries.
//
// One workgroup a CU, persistent: 8 waves walk the lists (the plan's tiles: lsp_internal.h), 4 fetch and stage the next chunk of G.
// 4096 x 16384, r = 512, d = 8, skewed columns: 91.0 -> 77.9 us with kernel B; 4096 x 11008: 52.6 -> 50.7; a 6.7B layer's seven matrices
// 234 -> 216; 3001 x 2999, r = 250, d = 5: 22.7 -> 20.9.
// What bounds it (11008 x 4096, cycles of a chunk, some 14000): the walk 10700, of it LDS reads at random 8-byte units, 7.6 cycles each instead of
// 2.7 (alone 8700), the plan from L2 behind the loads of G (alone 7500), adding up the tiles 1900; staging 900; storing T 1000 a block.
// Entries ordered against bank conflicts make the reads 1.7 times as fast and the kernel 3 to 4 % (the plan's loads remain), for a plan build
// that costs more than it gives; 512 threads and 8 rows, twice a CU, or 12 walking waves and narrower tiles were 2 to 8 % slower.
#include <algorithm>

#include "compress_common.h"

namespace lsp {

typedef short s16x4 __attribute__((ext_vector_type(4)));
#define LSP_LDS_AS __attribute__((address_space(3)))

constexpr int kPlaneBytes = (kChunk + 1) * 8;                         // 8-byte units of a plane; the last one stays zero
constexpr int kLdsMM = 160 * 1024;
constexpr int kWalkers = kWavesMM * kWave;                            // threads that walk the lists
constexpr int kFetchers = kChunk / 8;                                 // threads that fetch and stage G
constexpr int kThreadsMM = kWalkers + kFetchers;
constexpr int kResidentMM = 256;                                      // one workgroup a CU

template <int NP> constexpr int kRowsMM = 4 * NP;                     // rows of a block: NP planes of 4
template <int NP> constexpr int kTileBase = (NP * kPlaneBytes + 15) / 16 * 16;   // LDS offset of the sums

// Rows 2k and 2k+1 of two adjacent columns sit in the dwords a (row 2k) and b (row 2k+1); the unit
// of the even column takes their low halves, that of the odd column their high halves (one byte permute).
__device__ __forceinline__ uint32_t row_pair(uint32_t a, uint32_t b, bool odd_column) {
    return __builtin_amdgcn_perm(b, a, odd_column ? 0x07060302u : 0x05040100u);
}

// Fetches and stages rows of a chunk (NH planes of them, from row i0 on): 8 columns a thread, so that a wave's loads are 16 bytes a
// lane.  Rows past the matrix are read from its last row and columns past it from its first ones: what they hold is never used.
// WHOLE: n % 8 == 0.  Otherwise a piece that would end behind the matrix's last element is read from where it ends with it and put
// right when it is arranged.
template <int NH, bool WHOLE> struct RowStager {
    static constexpr int RT = 4 * NH;
    typedef u32x4 Loose __attribute__((aligned(2)));
    u32x4 pre[RT];
    int late, late_from;                                              // rows from late_from on were read `late` elements early

    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ G, int64_t i0, int m, int n, int c, int tid) {
        const uint32_t col0 = (uint32_t)c * kChunk + (uint32_t)tid * 8;
        const uint32_t byte0 = (col0 < (uint32_t)n ? col0 : 0u) * 2;
        if (i0 > m - 1) i0 = m - 1;
        const int last = (int)(m - 1 - i0 < RT - 1 ? m - 1 - i0 : RT - 1);   // rows of the part inside the matrix, less one
        const char* base = reinterpret_cast<const char*>(G + i0 * (int64_t)n);   // uniform over a wave, as the rows are
        const uint64_t stride = (uint64_t)n * 2;
        if constexpr (!WHOLE) {
            late = 0; late_from = RT;
            if (n < 8) {                                              // element by element
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    uint16_t x[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) x[q] = G[(i0 + (t < last ? t : last)) * n + (q < n ? q : n - 1)];
                    __builtin_memcpy(&pre[t], x, 16);
                }
                return;
            }
            if (i0 + last == m - 1) {
                late_from = last;
                if (col0 < (uint32_t)n && col0 + 8 > (uint32_t)n) late = (int)(col0 + 8 - (uint32_t)n);
            }
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            uint32_t at = byte0;
            if constexpr (!WHOLE) at -= t >= late_from ? (uint32_t)late * 2 : 0u;
            pre[t] = __builtin_nontemporal_load(reinterpret_cast<const Loose*>(base + at));
            base += t < last ? stride : 0;
        }
    }
    // turns rows into units, [plane][column]
    __device__ __forceinline__ void arrange(u32x2 (&unit)[NH][8]) {
        if constexpr (!WHOLE)
            if (late != 0) {
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    if (t >= late_from) {
                        unsigned __int128 v;
                        __builtin_memcpy(&v, &pre[t], 16);
                        v >>= 16 * late;
                        __builtin_memcpy(&pre[t], &v, 16);
                    }
            }
#pragma unroll
        for (int p = 0; p < NH; ++p)
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int k = 0; k < 2; ++k) unit[p][q][k] = row_pair(pre[4 * p + 2 * k][q >> 1], pre[4 * p + 2 * k + 1][q >> 1], q & 1);
    }
};
template <int NH> __device__ __forceinline__ void put_units(uint8_t* smem, const u32x2 (&unit)[NH][8], int tid) {
#pragma unroll
    for (int p = 0; p < NH; ++p)
#pragma unroll
        for (int q = 0; q < 8; ++q)                                   // local column 8 tid + q
            *reinterpret_cast<u32x2*>(smem + p * kPlaneBytes + (q * (kChunk / 8) + tid) * 8) = unit[p][q];
}

template <int CTRL> __device__ __forceinline__ float quad_lane(float x) {   // x of lane CTRL of this lane's four
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL * 0x55, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ uint32_t quad_lane(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL * 0x55, 0xF, 0xF, true);
}

// What a wave does in one chunk, with its first steps in registers.
struct WaveChunk {
    const u32x4* ahead;                                               // this lane's place kStepsAhead steps further on
    int steps;
    uint64_t len_lo, len_hi;                                          // steps of each of its tiles, 16 bits each
    u32x4 col_lo, col_hi;                                             // virtual columns of lists lane / 4 and 16 + lane / 4 of each tile, 16 bits each
    u32x4 ring[kStepsAhead];
    __device__ __forceinline__ void look_up(const uint8_t* plan, PlanHeaderPtr H, int c, int wave, int lane) {
        const auto* seg = as_const<uint64_t>(plan + H->off_m_seg) + ((size_t)c * kWavesMM + wave) * (sizeof(TileSeg) / 8);
        const u32x4* cols = reinterpret_cast<const u32x4*>(plan + H->off_m_cols) + (((size_t)c * kWavesMM + wave) * kSetCols + (lane >> 2)) * (kWaveTiles / 4);
        const uint64_t where = seg[0];
        len_lo = seg[1]; len_hi = seg[2];
        steps = (int)(where >> 32);
        const u32x4* at = reinterpret_cast<const u32x4*>(plan + H->off_m_steps) + (size_t)(uint32_t)where * kWave + lane;
#pragma unroll
        for (int q = 0; q < kStepsAhead; ++q) ring[q] = at[q * kWave];
        col_lo = cols[0]; col_hi = cols[1];
        ahead = at + kStepsAhead * kWave;
    }
    __device__ __forceinline__ int length(int t) const {              // (uniform)
        static_assert(kWaveTiles == 8, "two words");
        return t < kWaveTiles ? (int)(((t < 4 ? len_lo : len_hi) >> (16 * (t & 3))) & 0xFFFF) : 0;
    }
    __device__ __forceinline__ uint32_t columns(int t) const {
        const u32x4 x = t & 4 ? col_hi : col_lo;
        const uint32_t a = t & 1 ? x.y : x.x, b = t & 1 ? x.w : x.z;
        return t & 2 ? b : a;
    }
};

// Piece x (rows x, x + 4, ...) of a virtual column's sums, in LDS: the four pieces side by side, rotated so that the lanes of a
// wave that read the same piece of neighbouring columns meet all banks.
template <int R> __device__ __forceinline__ uint8_t* piece_of(uint8_t* sums, uint32_t v, uint32_t x) {
    return sums + v * (R * 4) + ((x + v / (256 / (R * 4))) & 3) * R;
}

// The sum of a list from the sums over the parts of its values, with the other sign: an FMA that subtracts is not written onto its addend, and as one
// that adds it kept the registers beside it from being used (the 16-row form spilled 16 of them, 50 us more on seven matrices of a 6.7B-style layer;
// ldexp and an addition instead: 1 % of a compress call).
__device__ __forceinline__ float minus_sum_of_parts(float first, float second, float third) {
    const float rest = fmaf(third, 1.0f / (1 << (kPartShift[2] - kPartShift[1])), second);
    return fmaf(rest, -1.0f / (1 << kPartShift[1]), -first);
}

// A wave's tiles of one staged chunk.
template <int NP>
__device__ __forceinline__ void walk_tiles(WaveChunk& w, uint8_t* sums, bool first_chunk, int mytiles, int lane) {
    constexpr int R = kRowsMM<NP>;
    typedef float Piece __attribute__((ext_vector_type(NP)));
    const int part = lane & 3;
    f32x4 D[2][NP];                                                   // [set of 16 lists][plane]
    int t = 0;
    // The tile's sums join those of the chunks before.  Lane q of a 4-lane group has the sums over the three parts of the values for row q of each plane, in three
    // registers (the fourth holds what the offsets gave).  With G as the A operand the parts would lie in three lanes, and took 16 more products a set to be brought
    // together: seven matrices of a 6.7B layer 403 -> 393 us, 4096 x 16384, skewed columns, 76.7 -> 73.3, 4096 x 4096, r = 2048, 98.1 -> 94.2 (steps and compress calls).
    Piece* dst[2];
    Piece before[2];                                                  // asked for when the tile begins
    auto begin = [&]() {
        const s16x4 none = {0, 0, 0, 0};
        const uint32_t cols = w.columns(t);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int p = 0; p < NP; ++p) D[h][p] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(none, none, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);   // (one instruction, not four)
            dst[h] = reinterpret_cast<Piece*>(piece_of<R>(sums, h ? cols >> 16 : cols & 0xFFFFu, (uint32_t)part));
            before[h] = Piece(0.0f);
        }
        if (!first_chunk) { before[0] = *dst[0]; before[1] = *dst[1]; }
    };
    auto flush = [&]() {
        Piece minus[2];
        float odd = 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                minus[h][p] = minus_sum_of_parts(D[h][p][0], D[h][p][1], D[h][p][2]);
                odd += fabsf(minus[h][p]);
            }
        // An infinity in G meets zeros among the lower parts: where the sum is no number the first part alone says what becomes of it.  (Nothing says
        // it for values below 2^-133, whose first part is zero: an infinity times one of them is NaN.)  An infinite sum stays one: the first part may
        // be finite where the value's product is not.
        if (__builtin_expect(__any(!(odd < __builtin_inff())), 0)) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int p = 0; p < NP; ++p) minus[h][p] = minus[h][p] == minus[h][p] ? minus[h][p] : -D[h][p][0];
        }
        *dst[0] = before[0] - minus[0];
        *dst[1] = before[1] - minus[1];
        ++t;
    };
    const uint32_t pick = (part & 1 ? 0x0C0C0302u : 0x0C0C0100u) + (part & 2 ? 0x0404u : 0u);   // bytes of this lane's offset among the four
    // The gathers of a step are asked for before the products of the step before; a slot is free, and takes the step kStepsAhead further
    // on, when its values have been used.  The barriers keep the compiler from waiting for each gather by itself and from giving
    // the refills registers of their own, which a loop would have to move.
    s16x4 g[2][2][NP];
    auto gather = [&](int k) {
        uint32_t off[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) off[h] = __builtin_amdgcn_perm(quad_lane<3>(w.ring[k][2 * h + 1]), quad_lane<3>(w.ring[k][2 * h]), pick);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            LSP_LDS_AS uint8_t* src = (LSP_LDS_AS uint8_t*)(uintptr_t)off[h];   // (the planes start where the LDS starts)
#pragma unroll
            for (int p = 0; p < NP; ++p) g[k & 1][h][p] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LSP_LDS_AS s16x4*)(src + p * kPlaneBytes));
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F | (2 * NP << 8));           // lgkmcnt(2 NP): what was asked for before is there
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int k, bool refill, uint32_t ends) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x2 x = {w.ring[k][2 * h], w.ring[k][2 * h + 1]};
            s16x4 v;
            __builtin_memcpy(&v, &x, 8);
#pragma unroll
            for (int p = 0; p < NP; ++p) D[h][p] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, g[k & 1][h][p], D[h][p], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (refill) w.ring[k] = w.ahead[k * kWave];
        if (__builtin_expect((ends >> k) & 1, 0)) {
            flush();
            begin();
        }
    };
    // which of the next kStepsAhead steps are the last of their tiles
    int end = w.length(0), coming = 1;                                // the present tile's last step from here on, counted from 1
    auto tile_ends = [&]() {
        uint32_t ends = 0;
        while (end <= kStepsAhead) {
            ends |= 1u << (end - 1);
            const int len = w.length(coming++);
            if (len == 0) { end = 1 << 30; break; }
            end += len;
        }
        end -= kStepsAhead;
        return ends;
    };
    begin();
    if (w.steps > 0) gather(0);
    for (int n = (w.steps - 1) / kStepsAhead; n > 0; --n) {
        const uint32_t ends = tile_ends();
#pragma unroll
        for (int k = 0; k < kStepsAhead; ++k) {
            gather((k + 1) % kStepsAhead);
            multiply(k, true, ends);
        }
        w.ahead += kStepsAhead * kWave;
    }
    const int rest = w.steps > 0 ? (w.steps - 1) % kStepsAhead + 1 : 0;
    const uint32_t ends = rest > 0 ? tile_ends() : 0;
#pragma unroll
    for (int k = 0; k < kStepsAhead; ++k) {
        if (k + 1 < rest) gather((k + 1) % kStepsAhead);
        if (k < rest) multiply(k, false, ends);
    }
    if (first_chunk)
        while (t < mytiles) { flush(); begin(); }                     // tiles without an entry in this chunk: their sums start at zero
}

// The sums of a block go out: a thread has one of the four pieces of a column at a time.
template <int R>
__device__ __forceinline__ void store_sums(uint8_t* sums, const uint8_t* plan, PlanHeaderPtr H, float* __restrict__ T, int64_t i0, int m, int r, int tid) {
    constexpr int Q = R / 4;
    typedef float Piece __attribute__((ext_vector_type(Q)));
    const bool shared = H->q_any_shared != 0;
    const auto* vcol = as_const<uint16_t>(plan + H->off_q_vcol);
    const auto* vcnt = as_const<uint16_t>(plan + H->off_q_vcnt);
    const int x = tid / (kWalkers / 4), V = H->nvcols;
    for (int v = tid % (kWalkers / 4); v < V; v += kWalkers / 4) {
        Piece out = *reinterpret_cast<const Piece*>(piece_of<R>(sums, v, x));
        int b = v;
        if (shared) {                                                 // the owners of a column sit side by side: added in their order
            const int owners = vcnt[v];
            if (owners == 0) continue;
            b = vcol[v] & 0x7FFF;
            for (int o = 1; o < owners; ++o) out += *reinterpret_cast<const Piece*>(piece_of<R>(sums, v + o, x));
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (i0 + 4 * q + x < m) T[(i0 + 4 * q + x) * (int64_t)r + b] = out[q];
    }
}

// The problem of a row block, read from the kernel's arguments with a run-time index (scalar loads): a workgroup looks several
// up, and group_pick's selects over all problems would keep the whole group in registers.
struct RowBlocks { const void* G; const uint8_t* plan; float* T; float* S; int32_t m, n, block, blocks; };
__device__ __forceinline__ RowBlocks problem_of(int block) {
    const auto* g = (const LSP_CONST_AS CompressGroup*)__builtin_amdgcn_kernarg_segment_ptr();   // the kernel's first argument
    int p = 0;
    while (p + 1 < g->count && block >= g->first_gq[p + 1]) ++p;
    return RowBlocks{g->G[p], g->plan[p], g->T[p], g->S[p], g->m[p], g->n[p], block - g->first_gq[p], g->first_gq[p + 1] - g->first_gq[p]};
}

// The row blocks of a workgroup, one after the other, as both kinds of waves see them; they meet at the same barriers.
// kind: blocks whose sums fit the LDS (whole), or the others.
template <int NP, bool HALVES> struct BlockWalk {
    int block;                                                        // past the last one: no more
    RowBlocks pr;
    PlanHeaderPtr H;
    int nchunks;
    // the first of the blocks from `block` on that is of this kind; visit: called for every block passed by or taken
    template <typename Visit> __device__ __forceinline__ void find(int from, int blocks, int r, int d, Visit&& visit) {
        for (block = from; block < blocks; block += gridDim.x) {
            pr = problem_of(block);
            H = as_const<PlanHeader>(pr.plan);
            const bool planned = plan_matches(H, pr.m, pr.n, r, d, true);
            visit(pr, H, planned);
            if (!planned) continue;
            nchunks = H->nchunks;
            const bool fits = (H->nvcols + kTileCols - 1) / kTileCols * kTileCols * (kRowsMM<NP> * 4) <= kLdsMM - kTileBase<NP>;
            if (fits != HALVES) return;
        }
    }
};

// Waves that fetch: chunks of G are on their way while the other waves walk the present one.
// They are waves of their own because loads return in order: behind a load of G from HBM the walkers' loads of the plan would wait.
// The first half of the rows of a chunk is asked for a chunk earlier than the second, so that loads are in flight at any time.
template <int NP, bool WHOLE>
__device__ __forceinline__ void fetch_blocks(uint8_t* smem, int blocks, int r, int d, int tid) {
    constexpr int R = kRowsMM<NP>, NH = NP / 2;
    auto none = [](const RowBlocks&, PlanHeaderPtr, bool) {};
    BlockWalk<NP, false> w;
    int c = 0;
    auto advance = [&]() {
        if (++c >= w.nchunks) { c = 0; w.find(w.block + gridDim.x, blocks, r, d, none); }
    };
    RowStager<NH, WHOLE> lo, hi;
    u32x2 ulo[NH][8], uhi[NH][8];
    const RowBlocks start = problem_of(blockIdx.x);                   // nearly always the first: its rows are asked for before its plan is looked at
    lo.fetch(static_cast<const uint16_t*>(start.G), (int64_t)start.block * R, start.m, start.n, 0, tid);
    hi.fetch(static_cast<const uint16_t*>(start.G), (int64_t)start.block * R + R / 2, start.m, start.n, 0, tid);
    w.find(blockIdx.x, blocks, r, d, none);
    bool have = w.block < blocks;
    if (have) {
        if (w.block != (int)blockIdx.x) {
            lo.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R, w.pr.m, w.pr.n, c, tid);
            hi.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R + R / 2, w.pr.m, w.pr.n, c, tid);
        }
        lo.arrange(ulo); hi.arrange(uhi);
        advance();
        if (w.block < blocks) lo.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R, w.pr.m, w.pr.n, c, tid);
    }
    while (have) {
        put_units<NH>(smem, ulo, tid);
        put_units<NH>(smem + NH * kPlaneBytes, uhi, tid);
        __syncthreads();                                              // staged
        have = w.block < blocks;
        if (have) {
            hi.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R + R / 2, w.pr.m, w.pr.n, c, tid);
            lo.arrange(ulo);
            advance();
            hi.arrange(uhi);
            if (w.block < blocks) lo.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R, w.pr.m, w.pr.n, c, tid);
        }
        __syncthreads();                                              // no longer read
    }
    if constexpr (NP == 4) {
        BlockWalk<NP, true> h;
        for (h.find(blockIdx.x, blocks, r, d, none); h.block < blocks; h.find(h.block + gridDim.x, blocks, r, d, none))
            for (int part = 0; part < 2; ++part)
                for (int k = 0; k < h.nchunks; ++k) {
                    lo.fetch(static_cast<const uint16_t*>(h.pr.G), (int64_t)h.pr.block * R + part * (R / 2), h.pr.m, h.pr.n, k, tid);
                    lo.arrange(ulo);
                    put_units<NH>(smem, ulo, tid);
                    __syncthreads();
                    __syncthreads();
                }
    }
}

__device__ __forceinline__ int tiles_of_wave(int V, int wave) {
    int count = 0;
#pragma unroll
    for (int i = 0; i < kWaveTiles; ++i) count += tile_of_wave(i, wave) * kTileCols < V ? 1 : 0;
    return count;
}

// Waves that walk the lists.
template <int NP>
__device__ __forceinline__ void walk_blocks(uint8_t* sums, int blocks, int r, int d, int tid) {
    constexpr int R = kRowsMM<NP>;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto clear_s = [&](const RowBlocks& pr, PlanHeaderPtr H, bool planned) {
        if (!planned) {                                               // not a plan for this problem
            fill_s(pr.S, __builtin_nanf(""), r, pr.block, pr.blocks, tid, kWalkers);
        } else if (H->p_any_split) fill_s(pr.S, 0.0f, r, pr.block, pr.blocks, tid, kWalkers);
    };
    WaveChunk t;
    BlockWalk<NP, false> w, next;
    w.find(blockIdx.x, blocks, r, d, clear_s);
    if (w.block < blocks) t.look_up(w.pr.plan, w.H, 0, wave, lane);
    while (w.block < blocks) {
        const int mytiles = tiles_of_wave(w.H->nvcols, wave);
        for (int c = 0; c < w.nchunks; ++c) {
            const bool last = c + 1 == w.nchunks;
            if (last) next.find(w.block + gridDim.x, blocks, r, d, clear_s);
            __syncthreads();                                          // the chunk is staged
            walk_tiles<NP>(t, sums, c == 0, mytiles, lane);
            if (!last) t.look_up(w.pr.plan, w.H, c + 1, wave, lane);  // in flight while the next chunk is staged
            else if (next.block < blocks) t.look_up(next.pr.plan, next.H, 0, wave, lane);
            __syncthreads();                                          // all sums are there
        }
        store_sums<R>(sums, w.pr.plan, w.H, w.pr.T, (int64_t)w.pr.block * R, w.pr.m, r, tid);
        w = next;
    }
    if constexpr (NP == 4) {                                          // more sums than the LDS has room for: 8 rows, then 8 rows
        auto none = [](const RowBlocks&, PlanHeaderPtr, bool) {};
        BlockWalk<NP, true> h;
        for (h.find(blockIdx.x, blocks, r, d, none); h.block < blocks; h.find(h.block + gridDim.x, blocks, r, d, none))
            for (int part = 0; part < 2; ++part) {
                for (int c = 0; c < h.nchunks; ++c) {
                    t.look_up(h.pr.plan, h.H, c, wave, lane);
                    __syncthreads();
                    walk_tiles<2>(t, sums, c == 0, tiles_of_wave(h.H->nvcols, wave), lane);
                    __syncthreads();
                }
                store_sums<R / 2>(sums, h.pr.plan, h.H, h.pr.T, (int64_t)h.pr.block * R + part * (R / 2), h.pr.m, r, tid);
            }
    }
}

template <int NP, bool WHOLE>
__global__ __launch_bounds__(kThreadsMM) void k_compress_mm(const CompressGroup grp, int r, int d, int blocks) {
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x;
    if (tid < NP) *reinterpret_cast<u32x2*>(smem + tid * kPlaneBytes + kChunk * 8) = u32x2{0, 0};
    if (__builtin_amdgcn_readfirstlane(tid) >= kWalkers) fetch_blocks<NP, WHOLE>(smem, blocks, r, d, tid - kWalkers);
    else walk_blocks<NP>(smem + kTileBase<NP>, blocks, r, d, tid);
}

template <int NP> static hipError_t launch_mm_rows(CompressGroup& g, int32_t r, int32_t d, hipStream_t st) {
    constexpr int R = kRowsMM<NP>;
    constexpr size_t lds = kLdsMM;
    bool whole = true;
    g.first_gq[0] = 0;
    for (int p = 0; p < g.count; ++p) {
        whole = whole && g.n[p] % 8 == 0;
        g.blocks_gq[p] = 1;
        g.first_gq[p + 1] = g.first_gq[p] + (g.m[p] + R - 1) / R;
    }
    const int blocks = g.first_gq[g.count];
    const dim3 grid((unsigned)std::min(blocks, kResidentMM));
    hipError_t e;
    if (whole) {
        if ((e = allow_dynamic_lds<k_compress_mm<NP, true>>(lds)) != hipSuccess) return e;
        hipLaunchKernelGGL((k_compress_mm<NP, true>), grid, dim3(kThreadsMM), lds, st, g, (int)r, (int)d, blocks);
    } else {
        if ((e = allow_dynamic_lds<k_compress_mm<NP, false>>(lds)) != hipSuccess) return e;
        hipLaunchKernelGGL((k_compress_mm<NP, false>), grid, dim3(kThreadsMM), lds, st, g, (int)r, (int)d, blocks);
    }
    return hipGetLastError();
}

// Blocks of 16 rows read the plan half as often as blocks of 8 and share each value between twice the rows (4096 x 4096, d = 8, with
// kernel B: r = 512 28.2 us, with 8 rows 29.6; r = 1024 34.6 and 38.6; seven matrices of a 6.7B layer 216 and 265).  8 rows are better
//   where there is at most one block of 8 for a CU, so that the blocks of 16 would leave CUs idle (2048 rows 18.4 us, with 16 22.8; 3001 rows 22.2
//   and 20.9);
//   where they take three rounds of one for every CU and the blocks of 16 two, the last of them little more than half full or less: 4097 to 6144 rows (us with 8
//   and with 16 rows: 5120 x 5120, r = 512, d = 8 45.5 and 47.2, zipf 61.8 and 64.1; r = 1024, d = 16 75.0 and 79.6; 6144 x 4096, r = 256, d = 16 56.7 and 60.9, r = 1024,
//   d = 4 41.3 and 45.0; in the mean of 36 such calls 3 % less, with zipf columns even: 4200 x 2048, r = 1024, d = 8 61.8 and 56.8); with five rounds and three
//   they are not (9000 x 2048, r = 512, d = 8 41.4 and 40.5);
//   and beyond r = 1024, where the sums of 16 rows do not fit the LDS (r = 1536 50.1 and 52.6, r = 2048 57.0 and 60.6).
static bool narrow_blocks(const CompressGroup& g, int32_t r) {
    int64_t of8 = 0, of16 = 0;
    for (int p = 0; p < g.count; ++p) {
        of8 += (g.m[p] + 7) / 8;
        of16 += (g.m[p] + 15) / 16;
    }
    const auto rounds = [](int64_t blocks) { return (blocks + kResidentMM - 1) / kResidentMM; };
    return r > 1024 || rounds(of8) == 1 || (rounds(of8) == 3 && rounds(of16) == 2);
}

// Every bf16 call with a kept plan comes here, whatever its rows: the sums of a row do not depend on the blocks it is in, so a matrix has the same
// result alone and in any group, which a second kernel with sums in another order would end.  Where the last round is nearly empty, k_compress_gq with
// its finer grain (8 rows, two workgroups a CU) is up to 16 % faster if the lists are long and even, and 4 to 30 % slower otherwise: 7 % slower in the mean of
// 40 calls with random sizes, counts and columns whose last round is less than 80 % full (us with kernel B, here and there; single matrices, uniform and zipf columns):
//   5120 x 5120  r = 512, d = 8 45.5 and 43.5, 61.8 and 70.9; r = 512, d = 4 37.5 and 36.9, 52.5 and 61.3; r = 1024, d = 8 57.7 and 57.1, 88.5 and 99.0
//   5120 x 13824 r = 512, d = 8 90.1 and 79.2, 111 and 120; r = 1024, d = 8 108 and 104, 151 and 151; d = 16 147 and 143, 191 and 199
//   6144 x 4096  r = 256, d = 4 28.6 and 34.2, 38.5 and 48.4; d = 16 56.7 and 52.5, 76.7 and 68.6; r = 512, d = 8 40.3 and 39.5, 56.1 and 65.4
//   9000 x 2048  r = 512, d = 8 40.5 and 39.9, 60.6 and 73.2; seven matrices of 5120 and 13824 rows and columns 292 and 319
// Beyond r = 1024, where the lists are a few steps long, it is on a par with k_compress_gq, and behind it for short lists on 4096 and 8192 rows: r = 2048,
//   4096 x 4096  d = 4 53.3 and 49.9, d = 8 58.8 and 55.4, d = 16 73.2 and 71.2; 5120 x 5120 77.0 and 80.1, 87.5 and 88.1, 109.4 and 113.3
//   4096 x 16384 110 and 103, 120 and 114, 153 and 156; r = 1536, d = 8 4096 x 4096 47.9 and 50.9, 8192 x 8192 128 and 133
hipError_t launch_mm_bf16(CompressGroup& g, int32_t r, int32_t d, hipStream_t st) {
    return narrow_blocks(g, r) ? launch_mm_rows<2>(g, r, d, st) : launch_mm_rows<4>(g, r, d, st);
}

}  // namespace lsp
