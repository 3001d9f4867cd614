// Compress, kernel A for bf16: T = G Q on the matrix cores.  See compress.hip for the path as a whole.
//
// A column of T is a sum over a list of (column of G, value), and the lists share nothing, so this is no matrix product.  But
// v_mfma_f32_4x4x4_16b_bf16 is 16 independent products [4 x 4] [4 x 4], and each can serve a list: its A operand is four values from the list
// as three bf16 parts that add up, each times its power of two, to the fp32 value exactly (in three of its rows), its B operand their four columns
// of G (4 rows; gathered by transposing LDS reads, which hand a lane one row's four values).  So a product of 16 bits by 24 is taken exactly, and
// the three sums, which a lane has for its row side by side, are added at the end: the error against 64 bits is 0.3 to 0.6 of that of a chain of fp32 FMAs.  An instruction does
// 4 rows x 64 entries; the vector ALUs took 8 widenings and FMAs for 8 rows x 64 entries.
//
// One workgroup a CU, persistent: 8 waves walk the lists (the plan's tiles: lsp_internal.h), 4 fetch and stage the next chunk of G and look up what the
// walkers have to know of it.  A block's 16 rows of a column lie side by side in LDS, 32 bytes: the values of a list are given to four blocks of the
// instruction (cbsz, abid), each with four of the rows, so that 16 lanes gather from four units instead of 16, and meet on a bank less often (5.1 cycles a
// read; from planes of 8 bytes a column 7.1, without conflicts 2.5).
// What bounds it: with long lists (r = 512, d = 8, 11008 x 4096) no single thing: some 10000 cycles a chunk, of them 1100 of staging, with the walkers idle, 7700 to 9000 of walking (the two
// walking waves of a SIMD do not keep step), of it the LDS 5900, 1300 for two or three tiles' ends, some 40 instructions a step and wave; storing T 1250 a block; the clock is down from
// 2.4 to 1.95 GHz.  With short ones (4096 x 16384, r = 256, d = 2) the reads of G, at about 4.6 TB/s.
// (us, with kernel B: planes of 8 bytes -> 32-byte units, chunks that begin with their steps in registers, and notes -> loads that stay in flight, other chunks first, two chunks in LDS,
// steps ahead by the length of the lists: 4096 x 4096, r = 512, d = 8 27.4 -> 26.1 -> 25.6; 4096 x 16384 62.2 -> 58.1 -> 53.4; r = 256, d = 2 43.4 -> 46.5 -> 34.0, zipf 49.3 -> 54.2 -> 42.2;
// 4096 x 4096, r = 2048 59.0 -> 49.0 -> 48.2.)
// 512 threads and 8 rows, twice a CU, or 12 walking waves and narrower tiles were 2 to 8 % slower; LDS atomics for the sums twice as slow.
#include <algorithm>

#include "compress_common.h"

namespace lsp {

typedef short s16x4 __attribute__((ext_vector_type(4)));
#define LSP_LDS_AS __attribute__((address_space(3)))

constexpr int kLdsMM = 160 * 1024;
constexpr int kWalkers = kWavesMM * kWave;                            // threads that walk the lists
constexpr int kFetchers = kChunk / 8;                                 // threads that fetch and stage G
constexpr int kThreadsMM = kWalkers + kFetchers;
constexpr int kResidentMM = 256;                                      // one workgroup a CU

// A block is 4 NP rows.  In LDS a column of a chunk is a unit of 8 NP bytes (its rows side by side); a unit behind the last one stays zero.
template <int NP> constexpr int kRowsMM = 4 * NP;
template <int NP> constexpr int kUnitBytes = 8 * NP;
template <int NP> constexpr int kNoteBase = (kChunk + 1) * kUnitBytes<NP>;       // LDS offset of the notes on the present chunk and the next
// What the fetching waves, which have the time to look it up, tell the walking ones about a chunk: found out by the walkers themselves, one dependent scalar load
// after the other, it took them 2000 cycles a block and 300 a chunk (of some 11000).
struct ChunkNote {
    uint32_t cols[kWavesMM][kSetCols][kWaveTiles];                    // as in the plan (off_m_cols)
    TileSeg seg[kWavesMM];                                            // as in the plan (off_m_seg)
    uint64_t steps[2][kWavesMM];                                      // where each wave's steps lie: of the chunk after it, and its own
    float* T;                                                         // the block's rows
    const uint8_t* plan;
    uint32_t vcol, vcnt;                                              // offsets of these tables in the plan
    int32_t rows, pad0;                                               // rows of the block inside the matrix
    int32_t nvcols;                                                   // virtual columns
    uint32_t flags, pad1[2];
};
constexpr uint32_t kFirstChunk = 1, kLastChunk = 2, kMoreChunks = 4, kSharedColumns = 8, kHalvesFollow = 16;
static_assert(sizeof(ChunkNote) % 16 == 0 && sizeof(TileSeg) == 32, "read in pieces of 16 bytes");
template <int NP> constexpr int kSecondBase = kNoteBase<NP> + 2 * (int)sizeof(ChunkNote);   // ... of a second chunk where there is room for two
template <int NP> __host__ __device__ constexpr int sums_base(bool two) { return kSecondBase<NP> + (two ? kNoteBase<NP> : 0); }   // ... and of the sums
// Floats from a row of the sums to the next: 16 rows of a column lie in 16 different banks, and four columns are 16 bytes.
__device__ __forceinline__ int sums_stride(int nvcols) { return (nvcols + kTileCols - 1) / kTileCols * kTileCols + 4; }

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
template <int NP> __device__ __forceinline__ void zero_unit(uint8_t* smem, int tid) {
    if (tid < NP) *reinterpret_cast<u32x2*>(smem + kChunk * kUnitBytes<NP> + tid * 8) = u32x2{0, 0};
}
// rows 4 NH half .. of a block's NP planes
template <int NP, int NH> __device__ __forceinline__ void put_units(uint8_t* smem, const u32x2 (&unit)[NH][8], int half, int tid) {
    static_assert(NH == 1 || NH == 2, "8 or 16 bytes");
#pragma unroll
    for (int q = 0; q < 8; ++q) {                                     // local column 8 tid + q
        uint8_t* dst = smem + (q * (kChunk / 8) + tid) * kUnitBytes<NP> + half * (NH * 8);
        if constexpr (NH == 2) *reinterpret_cast<u32x4*>(dst) = u32x4{unit[0][q].x, unit[0][q].y, unit[1][q].x, unit[1][q].y};
        else *reinterpret_cast<u32x2*>(dst) = unit[0][q];
    }
}

// All rows of a block, n % 8 == 0: four lanes write the first halves of their units while the next four write the second ones, so that a write falls on more banks (with
// kernel B: four matrices 4096 x 11008, r = 512, d = 8 158.8 -> 157.7 us; 4096 x 16384, r = 256, d = 2 48.6 -> 48.15; where pieces are loose the selects spill: 19.8 -> 20.5).
template <int NP, int NH> __device__ __forceinline__ void put_block(uint8_t* smem, const u32x2 (&lo)[NH][8], const u32x2 (&hi)[NH][8], int tid) {
    static_assert(NH == 2, "units of 32 bytes");
    const bool swap = (tid >> 2 & 1) != 0;
    uint8_t* const first = smem + tid * kUnitBytes<NP> + (swap ? 16 : 0);
    uint8_t* const second = smem + tid * kUnitBytes<NP> + (swap ? 0 : 16);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const u32x4 l = {lo[0][q].x, lo[0][q].y, lo[1][q].x, lo[1][q].y}, h = {hi[0][q].x, hi[0][q].y, hi[1][q].x, hi[1][q].y};
        *reinterpret_cast<u32x4*>(first + q * (kChunk / 8) * kUnitBytes<NP>) = swap ? h : l;
        *reinterpret_cast<u32x4*>(second + q * (kChunk / 8) * kUnitBytes<NP>) = swap ? l : h;
    }
}

template <int CTRL> __device__ __forceinline__ uint32_t quad_lane(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL * 0x55, 0xF, 0xF, true);
}

// One of the two offsets in a word, times SCALE, plus add: one instruction.
template <int SCALE, bool HIGH> __device__ __forceinline__ uint32_t unit_at(uint32_t two, uint32_t add) {
    uint32_t at;
    if constexpr (HIGH) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(at) : "v"(two), "n"(SCALE), "v"(add));
    else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(two), "n"(SCALE), "v"(add));
    return at;
}

// Of the 16 values x that the 4-lane groups hold (one each: lists 0 .. 15), that of list NP (lane / (4 NP)) + a: list a of the NP lists
// that share a lane's 4 NP rows.
template <int NP, int A> __device__ __forceinline__ uint32_t list_of(uint32_t x) {
    if constexpr (NP == 4) return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x150 + 4 * A, 0xF, 0xF, true);          // row_newbcast
    else if constexpr (A == 0) return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x114, 0xF, 0xA, false);   // row_shr:4, odd groups
    else return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x104, 0xF, 0x5, false);                         // row_shl:4, even groups
}

// The sum of a list from the sums over the parts of its values, with the other sign: an FMA that subtracts is not written onto its addend, and as one
// that adds it kept the registers beside it from being used (the 16-row form spilled 16 of them, 50 us more on seven matrices of a 6.7B-style layer;
// ldexp and an addition instead: 1 % of a compress call).
__device__ __forceinline__ float minus_sum_of_parts(float first, float second, float third) {
    const float rest = fmaf(third, 1.0f / (1 << (kPartShift[2] - kPartShift[1])), second);
    return fmaf(rest, -1.0f / (1 << kPartShift[1]), -first);
}

// The sums of a block go out: a wave a row at a time, or, where columns have several owners (which lie side by side, and are added in their order), a thread a quarter of a column.
template <int R>
__device__ __forceinline__ void store_sums(const float* sums, int stride, float LSP_GLOBAL_AS* T, const uint16_t LSP_GLOBAL_AS* vcol, const uint16_t LSP_GLOBAL_AS* vcnt,
                                           bool shared, int V, int rows, int r, int tid) {
    if (shared) {
        constexpr int Q = R / 4;
        const int row0 = tid / (kWalkers / 4) * Q;
        sums += row0 * stride;
        T += row0 * (int64_t)r;
        for (int v = tid % (kWalkers / 4); v < V; v += kWalkers / 4) {
            const int owners = vcnt[v], b = vcol[v] & 0x7FFF;
            if (owners == 0) continue;
            float out[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) out[q] = sums[q * stride + v];
#pragma unroll 4
            for (int o = 1; o < owners; ++o)
#pragma unroll
                for (int q = 0; q < Q; ++q) out[q] += sums[q * stride + v + o];
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (row0 + q < rows) T[q * (int64_t)r + b] = out[q];
        }
        return;
    }
    const int lane = tid & (kWave - 1);
    for (int row = tid / kWave; row < R && row < rows; row += kWavesMM) {
        const float* src = sums + row * stride;
        float LSP_GLOBAL_AS* dst = T + row * (int64_t)r;
        if ((r & 3) == 0) {
            for (int v = lane * 4; v < V; v += kWave * 4) *(f32x4 LSP_GLOBAL_AS*)(dst + v) = *reinterpret_cast<const f32x4*>(src + v);
        } else {
            for (int v = lane; v < V; v += kWave) dst[v] = src[v];
        }
    }
}

// The problem of a row block.
struct RowBlocks { const void* G; const uint8_t* plan; float* T; float* S; int32_t m, n, block, blocks; };
__device__ __forceinline__ RowBlocks row_blocks_of(int block) {
    const auto* g = group_args<CompressGroup>();
    const CompressProblem p = pick_problem(g, g->first_gq, block).p;
    return RowBlocks{p.G, p.plan, p.T, p.S, p.m, p.n, block - p.first_gq, p.wgs_gq};
}

__device__ __forceinline__ bool sums_fit(int nvcols, int rows, int base) { return sums_stride(nvcols) * rows * 4 <= kLdsMM - base; }

// Whether the LDS has room for two chunks beside the sums of every matrix of the call (16 rows: up to 352 virtual columns; 8 rows: always).  nvcols: those of one of them.
template <int NP> __device__ __forceinline__ bool two_chunks(int nvcols) {
    static_assert((kMaxSlots * kThreadsGQ + 4) * kRowsMM<2> * 4 <= kLdsMM - sums_base<2>(true), "8 rows");
    if constexpr (NP == 2) return true;
    const auto* g = group_args<CompressGroup>();
    uint32_t most = (uint32_t)nvcols;
    if (g->count > 1) {                                               // (of all of them the pointers, then the numbers)
        words16 lo = scalar_load<words16>(&g->plans[0]), hi = scalar_load<words16>(&g->plans[kMaxGroup / 2]);
        arrived(lo, hi);
        uint32_t v[kMaxGroup];
        auto nvcols_of = [](uint32_t a, uint32_t b) { return (uint32_t)((PlanHeaderPtr)((uint64_t)b << 32 | a))->nvcols; };
#pragma unroll
        for (int p = 0; p < kMaxGroup / 2; ++p) {
            v[p] = nvcols_of(lo[2 * p], lo[2 * p + 1]);
            v[kMaxGroup / 2 + p] = nvcols_of(hi[2 * p], hi[2 * p + 1]);
        }
#pragma unroll
        for (int p = 0; p < kMaxGroup; ++p) arrived(v[p]);
#pragma unroll
        for (int p = 0; p < kMaxGroup; ++p) most = v[p] > most ? v[p] : most;
    }
    return most <= (uint32_t)(kMaxSlots * kThreadsGQ) && sums_fit((int)most, kRowsMM<NP>, sums_base<NP>(true));
}

// Blocks begin with different chunks, and go around: rows a power of two apart would have all workgroups on the same few memory channels at a time (4096 x 16384, r = 256, d = 2
// 46.1 -> 39.5 us, r = 512, d = 8 58.4 -> 55.2; 8192 x 8192, r = 512, d = 8 62.6 -> 60.5; 3001 x 11008, r = 512, d = 4 32.9 -> 32.1).  With three chunks it does nothing, and where rows
// are few, workgroups that read the same part of the plan at a time are worth more (1106 x 6144, r = 512, d = 8 18.2 us, 18.7 with it; 2048 x 16384 36.9 and 35.2).
// Which one is a matter of the row and its matrix alone, so that the sums of a row do not depend on the blocks it is in.  (Golden-ratio steps: neighbouring blocks of 16 rows spread evenly.)
__device__ __forceinline__ int chunk_at(int k, int row0, int m, int nchunks) {
    const int at = k + (nchunks > 3 && m > 1536 ? (int)__umulhi((uint32_t)(row0 >> 4) * 0x9E3779B9u, (uint32_t)nchunks) : 0);
    return at < nchunks ? at : at - nchunks;
}

// The row blocks of a workgroup, one after the other, as both kinds of waves see them; they meet at the same barriers.
// kind: blocks whose sums fit the LDS (whole), or the others.
template <int NP, bool HALVES> struct BlockWalk {
    int block;                                                        // past the last one: no more
    bool others = false;                                              // blocks of the other kind were passed by
    RowBlocks pr;
    PlanHeaderPtr H;
    int nchunks, nvcols;
    // the first of the blocks from `block` on that is of this kind; visit: called for every block passed by or taken
    template <typename Visit> __device__ __forceinline__ void find(int from, int blocks, int r, int d, Visit&& visit) {
        for (block = from; block < blocks; block += gridDim.x) {
            pr = row_blocks_of(block);
            H = as_const<PlanHeader>(pr.plan);
            words8 head = scalar_load<words8>(H);
            uint32_t steps = H->m_total_steps;
            arrived(head, steps);
            const bool planned = same_problem(head[0], (int)head[1], (int)head[2], (int)head[3], (int)head[4], pr.m, pr.n, r, d) && steps != 0;
            visit(pr, H, planned);
            if (!planned) continue;
            nchunks = (int)head[5];
            nvcols = (int)head[7];
            if (sums_fit(nvcols, kRowsMM<NP>, sums_base<NP>(NP == 2)) != HALVES) return;
            others = true;
        }
    }
};

// Waves that fetch: chunks of G are on their way while the other waves walk the present one.
// They are waves of their own because loads return in order: behind a load of G from HBM the walkers' loads of the plan would wait.
// The first half of the rows of a chunk is asked for a chunk earlier than the second (where two chunks take turns, both), so that loads are in flight at any time.
template <int NP, bool WHOLE>
__device__ __forceinline__ void fetch_blocks(uint8_t* smem, int blocks, int r, int d, int tid) {
    constexpr int R = kRowsMM<NP>, NH = NP / 2;
    // (every block is passed by or taken here, and its part of S cleared where that is to be done)
    auto clear_s = [&](const RowBlocks& pr, PlanHeaderPtr H, bool planned) {
        if (!planned) {                                               // not a plan for this problem
            fill_s(pr.S, __builtin_nanf(""), r, pr.block, pr.blocks, tid, kFetchers);
        } else if (H->p_any_split) fill_s(pr.S, 0.0f, r, pr.block, pr.blocks, tid, kFetchers);
    };
    BlockWalk<NP, false> w;
    int c = 0;                                                        // the how manieth chunk of the block
    auto chunk = [&]() { return chunk_at(c, w.pr.block * R, w.pr.m, w.nchunks); };
    auto advance = [&]() {
        if (++c >= w.nchunks) { c = 0; w.find(w.block + gridDim.x, blocks, r, d, clear_s); }
    };
    RowStager<NH, WHOLE> lo, hi;
    u32x2 ulo[NH][8], uhi[NH][8];

    // The coming chunk's note, with the table of its columns: found out while the chunk before is walked.
    u32x4 cols, seg;                                                  // this thread's part of the tables
    uint32_t step_after = 0, step_here = 0;                           // threads 0 .. 7: a wave's first step in the chunk after, 8 .. 15: in this one
    const uint8_t *steps_here, *steps_after;
    struct { float* T; const uint8_t* plan; uint32_t vcol, vcnt, flags; int32_t rows, nvcols; } head;
    int turn = 0;
    static_assert(sizeof(ChunkNote::cols) == kFetchers * 16 && sizeof(ChunkNote::seg) == 16 * 16, "16 bytes a thread");
    auto segs = [](const RowBlocks& pr, PlanHeaderPtr H, int chunk) { return pr.plan + H->off_m_seg + (size_t)chunk * (kWavesMM * sizeof(TileSeg)); };
    auto look_up = [&](const RowBlocks& pr, PlanHeaderPtr H, int nchunks, int k, int rows_of, int row0) {
        const int chunk = chunk_at(k, row0, pr.m, nchunks);
        cols = reinterpret_cast<const u32x4*>(pr.plan + H->off_m_cols)[(size_t)chunk * kFetchers + tid];
        const uint8_t* here = segs(pr, H, chunk);
        if (tid < 16) seg = reinterpret_cast<const u32x4*>(here)[tid];
        if (tid >= kWavesMM && tid < 2 * kWavesMM) step_here = reinterpret_cast<const TileSeg*>(here)[tid - kWavesMM].first_step;
        steps_here = steps_after = pr.plan + H->off_m_steps;
        head.T = pr.T + (int64_t)row0 * r;
        head.plan = pr.plan;
        head.vcol = (uint32_t)H->off_q_vcol; head.vcnt = (uint32_t)H->off_q_vcnt;
        head.rows = pr.m - row0 < rows_of ? pr.m - row0 : rows_of;
        head.nvcols = H->nvcols;
        head.flags = (k == 0 ? kFirstChunk : 0) | (k + 1 == nchunks ? kLastChunk : 0) | (H->q_any_shared ? kSharedColumns : 0);
    };
    auto look_after = [&](const RowBlocks& pr, PlanHeaderPtr H, int chunk) {   // the chunk after the one above
        if (tid < kWavesMM) step_after = reinterpret_cast<const TileSeg*>(segs(pr, H, chunk))[tid].first_step;
        steps_after = pr.plan + H->off_m_steps;
        head.flags |= kMoreChunks;
    };
    auto put_note = [&]() {
        ChunkNote* note = reinterpret_cast<ChunkNote*>(smem + kNoteBase<NP>) + turn;
        turn ^= 1;
        reinterpret_cast<u32x4*>(note->cols)[tid] = cols;
        if (tid < 16) {
            reinterpret_cast<u32x4*>(note->seg)[tid] = seg;
            (&note->steps[0][0])[tid] = (uint64_t)(uintptr_t)((tid < kWavesMM ? steps_after : steps_here) + (size_t)(tid < kWavesMM ? step_after : step_here) * (kWave * 16));
        }
        if (tid == 0) {
            note->T = head.T; note->plan = head.plan; note->vcol = head.vcol; note->vcnt = head.vcnt;
            note->rows = head.rows; note->nvcols = head.nvcols; note->flags = head.flags;
        }
    };

    const RowBlocks start = row_blocks_of(blockIdx.x);                   // nearly always the first: its rows are asked for before its plan is looked at
    lo.fetch(static_cast<const uint16_t*>(start.G), (int64_t)start.block * R, start.m, start.n, chunk_at(0, start.block * R, start.m, (int)(((uint32_t)start.n + kChunk - 1) / kChunk)), tid);
    hi.fetch(static_cast<const uint16_t*>(start.G), (int64_t)start.block * R + R / 2, start.m, start.n, chunk_at(0, start.block * R, start.m, (int)(((uint32_t)start.n + kChunk - 1) / kChunk)), tid);
    w.find(blockIdx.x, blocks, r, d, clear_s);
    auto fetch_lo = [&]() { lo.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R, w.pr.m, w.pr.n, chunk(), tid); };
    auto fetch_hi = [&]() { hi.fetch(static_cast<const uint16_t*>(w.pr.G), (int64_t)w.pr.block * R + R / 2, w.pr.m, w.pr.n, chunk(), tid); };
    auto look_up_here = [&]() { look_up(w.pr, w.H, w.nchunks, c, R, w.pr.block * R); };
    // Arranges a half now: the compiler, which would rather do it where the units are stored, would have the next loads in other registers then, and wait for them to move them.
    auto arrange = [&](RowStager<NH, WHOLE>& half, u32x2 (&unit)[NH][8]) {
        half.arrange(unit);
#pragma unroll
        for (int p = 0; p < NH; ++p)
#pragma unroll
            for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(unit[p][q]));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto put = [&](uint8_t* units) {
        if constexpr (WHOLE && NP == 4) put_block<NP, NH>(units, ulo, uhi, tid);
        else {
            put_units<NP, NH>(units, ulo, 0, tid);
            put_units<NP, NH>(units, uhi, 1, tid);
        }
    };
    // Where there is room for two chunks, one is staged beside the one that is walked, and all waves meet once a chunk: it is staged, and the one before has been walked; and once more
    // after a block's last chunk: all sums are there.  Otherwise they meet twice: the chunk before is no longer read, then the new one is staged.
    if (w.block < blocks) {
        if (w.block != (int)blockIdx.x) {
            fetch_lo();
            fetch_hi();
        }
        const bool two = two_chunks<NP>(w.nvcols);
        bool after_last = false;
        look_up_here();
        auto stage = [&]() {
            uint8_t* const units = smem + (two ? turn * kSecondBase<NP> : 0);
            arrange(hi, uhi);
            put_note();
            if (!two) __syncthreads();                                // no longer read (at first: the first note is there)
            put(units);
        };
        auto meet = [&]() {
            if (two && after_last) __syncthreads();                   // the sums of a block are there
            __syncthreads();                                          // staged
        };
        for (;;) {
            arrange(lo, ulo);
            const bool last = c + 1 == w.nchunks;
            advance();
            if (w.block >= blocks) break;                             // (what a round fetches for the next it fetches always: what may stay as it was is moved as well)
            look_after(w.pr, w.H, chunk());
            fetch_lo();
            __builtin_amdgcn_sched_barrier(0);
            stage();
            if (!two) meet();
            __builtin_amdgcn_sched_barrier(0);
            fetch_hi();                                               // (some 900 cycles)
            look_up_here();
            if (two) meet();
            after_last = last;
        }
        if (w.others) head.flags |= kHalvesFollow;
        stage();
        meet();
        __syncthreads();                                              // no longer read; the sums of the last block are there
    }
    if constexpr (NP == 4) {
        if (!w.others) return;
        auto none = [](const RowBlocks&, PlanHeaderPtr, bool) {};
        BlockWalk<NP, true> h, following;                             // the present block and the one after it
        int part = 0, k = 0;
        h.find(blockIdx.x, blocks, r, d, none);
        if (h.block >= blocks) return;
        following.find(h.block + gridDim.x, blocks, r, d, none);
        turn = 0;
        auto tell = [&]() {
            look_up(h.pr, h.H, h.nchunks, k, R / 2, h.pr.block * R + part * (R / 2));
            if (k + 1 < h.nchunks) look_after(h.pr, h.H, chunk_at(k + 1, h.pr.block * R, h.pr.m, h.nchunks));
            else if (part == 0) look_after(h.pr, h.H, chunk_at(0, h.pr.block * R, h.pr.m, h.nchunks));
            else if (following.block < blocks) look_after(following.pr, following.H, chunk_at(0, following.pr.block * R, following.pr.m, following.nchunks));
            put_note();
        };
        __syncthreads();                                              // nobody reads the last note of the other blocks any more
        tell();
        __syncthreads();                                              // the first note is there
        while (h.block < blocks) {
            lo.fetch(static_cast<const uint16_t*>(h.pr.G), (int64_t)h.pr.block * R + part * (R / 2), h.pr.m, h.pr.n, chunk_at(k, h.pr.block * R, h.pr.m, h.nchunks), tid);
            lo.arrange(ulo);
            put_units<2, 2>(smem, ulo, 0, tid);
            zero_unit<2>(smem, tid);                                  // (inside the larger units)
            __syncthreads();                                          // staged
            if (++k == h.nchunks) {
                k = 0;
                if (part ^= 1; part == 0) {
                    h = following;
                    if (h.block < blocks) following.find(h.block + gridDim.x, blocks, r, d, none);
                }
            }
            if (h.block < blocks) tell();
            __syncthreads();                                          // no longer read
        }
    }
}

__device__ __forceinline__ int tiles_of_wave(int V, int wave) {
    int count = 0;
#pragma unroll
    for (int i = 0; i < kWaveTiles; ++i) count += tile_of_wave(i, wave) * kTileCols < V ? 1 : 0;
    return count;
}

template <typename F, int... k> __device__ __forceinline__ void every_slot(F& f, std::integer_sequence<int, k...>) { (f(std::integral_constant<int, k>{}), ...); }

// Waves that walk the lists, in blocks of 4 NP rows; HALVES: in blocks whose sums do not fit the LDS, of which they take 8 rows, then the other 8.
//
// RING: steps of the plan a wave holds in registers.  Returns whether there may be blocks of the other kind (looking for them takes 1000 cycles).
template <int NP, int RING, bool HALVES>
__device__ __forceinline__ bool walk_blocks(uint8_t* smem, int blocks, int r, int d, int tid) {
    static_assert(RING % 2 == 0 && RING <= kStepsAhead, "the gathers take turns; so many steps are readable behind a plan's last");
    constexpr int NW = HALVES ? 2 : NP;                               // lists that share a lane's rows
    constexpr int R = kRowsMM<NW>;
    constexpr int kGroup = NW == 4 ? 2 : 1;                           // log2 of the blocks that one list's values go to
    const int lane = tid & (kWave - 1), part = lane & 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ChunkNote* const first_note = reinterpret_cast<const ChunkNote*>(smem + kNoteBase<NP>);
    const ChunkNote* note = first_note;
    auto column = [&](int i) { return note->cols[wave][lane >> 2][i]; };   // of this 4-lane group's two lists in tile i
    BlockWalk<NP, HALVES> w;
    w.find(blockIdx.x, blocks, r, d, [](const RowBlocks&, PlanHeaderPtr, bool) {});
    if (w.block >= blocks) return w.others;
    const bool two = !HALVES && two_chunks<NP>(w.nvcols);                  // (see fetch_blocks)
    const uint32_t sums_at = (uint32_t)sums_base<NP>(two);

    // A chunk's steps lie one behind the other.  ring: the next RING, from slot 0 on; those of the next chunk take the places of the last ones.
    u32x4 ring[RING];
    const uint32_t lane16 = lane * 16;
    auto step_at = [&](uint64_t steps, int k) { return *(const u32x4 LSP_GLOBAL_AS*)(steps + (uint64_t)k * (kWave * 16) + lane16); };
    int stride, t = 0, steps;
    uint32_t flags;
    uint64_t ahead, next;                                                 // the present chunk's step that the next round begins with; the next chunk's first
    uint64_t len_lo, len_hi;                                          // steps of each tile of the chunk, 16 bits each
    auto length = [&](int i) {                                        // (uniform)
        static_assert(kWaveTiles == 8, "two words");
        return i < kWaveTiles ? (int)(((i < 4 ? len_lo : len_hi) >> (16 * (i & 3))) & 0xFFFF) : 0;
    };
    // A tile's sums join those of the chunks before.  Lane l has the sums over the three parts of the values for row l % R of lists NW (l / R) + a, in three
    // registers (the fourth holds what the offsets gave).  With G as the A operand the parts would lie in three lanes, and took 16 more products a set to be brought
    // together: seven matrices of a 6.7B layer 403 -> 393 us, 4096 x 16384, skewed columns, 76.7 -> 73.3, 4096 x 4096, r = 2048, 98.1 -> 94.2 (steps and compress calls).
    f32x4 D[2][NW];                                                   // [set of 16 lists][list of the NW that share these lanes' rows]
    float LSP_LDS_AS* dst[2][NW];
    float before[2][NW];                                              // asked for when the tile begins
    uint32_t own_cols;                                                // columns of this 4-lane group's two lists in the next tile
    auto places = [&](uint32_t both) {
        const uint32_t mine = sums_at + (lane & (R - 1)) * stride * 4;   // (LDS address)
        auto place = [&](auto which) {
            constexpr int a = decltype(which)::value;
            const uint32_t x = list_of<NW, a>(both);
            dst[0][a] = (float LSP_LDS_AS*)(uintptr_t)unit_at<4, false>(x, mine);
            dst[1][a] = (float LSP_LDS_AS*)(uintptr_t)unit_at<4, true>(x, mine);
        };
        place(std::integral_constant<int, 0>{});
        place(std::integral_constant<int, 1>{});
        if constexpr (NW == 4) {
            place(std::integral_constant<int, 2>{});
            place(std::integral_constant<int, 3>{});
        }
    };
    auto begin = [&]() {
        const s16x4 none = {0, 0, 0, 0};
        places(own_cols);
        own_cols = column((t + 1) & (kWaveTiles - 1));
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < NW; ++a) D[h][a] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(none, none, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < NW; ++a) before[h][a] = 0.0f;
        if (!(flags & kFirstChunk)) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < NW; ++a) before[h][a] = *dst[h][a];
        }
    };
    auto flush = [&]() {
        float minus[2][NW];
        float odd = 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < NW; ++a) {
                minus[h][a] = minus_sum_of_parts(D[h][a][0], D[h][a][1], D[h][a][2]);
                odd += fabsf(minus[h][a]);
            }
        // An infinity in G meets zeros among the lower parts: where the sum is no number the first part alone says what becomes of it.  (Nothing says
        // it for values below 2^-133, whose first part is zero: an infinity times one of them is NaN.)  An infinite sum stays one: the first part may
        // be finite where the value's product is not.
        if (__builtin_expect(__any(!(odd < __builtin_inff())), 0)) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int a = 0; a < NW; ++a) minus[h][a] = minus[h][a] == minus[h][a] ? minus[h][a] : -D[h][a][0];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < NW; ++a) *dst[h][a] = before[h][a] - minus[h][a];
    };

    // The transposing read takes entry e of a list from lanes 4 e .. 4 e + 3 of 16, lane 4 e + s the s-th 8 bytes, and hands lane l the l-th row's four values:
    // with NW = 4 all of one unit, with NW = 2 of the units of two lists.  The offsets of entry e of the 16 lanes' four lists are in the fourth lane of their 4-lane group.
    uint32_t piece = (part & (NW - 1)) * 8;                           // (of the present chunk)
    s16x4 g[2][2][NW];
    auto gather = [&](auto slot) {
        constexpr int k = decltype(slot)::value;
        auto read = [&](int h, int a, uint32_t two, auto high) {      // (the units start where the LDS starts)
            const uint32_t off = unit_at<(1 << kGroup), decltype(high)::value>(two, piece);
            g[k & 1][h][a] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LSP_LDS_AS s16x4*)(uintptr_t)off);
        };
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t lo = quad_lane<3>(ring[k][2 * h]), hi = quad_lane<3>(ring[k][2 * h + 1]);
            const uint32_t x = NW == 4 || !(part & 2) ? lo : hi;
            read(h, 0, x, std::false_type{});
            read(h, 1, x, std::true_type{});
            if constexpr (NW == 4) {
                read(h, 2, hi, std::false_type{});
                read(h, 3, hi, std::true_type{});
            }
        }
    };
    auto multiply = [&](auto slot, uint64_t refill) {
        constexpr int k = decltype(slot)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x2 x = {ring[k][2 * h], ring[k][2 * h + 1]};
            const s16x4 (&y)[NW] = g[k & 1][h];
            s16x4 v;
            __builtin_memcpy(&v, &x, 8);
            D[h][0] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, y[0], D[h][0], kGroup, 0, 0);
            D[h][1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, y[1], D[h][1], kGroup, 1, 0);
            if constexpr (NW == 4) {
                D[h][2] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, y[2], D[h][2], kGroup, 2, 0);
                D[h][3] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(v, y[3], D[h][3], kGroup, 3, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        ring[k] = step_at(refill, k);
    };
    // The gathers of a step are asked for before the products of the one before.  The barriers keep the compiler from waiting for each gather by itself and from
    // giving the refills registers of their own, which a loop would have to move.
    auto slots = [](auto&& f) {                                       // f of every slot of the ring, in turn
        every_slot(f, std::make_integer_sequence<int, RING>{});
    };
    // The steps of a chunk, of which the first is in slot 0: whole rounds, then the rest as nested conditions.  A way out of the middle of a loop would cost the compiler its
    // knowledge of what is in flight; for the same reason the last step also gathers for a step behind it, for nothing, and a tile begins behind the last one.
    auto walk_chunk = [&]() {
        int left = length(0), remaining = steps;                      // steps of the tile, and of the chunk
        auto step = [&](auto slot, uint64_t refill) {
            constexpr int k = decltype(slot)::value;
            gather(std::integral_constant<int, (k + 1) % RING>{});
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC07F | (2 * NW << 8));       // lgkmcnt(2 NW): what was asked for before is there
            __builtin_amdgcn_sched_barrier(0);
            multiply(slot, refill);
            if (__builtin_expect(--left == 0, 0)) {
                flush();
                left = length(++t);
                begin();
            }
        };
        gather(std::integral_constant<int, 0>{});
        begin();
        for (; remaining > RING; ahead += RING * kWave * 16)
            slots([&](auto slot) { step(slot, remaining-- > RING ? ahead : next); });
        auto rest = [&](auto&& self, auto slot) -> void {
            constexpr int k = decltype(slot)::value;
            if (k < remaining) {
                step(slot, next);
                if constexpr (k + 1 < RING) self(self, std::integral_constant<int, k + 1>{});
            }
        };
        rest(rest, std::integral_constant<int, 0>{});
    };

    auto ring_of = [&](uint64_t from) {
        slots([&](auto slot) { ring[decltype(slot)::value] = step_at(from, decltype(slot)::value); });
    };
    // A chunk's first steps are waited for all together (the last of them was asked for before the chunk was staged).  Without this the compiler, which cannot know
    // how many loads lie behind them, would wait for every load in flight in every round of the ring.
    auto wait_for_loads = []() {
        __builtin_amdgcn_s_waitcnt(0x0F70);                           // vmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
    };
    ring_of((uint64_t)(uintptr_t)w.pr.plan + w.H->off_m_steps + (uint64_t)as_const<TileSeg>(w.pr.plan + w.H->off_m_seg)[chunk_at(0, w.pr.block * kRowsMM<NP>, w.pr.m, w.nchunks) * kWavesMM + wave].first_step * (kWave * 16));
    const auto uniform = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    const auto uniform2 = [&](uint32_t lo, uint32_t hi) { return (uint64_t)uniform(hi) << 32 | uniform(lo); };
    const auto piece16 = [&](const void* p) { return *static_cast<const u32x4*>(p); };
    if (HALVES) __syncthreads();                                      // the other blocks' last note has been read
    if (!two) __syncthreads();                                        // the first note is there
    int nvcols;
    auto read_note = [&]() {
        const u32x4 seg0 = piece16(&note->seg[wave]), seg1 = piece16(reinterpret_cast<const uint8_t*>(&note->seg[wave]) + 16);
        const u32x2 after = *reinterpret_cast<const u32x2*>(&note->steps[0][wave]), here = *reinterpret_cast<const u32x2*>(&note->steps[1][wave]);
        const u32x2 head = *reinterpret_cast<const u32x2*>(&note->nvcols);
        own_cols = column(0);
        steps = (int)uniform(seg0.y);
        len_lo = uniform2(seg0.z, seg0.w); len_hi = uniform2(seg1.x, seg1.y);
        next = uniform2(after.x, after.y);
        ahead = uniform2(here.x, here.y) + RING * (kWave * 16);
        nvcols = (int)uniform(head.x);
        flags = uniform(head.y);
        stride = sums_stride(nvcols);
    };
    for (;;) {
        if (!two) read_note();
        __syncthreads();                                              // the chunk is staged
        if (two) read_note();
        wait_for_loads();
        t = 0;
        if (steps > 0) walk_chunk();
        if (steps < RING)
            slots([&](auto slot) {
                constexpr int k = decltype(slot)::value;
                if (k >= steps) ring[k] = step_at(next, k);
            });
        if (flags & kFirstChunk)
            for (const int mytiles = tiles_of_wave(nvcols, wave); t < mytiles; ++t) {   // tiles without an entry in a block's first chunk: their sums start at zero
                places(column(t));
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int a = 0; a < NW; ++a) *dst[h][a] = 0.0f;
            }
        if (!two || (flags & kLastChunk)) __syncthreads();            // no longer read; all sums are there
        if (flags & kLastChunk) {
            int thread = tid;                                         // (opaque, so that nothing of this is made outside the loop, and kept in registers all along)
            asm volatile("" : "+v"(thread));
            const u32x4 head0 = piece16(&note->T), head1 = piece16(&note->vcol);
            const uint64_t plan = uniform2(head0.z, head0.w);
            store_sums<R>(reinterpret_cast<const float*>(smem + sums_at), stride, (float LSP_GLOBAL_AS*)uniform2(head0.x, head0.y), (const uint16_t LSP_GLOBAL_AS*)(plan + uniform(head1.x)),
                          (const uint16_t LSP_GLOBAL_AS*)(plan + uniform(head1.y)), (flags & kSharedColumns) != 0, nvcols, (int)uniform(head1.z), r, thread);
        }
        if (!(flags & kMoreChunks)) return (flags & kHalvesFollow) != 0;
        const bool second = note == first_note;
        note = first_note + second;
        if (two) piece = (part & (NW - 1)) * 8 + (second ? (uint32_t)kSecondBase<NP> : 0u);
    }
}

template <int NP, int RING, bool WHOLE>
__global__ __launch_bounds__(kThreadsMM) void k_compress_mm(const CompressGroup) {
    extern __shared__ __align__(16) uint8_t smem[];
    words4 head = scalar_load<words4>(group_args<CompressGroup>());
    const int r = (int)head[1], d = (int)head[2], blocks = (int)head[3];
    const int tid = threadIdx.x;
    zero_unit<NP>(smem, tid);
    zero_unit<NP>(smem + kSecondBase<NP>, tid);                       // (where there is no second chunk, sums of later on)
    if (__builtin_amdgcn_readfirstlane(tid) >= kWalkers) fetch_blocks<NP, WHOLE>(smem, blocks, r, d, tid - kWalkers);
    else {
        const bool others = walk_blocks<NP, RING, false>(smem, blocks, r, d, tid);
        if constexpr (NP == 4)
            if (others) walk_blocks<NP, RING, true>(smem, blocks, r, d, tid);   // more sums than the LDS has room for: 8 rows, then 8 rows
    }
}

template <int NP, int RING> static hipError_t launch_mm_rows(CompressGroup& g, hipStream_t st) {
    constexpr int R = kRowsMM<NP>;
    constexpr size_t lds = kLdsMM;
    bool whole = true;
    g.blocks = 0;
    for (int p = 0; p < kMaxGroup; ++p) {
        CompressProblem& x = g.p[p];
        g.first_gq[p] = INT32_MAX;
        g.plans[p] = g.p[p < g.count ? p : 0].plan;
        if (p >= g.count) continue;
        whole = whole && x.n % 8 == 0;
        x.blocks_gq = 1;
        x.wgs_gq = (x.m + R - 1) / R;
        g.first_gq[p] = x.first_gq = g.blocks;
        g.blocks += x.wgs_gq;
    }
    const dim3 grid((unsigned)std::min(g.blocks, kResidentMM));
    hipError_t e;
    if (whole) {
        if ((e = allow_dynamic_lds<k_compress_mm<NP, RING, true>, lds>()) != hipSuccess) return e;
        hipLaunchKernelGGL((k_compress_mm<NP, RING, true>), grid, dim3(kThreadsMM), lds, st, g);
    } else {
        if ((e = allow_dynamic_lds<k_compress_mm<NP, RING, false>, lds>()) != hipSuccess) return e;
        hipLaunchKernelGGL((k_compress_mm<NP, RING, false>), grid, dim3(kThreadsMM), lds, st, g);
    }
    return hipGetLastError();
}

// Blocks of 16 rows read the plan half as often as blocks of 8 and share each value between twice the rows (us with kernel B, 16 and 8 rows: 4096 x 4096, d = 8, r = 512 25.6 and 27.3,
// r = 1024 35.2 and 36.1; 3001 x 3001, r = 512, d = 8 22.2 and 24.0; 9000 x 2048 36.4 and 38.5, zipf 54.5 and 58.0; 4096 x 1024, r = 64, d = 2 14.1 and 15.3).  8 rows are better
//   where there is at most one block of 8 for a CU, so that the blocks of 16 would leave CUs idle (2048 x 4096, r = 512, d = 8 16.9 us, with 16 20.9; 1024 x 1024, r = 128, d = 4 10.1 and 12.0);
//   where they take three rounds of one for every CU and the blocks of 16 two, the last of them little more than half full or less: 4097 to 6144 rows (us with 8
//   and with 16 rows: 5120 x 5120, r = 512, d = 8 40.2 and 41.3, zipf 55.1 and 55.6; r = 1024, d = 8 48.4 and 53.2; d = 16 66.8 and 71.1; 6144 x 4096, r = 512, d = 8 even, r = 1024,
//   d = 4 37.3 and 40.1, r = 256, d = 4 29.1 and 28.4; 4200 x 2048, r = 1024, d = 8, zipf 53.9 and 51.6);
//   and beyond r = 1024, where the sums of 16 rows do not fit the LDS (4096 x 4096, d = 8, r = 1536 43.5 and 46.0, r = 2048 49.2 and 51.5, d = 16 65.7 and 64.9; 5120 x 5120, r = 2048,
//   d = 8 69.6 and 89.3).
static bool narrow_blocks(const CompressGroup& g) {
    int64_t of8 = 0, of16 = 0;
    for (int p = 0; p < g.count; ++p) {
        of8 += (g.p[p].m + 7) / 8;
        of16 += (g.p[p].m + 15) / 16;
    }
    const auto rounds = [](int64_t blocks) { return (blocks + kResidentMM - 1) / kResidentMM; };
    return g.r > 1024 || rounds(of8) == 1 || (rounds(of8) == 3 && rounds(of16) == 2);
}

// Every bf16 call with a kept plan comes here, whatever its rows: the sums of a row do not depend on the blocks it is in, so a matrix has the same
// result alone and in any group, which a second kernel with sums in another order would end.  k_compress_gq is behind nearly everywhere (us with kernel B, here and there):
//   5120 x 5120  r = 512, d = 8 40.3 and 43.6, zipf 55.1 and 72.6; r = 512, d = 4 33.1 and 36.1; r = 1024, d = 8 48.4 and 57.9; r = 2048, d = 8 70.0 and 88.1
//   5120 x 13824 r = 512, d = 8 78.2 and 81.2; r = 1024, d = 16 131.9 and 144.4      6144 x 4096 r = 256, d = 4 29.0 and 35.4, d = 16 53.5 and 52.3, zipf 67.2 and 71.9
//   4096 x 4096  r = 2048, d = 4 41.6 and 50.9, d = 8 49.4 and 55.9, d = 16 66.0 and 72.1      9000 x 2048 r = 512, d = 8 37.1 and 40.6
// Steps of the plan that a wave holds in registers: eight hide the plan's latency behind the loads of G, but a chunk loads as many of the next one's, whether it has them or not (some
// 2 d steps a wave and chunk).  us with 8, 6 and 4: 4096 x 16384, r = 512, d = 2 40.8, 38.8 and 37.5, d = 4 41.4, 42.3 and 44.1, d = 8 53.2, 53.7 and 55.9; 4096 x 1024, r = 64, d = 2
// 14.6, 14.4 and 14.0.  Blocks of 8 rows: 2048 x 8192, r = 512, d = 4 19.8, 19.7 and 20.2; 5120 x 5120 34.2, 33.5 and 33.6, d = 8 40.6, 40.6 and 42.0; with 6 and 4, two chunks and fewer:
// 5120 x 4096, r = 512, d = 8 33.3 and 34.4; 4096 x 4096, r = 2048, d = 8 49.0 and 49.6, d = 16 62.6 and 64.8; 2048 x 4096, r = 128, d = 4 15.6 and 15.9; 264 x 657, r = 21, d = 3 10.9 and 10.8.
hipError_t launch_mm_bf16(CompressGroup& g, hipStream_t st) {
    if (narrow_blocks(g)) return g.d <= 2 ? launch_mm_rows<2, 4>(g, st) : launch_mm_rows<2, 6>(g, st);
    return g.d <= 2 ? launch_mm_rows<4, 4>(g, st) : launch_mm_rows<4, 8>(g, st);
}

}  // namespace lsp
