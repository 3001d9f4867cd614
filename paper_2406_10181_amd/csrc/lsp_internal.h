// Internal declarations shared by the translation units of the HIP library (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "lsp.h"

namespace lsp {

// ------------------------------------------------------------------------------------------
// Tiling constants of the compress kernels (the plan layout depends on them).
// ------------------------------------------------------------------------------------------
constexpr int kChunk      = 2048;  // columns of G staged in LDS at a time
constexpr int kWave       = 64;    // gfx950 wavefront
constexpr int kThreadsGQ  = 512;   // threads of the T = G Q kernel: one lane per (virtual) column of T
constexpr int kWavesGQ    = kThreadsGQ / kWave;
constexpr int kMaxSlots   = 4;     // a lane owns at most this many virtual columns
constexpr int kSegBatch   = 4;     // segment lengths are multiples of this many rows
constexpr int kPrefetch   = 4;     // batches of plan rows a wave holds in registers (one consumed, the rest in flight)
constexpr int kStreamSlack = kPrefetch * kSegBatch;   // readable padding rows after the last segment
constexpr int kRowPiece   = 256;   // a row list of P^T longer than this is cut into pieces
// bf16 goes through matrix instructions (compress_mm.hip): tiles of 32 lists, two sets of 16, four entries of each a step
constexpr int kSetCols    = 16;    // lists of a set: the 16 blocks of v_mfma_f32_4x4x4_16b_bf16
constexpr int kTileCols   = 2 * kSetCols;
constexpr int kStepEntries = 4;    // entries of every list a step takes: the K of a block
constexpr int kWavesMM    = 8;     // waves of that kernel that walk the lists
constexpr int kWaveTiles  = kMaxSlots * kThreadsGQ / kTileCols / kWavesMM;   // most tiles of a wave in one chunk
constexpr int kStepsAhead = 10;     // so many readable steps follow the last one of a plan; a wave may ask for as many ahead
constexpr uint32_t kNoColumn = 0xFFFFu;      // virtual column slot without a column
constexpr uint32_t kSharedColumn = 0x8000u;  // flag: the column is owned by several lanes

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Remembers the raw HIP error for lsp_last_hip_error() and returns LSP_ERR_LAUNCH.
int note_hip_error(hipError_t e);

// LDS byte offset, inside one 4-row plane, of local column j of a staged chunk.
// Columns are stored as [j & 7][j >> 3] in units of 16 bytes (4 rows x fp32), so that the 64
// lanes of a staging wave, which hold 8 consecutive columns each, write consecutive units.
__host__ __device__ static inline uint32_t chunk_col_offset(uint32_t j) {
    return (((j & 7u) * (kChunk / 8)) + (j >> 3)) * 16u;
}

// The same for the bf16 kernel, for units of 8 bytes: it has a column's 8 or 16 rows side by side, 16 or 32 bytes, and multiplies the offset by 2 or 4 as it reads it.
__host__ __device__ static inline uint32_t chunk_unit_offset(uint32_t j) { return chunk_col_offset(j) / 2; }

// ------------------------------------------------------------------------------------------
// Plan: column-sorted projector copies, laid out for the compress kernels.
// All offsets are bytes from the start of the plan buffer and multiples of 16.
//
// Q part.  Every column b of T = G Q is owned by one lane of the 512-thread workgroup, which keeps
// the column's partial sums in registers.  A column whose list of (column j of
// G, value) pairs is longer than list_cap inside some chunk gets several owners ("virtual
// columns"), each taking an equal share of the list in every chunk; the owners' sums are added at
// the end, in a fixed order.  Lanes left over (r < 512) are given to the columns with the longest
// shares, so that all lanes of the workgroup carry about the same load.  Virtual column v sits in
// slot v / 512, lane v % 512 -- except that with one slot (q_permuted) the lane that walks a
// column's list changes from chunk to chunk: inside each chunk the 512 lists are dealt to the waves
// by length, longest first (a wave is as slow as its longest list, so lists of like length go
// together; the two waves that share a SIMD get a long and a short group), and the kernel hands
// the partial sums from lane to lane between chunks.  q_perm[c][t] is the virtual column that
// thread t walks in chunk c.  For each (chunk, slot, wave) the
// 64 lists are padded to a common length (a multiple of kSegBatch) with pairs that point at an
// always-zero LDS unit, and stored lane-interleaved two rows at a time: rows 2p and 2p+1 form
// 64 x (LDS offset, value bits, LDS offset, value bits), one 128-bit load per lane.
// The rows of one wave are contiguous over all chunks and slots (chunk-major), so a wave reads
// one linear stream.
//
// The lists once more for the bf16 kernel.  Per chunk all virtual columns are sorted by length, longest first, and cut into
// tiles of 32; they are dealt to 8 waves in rounds, some backwards (tile_of_wave), so that the waves get about the same number of
// steps.  A step is four entries of every list of a tile: 64 x 16 bytes, the first 8 for lists 0..15 and the others for 16..31.
// In each half, with 4-lane group b = lane / 4 and s = lane % 4:
//   s < 3    part s of the values of list b's four entries (value_parts, bf16 each: the A operand as it is)
//   s = 3    the LDS offsets of entry b % 4 of the four lists b / 4 * 4 .. + 3 (the transposing LDS read takes the entries of
//            a list from lanes 4 apart)
// A list shorter than the tile's longest is filled up with zero values at the always-zero unit.
// ------------------------------------------------------------------------------------------
struct PlanHeader {            // first 256 bytes of the plan buffer
    uint32_t magic;            // kPlanMagic
    int32_t  m, n, r, d;
    int32_t  nchunks;          // ceil(n / kChunk)
    int32_t  nslots;           // virtual columns per lane (1 .. kMaxSlots)
    int32_t  nvcols;           // virtual columns in use
    int32_t  q_total_rows;     // rows of all wave streams, slack included
    int32_t  p_nitems;         // pieces of rows of P^T
    int32_t  p_any_split;      // 1 if some row of P^T was cut (S must start at zero)
    int32_t  list_cap;         // longest list a lane walks in one chunk
    uint32_t q_stream_row[kWavesGQ];   // first row of each wave's stream
    int32_t  q_any_shared;     // 1 if some column of T has several owners
    int32_t  q_permuted;       // 1 if the owner of a virtual column changes per chunk (q_perm; one slot only)
    uint32_t pad[2];
    // section offsets
    uint64_t off_q_seg;        // uint32[nchunks][nslots][kWavesGQ]  rows of each segment
    uint64_t off_q_vcol;       // uint16[nslots * 512]               column b (| kSharedColumn) or kNoColumn
    uint64_t off_q_rows;       // uint4[q_total_rows / 2][64]
    uint64_t off_p_item;       // RowItem[p_nitems]
    uint64_t off_p_ent;        // uint2[m*d]                         (row i, value bits)
    uint64_t total_bytes;
    uint64_t off_q_vcnt;       // uint16[nslots * 512]               owners of the column if this is its first owner, else 0
    uint64_t off_q_perm;       // uint16[nchunks][512]               virtual column walked by thread t in chunk c
    // where every stored value came from, so that new values can be dropped into an existing plan when only
    // the values of the projectors change (lsp_plan_refresh_values): flat ELL positions row * d + k
    uint64_t off_q_src;        // uint32[q_total_rows][64], laid out like q_rows; kNoSource for padding pairs
    uint64_t off_p_src;        // uint32[m*d], parallel to p_ent
    // tiles of lists (bf16)
    uint64_t off_m_seg;        // TileSeg[nchunks][kWavesMM]
    uint64_t off_m_cols;       // uint16[nchunks][kWavesMM][16][kWaveTiles][2]   virtual columns of lists b and 16 + b of the wave's tile t; lists
                               // that fill up the last tile count on from nvcols
    uint64_t off_m_steps;      // uint4[m_total_steps][64]
    uint64_t off_m_src;        // uint32[m_total_steps][2][16][4]     flat ELL position of entry k of list 16 h + b; kNoSource: none
    uint32_t m_total_steps;    // kStepsAhead readable ones behind the last included; 0: no tiles (raw calls)
    uint32_t pad2;
};
static_assert(sizeof(PlanHeader) == 216, "PlanHeader layout");
constexpr uint32_t kPlanMagic = 0x4C535039u;   // "LSP9"; another one for every change of the layout, so that kept plans of an older one are refused
constexpr uint32_t kNoSource = 0xFFFFFFFFu;    // q_src of a padding pair
constexpr size_t   kPlanHeaderBytes = 256;

struct RowItem   { int32_t a; int32_t start; int32_t len; int32_t atomic; };

// What wave w does in chunk c: its steps (consecutive) and how many of them each of its tiles has.
struct TileSeg   { uint32_t first_step; uint32_t steps; uint16_t len[kWaveTiles]; uint32_t pad[2]; };
static_assert(sizeof(TileSeg) == 32, "one scalar load");
// Tile i of wave w, as a position in the sorted order (0: the longest lists).  Round i goes backwards where i has an odd number of
// bits set: no wave is first or last in most rounds.
__host__ __device__ static inline int tile_of_wave(int i, int w) { return kWavesMM * i + (((0x6996 >> i) & 1) ? kWavesMM - 1 - w : w); }

// The three bf16 parts of a value, highest first: v = part[0] + 2^-kPartShift[1] part[1] + 2^-kPartShift[2] part[2].  Each takes the leading 8 significant
// bits of what is left, which is scaled by a power of two so that it is about as large as v, and no larger (so products and sums of a part
// overflow only where those of v could): exact for |v| >= 2^-125, and for smaller ones but for a last bit of 2^-149.  (Not scaled, the parts of
// values below 2^-110 would lose what lies under the smallest bf16, 2^-133.)  An infinity or NaN is its first part.
constexpr int kPartShift[3] = {0, 7, 15};
// (Without a loop or a branch: the parts of a loop the compiler kept in LDS, and lsp_plan_refresh_values took 11 us instead of 4 on 4096 x 4096, d = 8.)
__host__ __device__ static inline uint32_t bits_of(float x) { uint32_t u; __builtin_memcpy(&u, &x, 4); return u; }
__host__ __device__ static inline float without_low_half(float x) {
    const uint32_t u = bits_of(x) & 0xFFFF0000u;
    float head;
    __builtin_memcpy(&head, &u, 4);
    return head;
}
__host__ __device__ static inline void value_parts(float v, uint16_t (&part)[3]) {
    const uint32_t u = bits_of(v);
    const bool odd = (u & 0x7F800000u) == 0x7F800000u;
    const float second = odd ? 0.0f : (v - without_low_half(v)) * (float)(1 << kPartShift[1]);
    const float third = (second - without_low_half(second)) * (float)(1 << (kPartShift[2] - kPartShift[1]));
    part[0] = (uint16_t)((u >> 16) | (odd && (u & 0x007FFFFFu) ? 0x40u : 0u));
    part[1] = (uint16_t)(bits_of(second) >> 16);
    part[2] = (uint16_t)(bits_of(third) >> 16);
}

// Copy of an ELL projector with the entries of each row ordered against LDS bank conflicts in the
// decompress kernels (host arrays; the matrix itself is unchanged).
int reorder_rows_host(const int32_t* idx, const float* val, int64_t rows, int32_t d, int32_t r,
                      int32_t* idx_out, float* val_out);

// Byte offsets of the plan's sections (they depend on the shape only).
struct PlanLayout { size_t off_q_seg, off_q_vcol, off_q_vcnt, off_q_perm, off_q_rows, off_p_item, off_p_ent, off_q_src, off_p_src,
                           off_m_seg, off_m_cols, off_m_steps, off_m_src, total; };
PlanLayout plan_layout(int64_t m, int64_t n, int32_t r, int32_t d);

// Upper bounds (depend on shapes only) used to size the plan buffer.
int    plan_list_cap(int32_t r, int32_t d);
size_t plan_max_rows(int64_t n, int32_t r, int32_t d);
size_t plan_max_steps(int64_t n, int32_t r, int32_t d);
size_t plan_max_items(int64_t m, int32_t r, int32_t d);
size_t plan_bytes(int64_t m, int64_t n, int32_t r, int32_t d);

// Host-side builder: fills `host_plan` (plan_bytes() bytes) from host copies of the ELL arrays.
// Returns LSP_OK, or LSP_ERR_SKEW when the columns of Q are so unevenly used that more than
// kMaxSlots * 512 virtual columns would be needed.
int build_plan_host(const int32_t* P_idx, const float* P_val, const int32_t* Q_idx, const float* Q_val,
                    int64_t m, int64_t n, int32_t r, int32_t d, uint8_t* host_plan);

// ------------------------------------------------------------------------------------------
// Groups: several independent problems (same r, d, dtype) served by one launch per kernel, so that
// workgroups of different matrices fill the CUs together.  Passed to the kernels by value, as their first argument.
// A kernel's first work is a chain of dependent scalar loads, each a trip to memory, so everything that it needs to know of a problem is one record of 64
// bytes, and what is the same for all lies before the first of them: a call of one problem has it all from one trip, a group from two.  (One array per
// field took four to ten trips, which were 0.7 to 1.7 us of every launch.)
// ------------------------------------------------------------------------------------------
constexpr int kMaxGroup = LSP_MAX_GROUP;
struct CompressProblem {
    const void*    G;
    const uint8_t* plan;
    float*         T;
    float*         S;
    int32_t        m, n;
    int32_t        first_gq, wgs_gq;             // workgroups of the T = G Q kernel (bf16: row blocks): the first, and how many
    int32_t        blocks_gq;                    // row blocks of each of them
    int32_t        first_pt;                     // first workgroup of the S = P^T T kernel
    int32_t        round_pt;                     // workgroups of one of its rounds (k_compress_pt8)
    int32_t        pad;
};
struct CompressGroup {
    int32_t         count, r, d;
    int32_t         blocks;                      // all row blocks (bf16)
    int32_t         quads;                       // column quads of a stripe (k_compress_pt8), stripes (k_compress_pt)
    int32_t         tiles;                       // whether kernel A of this call walks the tiles
    int32_t         pad[10];
    CompressProblem p[kMaxGroup];
    int32_t         first_gq[kMaxGroup], first_pt[kMaxGroup];   // those of the problems once more; past the last problem INT32_MAX
    const uint8_t*  plans[kMaxGroup];            // and their plans (bf16); past the last problem the first one's
};
struct ApplyProblem {
    void*          W;
    const float*   S;
    const int32_t* P_idx;
    const float*   P_val;
    const int32_t* Q_idx;
    const float*   Q_val;
    int32_t        m, n;
    int32_t        first;                        // first workgroup
    int32_t        parts;                        // workgroups that share a row block
};
struct ApplyGroup {
    int32_t      count, r, d;
    int32_t      pad0[5];
    float*       partial;                        // bias: a pair of sums for every workgroup
    int32_t      pad[6];
    ApplyProblem p[kMaxGroup];
    int32_t      first[kMaxGroup];               // those of the problems once more; past the last problem INT32_MAX
};
static_assert(kMaxGroup == 16 && sizeof(CompressProblem) == 64 && sizeof(ApplyProblem) == 64 && offsetof(CompressGroup, p) == 64 && offsetof(ApplyGroup, p) == 64,
              "records of 64 bytes, loaded whole");

#if defined(__HIPCC__)
// Read-only tables (kernel arguments; the plan's header, segment lengths, column tables) are read through the
// constant address space: the kernels never write them, and a uniform load from that address
// space is a scalar load, which does not share the counter (and the waits) of the vector loads
// that stream G and the plan rows.
#define LSP_CONST_AS __attribute__((address_space(4)))
template <typename T> __device__ __forceinline__ const LSP_CONST_AS T* as_const(const void* p) {
    return (const LSP_CONST_AS T*)(uintptr_t)p;
}
#define LSP_GLOBAL_AS __attribute__((address_space(1)))               // (of addresses that come out of memory the compiler would not know it)
template <typename T> __device__ __forceinline__ T* global_pointer(T* p) { return (T*)(T LSP_GLOBAL_AS*)(uintptr_t)p; }
// Scalar loads that are waited for together, and not where each is first used: one trip to memory.
typedef uint32_t words16 __attribute__((ext_vector_type(16)));
typedef uint32_t words8 __attribute__((ext_vector_type(8)));
typedef uint32_t words4 __attribute__((ext_vector_type(4)));
typedef uint32_t words2 __attribute__((ext_vector_type(2)));
template <typename V> __device__ __forceinline__ V scalar_load(const LSP_CONST_AS void* p, int word = 0) {
    return *(const LSP_CONST_AS V*)((const LSP_CONST_AS uint32_t*)p + word);
}
template <typename V> __device__ __forceinline__ void arrived(V& x) { asm volatile("" : "+s"(x)); }
template <typename V, typename... W> __device__ __forceinline__ void arrived(V& x, W&... rest) { arrived(x); arrived(rest...); }
// A kernel's first argument
template <typename Group> __device__ __forceinline__ const LSP_CONST_AS Group* group_args() {
    return (const LSP_CONST_AS Group*)__builtin_amdgcn_kernarg_segment_ptr();
}
// Brings the first N x 64 bytes of a kernel's arguments into the scalar cache in one trip; what is loaded of them later, where it is used, is there.
template <int N> __device__ __forceinline__ void touch_args() {
    const auto* p = group_args<uint32_t>();
    uint32_t x[N];
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = p[16 * k];
#pragma unroll
    for (int k = 0; k < N; ++k) arrived(x[k]);
}
__device__ __forceinline__ void know_pointers(CompressProblem& p) {
    p.G = global_pointer(p.G); p.plan = global_pointer(p.plan); p.T = global_pointer(p.T); p.S = global_pointer(p.S);
}
__device__ __forceinline__ void know_pointers(ApplyProblem& p) {
    p.W = global_pointer(p.W); p.S = global_pointer(p.S);
    p.P_idx = global_pointer(p.P_idx); p.P_val = global_pointer(p.P_val); p.Q_idx = global_pointer(p.Q_idx); p.Q_val = global_pointer(p.Q_val);
}
// The group's first words, and the problem that owns workgroup (or row block) `block`; first: where each problem begins.  Uniform, and in scalar registers.
template <typename Problem> struct Picked { int32_t count, r, d, blocks, quads, tiles; Problem p; };
template <typename Group> __device__ __forceinline__ auto pick_problem(const LSP_CONST_AS Group* g, const LSP_CONST_AS int32_t (&first)[kMaxGroup], int block) {
    words8 head = scalar_load<words8>(g);
    words16 record = scalar_load<words16>(&g->p[0]);
    arrived(head, record);
    if ((int)head[0] > 1) {                                           // (one problem: nothing but the head and its record is read)
        const words16 f = scalar_load<words16>(&first[0]);
        // (the number of problems that begin at this workgroup or before, less one, by sums of signs; the second half only where the first does not tell)
        int before = 0;
#pragma unroll
        for (int p = 1; p < kMaxGroup / 2; ++p) before += (block - (int)f[p]) >> 31;
        int k = kMaxGroup / 2 - 1 + before;
        if (k == kMaxGroup / 2 - 1) {
            before = 0;
#pragma unroll
            for (int p = kMaxGroup / 2; p < kMaxGroup; ++p) before += (block - (int)f[p]) >> 31;
            k = kMaxGroup - 1 + before;
        }
        record = scalar_load<words16>(&g->p[k]);
    }
    Picked<std::remove_cv_t<std::remove_reference_t<decltype(Group::p[0])>>> out;
    out.count = (int)head[0]; out.r = (int)head[1]; out.d = (int)head[2]; out.blocks = (int)head[3]; out.quads = (int)head[4]; out.tiles = (int)head[5];
    __builtin_memcpy(&out.p, &record, 64);
    know_pointers(out.p);
    return out;
}
#endif

// ------------------------------------------------------------------------------------------
// Kernel launchers (each returns hipSuccess or the launch error).  The group launchers fill in
// first_* themselves.
// ------------------------------------------------------------------------------------------
// A call on raw ELL arrays, whose plan was built just before on the same stream: kernel A looks here where it finds no plan.
// If *status (device, of the plan build) is LSP_ERR_SKEW it adds to S in scatter form (the build has set S to zero), any other error
// makes S NaN.
struct RawCall {
    const int32_t* P_idx; const float* P_val; const int32_t* Q_idx; const float* Q_val;
    const int32_t* status;                         // null: not such a call, no plan makes S NaN
};
hipError_t launch_compress_planned(CompressGroup& g, int32_t r, int32_t d, lsp_dtype dtype, hipStream_t st, const RawCall& raw = RawCall{});
hipError_t launch_decompress(ApplyGroup& g, int32_t r, int32_t d, lsp_dtype dtype, hipStream_t st);
// Dense-projector ablation of compress on the matrix cores (dense.hip): Pt = P^T [r][m], Qt = Q^T [r][n] in the
// storage type of G (fp16 / bf16); workspace of dense_workspace_bytes(m, r); shapes must pass dense_shape_ok.
bool       dense_shape_ok(int64_t m, int64_t n, int32_t r);
size_t     dense_workspace_bytes(int64_t m, int32_t r);
hipError_t launch_compress_dense(const void* G, const void* Pt, const void* Qt, int64_t m, int64_t n, int32_t r, float* S,
                                 uint8_t* workspace, lsp_dtype dtype, hipStream_t st);
// Estimation bias (Def. 2): `partial` holds bias_blocks(m, n, r, d) pairs of floats (enough for every storage type), `out` three floats.
int64_t    bias_blocks(int64_t m, int64_t n, int32_t r, int32_t d);
hipError_t launch_bias(ApplyGroup& g, int32_t r, int32_t d, lsp_dtype dtype, float* partial, float* out, hipStream_t st);
// Optimiser-state re-projection (MaybeUpdate, Alg. 1): workspace holds 4 r^2 floats; V may be null.
hipError_t launch_reproject(const int32_t* P_idx, const float* P_val, const int32_t* Pp_idx, const float* Pp_val,
                            const int32_t* Q_idx, const float* Q_val, const int32_t* Qp_idx, const float* Qp_val,
                            int64_t m, int64_t n, int32_t r, int32_t d, float* M, float* V, float* workspace,
                            hipStream_t st);
hipError_t launch_validate(const int32_t* idx, int64_t count, int32_t r, int32_t* flag, hipStream_t st);
// Values-only refresh of a plan (same indices, new values).
hipError_t launch_plan_refresh(uint8_t* plan, const float* P_val, const float* Q_val,
                               int64_t m, int64_t n, int32_t r, int32_t d, hipStream_t st);
// Device-side plan build (plan_device.hip): the bytes of build_plan_host, from kernels on `st`; workspace of
// plan_build_workspace_bytes(); status_out (device, may be null) receives LSP_OK / LSP_ERR_INDEX / LSP_ERR_SKEW.
size_t     plan_build_workspace_bytes(int64_t m, int64_t n, int32_t r, int32_t d);
// with_tiles: false for a plan that the bf16 kernel will not follow.
// zero: r x r floats to set to zero if there is no plan to be made of these projectors.
hipError_t launch_plan_build(const int32_t* P_idx, const float* P_val, const int32_t* Q_idx, const float* Q_val,
                             int64_t m, int64_t n, int32_t r, int32_t d, uint8_t* plan, uint8_t* workspace,
                             int32_t* status_out, hipStream_t st, bool with_tiles = true, float* zero = nullptr);
// C = op(A) op(B) + beta E on r x r fp32 matrices (matrix cores): up to kMaxGemmBatch independent products of
// one size in a launch (no product may read what another of the same launch writes).  flags: transpose an
// operand (not both), square an operand element by element; E may be null.
constexpr int kMaxGemmBatch = 3;
constexpr int kGemmTA = 1, kGemmTB = 2, kGemmSqA = 4, kGemmSqB = 8;
struct GemmProblem { const float* A; const float* B; float* C; const float* E; float beta; int32_t flags; float* Ct; int32_t pad[4]; };   // Ct: a transposed copy of C, may be null
struct GemmBatch { int32_t r, pad[15]; GemmProblem p[kMaxGemmBatch]; };   // (r: the launcher fills it in)
static_assert(sizeof(GemmProblem) == 64, "a record, loaded whole");
hipError_t launch_gemm_rr_batch(const GemmBatch& batch, int count, int32_t r, hipStream_t st);
// C = L^T R (r x r, overwritten) for two ELL matrices with the same number of rows; one or two independent
// pairs per launch.
struct GramPair { const int32_t* L_idx; const float* L_val; const int32_t* R_idx; const float* R_val; int64_t rows; float* C; int32_t pad[4]; };
struct GramBatch { GramPair p[2]; };
// `clear` (may be null): floats to set to zero if the plan cuts rows of P^T into pieces.
struct GramClear { const uint8_t* plan; float* p; int64_t count; };
hipError_t launch_gram(const GramBatch& batch, int count, int32_t d, int32_t r, const GramClear* clear, hipStream_t st);
// Gradient of 1/2 ||P P^T G Q Q^T - G||_F^2 with respect to the stored projector values (fitgrad.hip).
size_t     fitgrad_workspace_floats(int64_t m, int64_t n, int32_t r, int32_t d);
hipError_t launch_fitgrad(const void* G, const uint8_t* plan, const int32_t* P_idx, const float* P_val,
                          const int32_t* Q_idx, const float* Q_val, int64_t m, int64_t n, int32_t r, int32_t d,
                          float* gP, float* gQ, float* workspace, lsp_dtype dtype, hipStream_t st);

// ------------------------------------------------------------------------------------------
// Storage types on the device.
// ------------------------------------------------------------------------------------------
struct F32 { using elem = float;    static constexpr int size = 4; };
struct F16 { using elem = uint16_t; static constexpr int size = 2; };
struct BF16{ using elem = uint16_t; static constexpr int size = 2; };

#if defined(__HIPCC__)
// Lets kernel `Kern` use up to `Bytes` of dynamic LDS: the most that any launch of it asks for, a constant, so that it does not depend on which
// call comes first.  The attribute belongs to the (kernel, device) pair and does not change afterwards, so the runtime is asked once per pair,
// not on every launch of the per-step path.
template <auto Kern, size_t Bytes>
static inline hipError_t allow_dynamic_lds() {
    static_assert(Bytes <= 160 * 1024, "the LDS of a CU");
    static std::atomic<uint64_t> done{0};                   // bit k: set on device k (devices >= 64: always asked)
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 64 && ((done.load(std::memory_order_acquire) >> dev) & 1u)) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(Kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)Bytes);
    if (e == hipSuccess && dev < 64) done.fetch_or((uint64_t)1 << dev, std::memory_order_release);
    return e;
}

// Streaming accesses to the big matrices (each byte of G and W is touched once per call): marked
// non-temporal so that they do not evict the small, heavily re-read operands (S, the projector
// arrays, the plan) from the XCD's L2.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <typename V> __device__ __forceinline__ V stream_load(const V* p) {
    static_assert(sizeof(V) == 4 || sizeof(V) == 8 || sizeof(V) == 16, "4, 8 or 16 bytes");
    V out;
    if constexpr (sizeof(V) == 4) { uint32_t t = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p)); __builtin_memcpy(&out, &t, 4); }
    else if constexpr (sizeof(V) == 8) { u32x2 t = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p)); __builtin_memcpy(&out, &t, 8); }
    else { u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); __builtin_memcpy(&out, &t, 16); }
    return out;
}

typedef const LSP_CONST_AS PlanHeader* PlanHeaderPtr;
// A plan's header, loaded at once.  (The offsets in it are followed only when plan_matches says that it is this problem's.)
struct LoadedHeader {
    PlanHeader h;
    __device__ __forceinline__ const PlanHeader* operator->() const { return &h; }
};
__device__ __forceinline__ LoadedHeader load_header(const uint8_t* plan) {
    const auto* p = as_const<uint32_t>(plan);
    words16 a = scalar_load<words16>(p), b = scalar_load<words16>(p, 16), c = scalar_load<words16>(p, 32);
    words4 e = scalar_load<words4>(p, 48);
    words2 f = scalar_load<words2>(p, 52);
    arrived(a, b, c, e, f);
    LoadedHeader H;
    char* o = reinterpret_cast<char*>(&H.h);
    __builtin_memcpy(o, &a, 64); __builtin_memcpy(o + 64, &b, 64); __builtin_memcpy(o + 128, &c, 64); __builtin_memcpy(o + 192, &e, 16); __builtin_memcpy(o + 208, &f, 8);
    return H;
}

// Whether a header names this problem.  (One condition and no chain of them: each would wait for the one before.)
__device__ __forceinline__ bool same_problem(uint32_t magic, int32_t hm, int32_t hn, int32_t hr, int32_t hd, int m, int n, int r, int d) {
    return ((magic ^ kPlanMagic) | (uint32_t)(hm ^ m) | (uint32_t)(hn ^ n) | (uint32_t)(hr ^ r) | (uint32_t)(hd ^ d)) == 0;
}

template <typename D> __device__ __forceinline__ float widen(typename D::elem x);
template <> __device__ __forceinline__ float widen<F32>(float x) { return x; }
template <> __device__ __forceinline__ float widen<F16>(uint16_t x) {
    _Float16 h; __builtin_memcpy(&h, &x, 2); return (float)h;
}
template <> __device__ __forceinline__ float widen<BF16>(uint16_t x) {
    return __uint_as_float(((uint32_t)x) << 16);
}
template <typename D> __device__ __forceinline__ typename D::elem narrow(float x);
template <> __device__ __forceinline__ float narrow<F32>(float x) { return x; }
template <> __device__ __forceinline__ uint16_t narrow<F16>(float x) {
    _Float16 h = (_Float16)x; uint16_t u; __builtin_memcpy(&u, &h, 2); return u;   // nearest-even
}
template <> __device__ __forceinline__ uint16_t narrow<BF16>(float x) {
    __bf16 h = (__bf16)x; uint16_t u; __builtin_memcpy(&u, &h, 2); return u;       // nearest-even
}
#endif

}  // namespace lsp
