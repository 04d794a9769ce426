// Internal declarations shared by the translation units of libturborag_hip.so.
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <stddef.h>
#include <vector>

#include "../../include/turborag.h"

// ---- error plumbing -------------------------------------------------------------------------------------
int tr_fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void tr_clear_error();
#define TR_HIP(expr)                                                                           \
    do {                                                                                       \
        hipError_t e__ = (expr);                                                               \
        if (e__ != hipSuccess) return tr_fail(TR_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e__)); \
    } while (0)

// A kernel that needs more dynamic LDS than the default limit has the limit raised once per device: the attribute
// belongs to the function on the device that is current, so a process that uses a second device must set it there
// too.  `done` holds one bit per device ordinal (mod 64) and is safe to race on: the worst case sets it twice.
static inline int tr_raise_lds_limit(const void* kernel, int bytes, std::atomic<uint64_t>* done)
{
    int dev = 0;
    TR_HIP(hipGetDevice(&dev));
    const uint64_t bit = 1ull << (dev & 63);
    if (!(done->load(std::memory_order_acquire) & bit)) {
        TR_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
        done->fetch_or(bit, std::memory_order_release);
    }
    return TR_OK;
}

int tr_check_shape(const tr_shape* s);
static inline int tr_elem_bytes(const tr_shape* s) { return s->dtype == TR_F32 ? 4 : 2; }
static inline size_t tr_align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct tr_store {
    tr_shape shape;
    const void* k;
    const void* v;
    std::vector<int64_t> row_start; // n_chunks + 1
};

// ---- launch-policy overrides (tr_set_tuning) --------------------------------------------------------------------
// The library reads no environment variable.  Tests and sweeps override a policy value through tr_set_tuning();
// tr_knob() returns the override, or dflt when none is set (0 = not set).
enum TrKnob {
    TR_KNOB_WG_ROWS,        // packed rows per attention workgroup: 32, 128 or 256
    TR_KNOB_TARGET_ITEMS,   // workgroups a single request's key split aims for
    TR_KNOB_MIN_SPLIT_KEYS, // shortest key split
    TR_KNOB_ASM_SPAN,       // 16-byte units of K (and V) per assemble workgroup
    TR_KNOB_BD_PIECE_TILES, // key tiles per piece when the one-pass kernel cuts a long key range
    TR_KNOB_BD_SLOTS,       // resident workgroups the one-pass planner balances for
    TR_KNOB_LIN_SPLIT,      // slices of k in tr_linear
    TR_KNOB_LIN_MSPLIT,     // 1: never split the rows of x over two workgroups
    TR_KNOB_COUNT
};
int tr_knob(int which, int dflt);

// ---- the chip the launch planners are written for (MI355X, gfx950) ------------------------------------------------
// One table instead of constants scattered over the planners.  The *_US and *_PER_US figures are measured on that
// part and only steer how work is cut; no result depends on them.
struct TrChip {
    static constexpr int XCDS = 8;                 // accelerator dies; blocks are dealt to them round-robin
    static constexpr int CUS = 256;                // compute units, 32 per XCD
    static constexpr int SLOTS_128 = 512;          // resident 128-row attention workgroups (two per CU)
    static constexpr int SLOTS_256 = 256;          // resident 256-row attention workgroups (one per CU)
    static constexpr double KEY_TILE_STEP_US = 2.0;        // one 64-key step of a resident attention workgroup
    static constexpr double WORKGROUP_FIXED_STEPS = 3.0;   // prologue + epilogue of a workgroup, in such steps
    static constexpr double PARTIAL_BYTES_PER_US = 2.0e6;  // split partials, written and read back: ~4 TB/s for both
};

// theta_m = base^(-2m/d) in double (text after Eq. 3)
void tr_fill_theta(const tr_shape* s, double* theta /*[64]*/);

// Sine and cosine of a rotation angle, a position id times a theta of at most 1, in fp64.  A thread of the rotation kernels works
// out one or a few angles and everything it stores waits for them, so the length of the dependent chain counts.  The angle is
// reduced by multiples of pi/2 in two parts; the fused product with the first is exact for every quotient of 31 bits, and so
// is the difference.  What the second step rounds off is carried to the end, as is what 1 - z/2 rounds off.  At most pi/4 is
// left, where both functions are their Taylor polynomials with first terms left out of less than 2.1e-18.
// Largest error (root of mean squares) over 10^5 angles each up to 1, 100, 32768, 1e6 and 2^31: 8.2 .. 8.5e-17 (2.8e-17), the library's
// function 8.3 .. 8.5e-17 (2.8e-17).  6200 rows of un-rotated keys and 37 query tokens: 28.4 -> 28.0 us.
__device__ __forceinline__ void tr_sincos(double angle, double* sine, double* cosine)
{
    const double q = rint(angle * 0.6366197723675814);      // 2 / pi
    const double r1 = fma(-q, 1.5707963267948966, angle);   // pi / 2 = 1.5707963267948966 + 6.123233995736766e-17
    const double r = fma(-q, 6.123233995736766e-17, r1);
    const double t = fma(-q, 6.123233995736766e-17, r1 - r); // the angle is r + t
    const double z = r * r;
    double s = 1.0 / 355687428096000.0, c = 1.0 / 20922789888000.0; // 1 / 17!, 1 / 16!
    s = fma(s, z, -1.0 / 1307674368000.0);
    c = fma(c, z, -1.0 / 87178291200.0);
    s = fma(s, z, 1.0 / 6227020800.0);
    c = fma(c, z, 1.0 / 479001600.0);
    s = fma(s, z, -1.0 / 39916800.0);
    c = fma(c, z, -1.0 / 3628800.0);
    s = fma(s, z, 1.0 / 362880.0);
    c = fma(c, z, 1.0 / 40320.0);
    s = fma(s, z, -1.0 / 5040.0);
    c = fma(c, z, -1.0 / 720.0);
    s = fma(s, z, 1.0 / 120.0);
    c = fma(c, z, 1.0 / 24.0);
    s = fma(s, z, -1.0 / 6.0);
    s = r + fma(r * z, s, fma(-0.5 * z, t, t));             // sin(r + t) = sin r + t cos r
    const double w = fma(-0.5, z, 1.0);
    c = w + fma(z * z, c, fma(-0.5, z, 1.0 - w) - r * t);   // cos(r + t) = cos r - t sin r
    const int n = (int)q; // quadrant
    const double a = (n & 1) ? c : s, b = (n & 1) ? s : c;
    *sine = (n & 2) ? -a : a;
    *cosine = ((n + 1) & 2) ? -b : b;
}

// Divisor of the attention kernels' packed rows by the heads of a GQA group (x * magic >> 16 = x / group for x < 256; a larger
// group does not fit a row tile).
static inline int32_t tr_group_magic(int32_t group) { return (65536 + group - 1) / group; }

// ---- kernel argument blocks (passed by value; each stays below 4 KB of kernarg) ------------------------------

// One contiguous run of rows to move: src rows [src_row, src_row+n_rows) -> dst rows [dst_row, ...),
// keys additionally turned by delta positions (0: plain copy).
struct TrCopyDesc {
    int32_t src_row;
    int32_t dst_row;
    int32_t n_rows;
    int32_t delta;
    int32_t blk_start; // first block of the grid that works on this run
};
// Index of the last of n ascending entries that is <= x, for a wave-uniform x >= first(0): every lane looks at its own
// entry and a ballot counts.  One trip to the argument block, where a search takes one for every step, some hundred
// nanoseconds each, before a workgroup knows what to load (64 decode requests: six).  Every lane must be active.
template <class First> __device__ __forceinline__ int last_not_above(int n, int x, First first)
{
    if (n == 1) return 0;
    const int lane = threadIdx.x & 63;
    int count = 0;
    for (int i0 = 0; i0 < n; i0 += 64) count += __popcll(__ballot(i0 + lane < n && first(min(i0 + lane, n - 1)) <= x));
    return count - 1;
}

// Query append: a token's row is walked by groups of half_dim = head_dim / 2 lanes (a lane per pair of a head), each of which
// owns TR_APPEND_UNITS 16-byte units per lane; four waves to a workgroup.
#define TR_APPEND_UNITS 2
#define TR_APPEND_WAVES_PER_BLOCK 4
__host__ __device__ static inline int tr_append_shift(int half_dim) { return half_dim == 64 ? 6 : 5; }
__host__ __device__ static inline int tr_append_groups(int row_units, int half_dim)
{
    const int shift = tr_append_shift(half_dim) + 1;
    static_assert(TR_APPEND_UNITS == 2, "");
    return (row_units + (1 << shift) - 1) >> shift;
}
static inline int64_t tr_append_blocks(int64_t tokens, int row_units, int half_dim)
{
    const int per_block = 64 / half_dim * TR_APPEND_WAVES_PER_BLOCK;
    return (tokens * tr_append_groups(row_units, half_dim) + per_block - 1) / per_block;
}
// A launch has fewer than 2^32 threads.  More groups than this (at most 2^31 threads) are appended by several launches, and
// blocks of 256 threads beyond that count are never put into one.
#define TR_MAX_APPEND_TOKENS (1 << 25) // of one group each
#define TR_MAX_BLOCKS_256 ((1 << 24) - 1)
#define TR_MAX_COPY_DESC 168 // what the 4 KB argument block holds
// optional tail of an assemble launch: one request's query tokens appended by the blocks from first_block on
struct TrAppendTail {
    const void* k_new;
    const void* v_new;
    const int32_t* q_pos;
    int32_t n_q; // 0: no tail
    int32_t dst_row0;
    int32_t first_block;
    int32_t pad_;
};
struct TrAssembleArgs {
    const void* k_src;
    const void* v_src;
    void* k_dst;
    void* v_dst;
    int32_t n_desc;
    int32_t row_units;  // 16-byte units per row (n_kv_heads * head_dim * elem / 16)
    int32_t head_units; // 16-byte units per head
    int32_t span_units; // units of K (and of V) one block moves; multiple of 256
    int32_t half_dim;   // head_dim / 2
    int32_t rope_half;  // 1: pairs are (m, m + d/2) instead of (2m, 2m+1)
    int64_t formed_bytes; // of K and V, over all launches of the call: decides how they are stored
    double theta[64];
    TrAppendTail app;
    TrCopyDesc desc[TR_MAX_COPY_DESC];
};

// append: request r's tokens [q_row0, q_row0+n_q) go to cache rows [dst_row0, dst_row0+n_q)
struct TrAppendDesc {
    int32_t q_row0;
    int32_t n_q;
    int32_t dst_row0;
    int32_t pos0; // position id of the first token when the launch carries no q_pos array (raw-store assembly)
};
#define TR_MAX_APPEND_DESC 128
struct TrAppendArgs {
    const void* k_new;
    const void* v_new;
    const int32_t* q_pos;
    void* cache_k;
    void* cache_v;
    int32_t n_desc;
    int32_t n_kv_heads;
    int32_t head_dim;
    int32_t total_tokens; // tokens covered by this launch (sum of n_q)
    int32_t rope_half;
    int32_t pad_;
    double theta[64];
    TrAppendDesc desc[TR_MAX_APPEND_DESC];
    int32_t tok0[TR_MAX_APPEND_DESC]; // first token of each run among the launch's tokens
};

// prefix attention: one request
struct TrSeqDesc {
    int32_t q_row0;    // first packed query token of the request (row of q / out / q_pos)
    int32_t n_q;
    int32_t kv_row0;   // first cache row of the request
    int32_t kv_len;
    int32_t item0;     // first work item of the request in this launch
    int32_t n_tiles;   // row tiles
    int32_t n_split;   // KV splits (>= 1)
    int32_t split_len; // keys per split, multiple of the key tile
    int32_t ws_row0;   // first partial row of the request in the workspace
    uint32_t split_magic; // 2^32 / n_split + 1 for n_split > 1: x / n_split is the high half of x * split_magic (x n_split < 2^32)
};
#define TR_MAX_SEQ 64
struct TrPrefixArgs {
    const void* q;
    const void* k;
    const void* v;
    const int32_t* q_pos;
    void* out;
    _Float16* ws_o; // [partial rows][head_dim] partial outputs, each normalised by its own denominator; fp32 where partial_f32
    float* ws_ml; // [partial rows][2] reference maximum (log2 domain) and softmax denominator
    int32_t n_seq;
    int32_t n_items;
    int32_t n_q_heads;
    int32_t n_kv_heads;
    int32_t group;
    int32_t tok_per_tile;
    float scale_log2e; // log2(e) / sqrt(head_dim)
    float scale;       // 1 / sqrt(head_dim)
    int32_t rope_half;
    int32_t group_magic; // tr_group_magic(group)
    int32_t partial_f32; // short-query kernel and its merge: ws_o holds fp32
    int32_t pad_;
    double theta_rev[64]; // theta_m / (2 pi): position * theta_rev = angle in revolutions
    double theta[64];
    TrSeqDesc seq[TR_MAX_SEQ];
};

// gather attention: the keys of one request, read where they lie.  A segment is one retrieved chunk in the store
// (rows src_row .. +n_rows, keys stored at chunk-local positions, delta = the chunk's offset under reordered
// positions, else 0), or, last, the request's own query tokens in its cache (delta 0).
struct TrGatherSeg {
    int32_t src_row;
    int32_t n_rows;
    int32_t delta;
    int32_t tile0;     // first 64-key tile of the segment in the request's tile list
    int32_t cache_row; // cache row its first key would have after assembly
};
#define TR_MAX_GATHER_SEG 96
struct TrGatherArgs {
    const void* q;
    const void* k_store;
    const void* v_store;
    const void* k_cache;
    const void* v_cache;
    const int32_t* q_pos;
    void* out;
    _Float16* ws_o;
    float* ws_ml;
    int32_t n_q;
    int32_t n_doc;
    int32_t n_seg;           // segments, the query-token segment included (it is the last)
    int32_t n_tiles_total;
    int32_t n_split;
    int32_t tiles_per_split;
    int32_t row_tiles;
    int32_t n_items;
    int32_t n_q_heads;
    int32_t n_kv_heads;
    int32_t group;
    int32_t tok_per_tile;
    float scale_log2e;
    int32_t rope_half;
    int32_t group_magic;
    int32_t pad_;
    double theta_rev[64];
    TrGatherSeg seg[TR_MAX_GATHER_SEG];
};

// A run of consecutive row tiles of the block-diagonal kernel that share one split count.  Items of a KV head are
// numbered segment by segment, tiles in DESCENDING order inside a segment, the splits of a tile next to each other.
struct TrBdSeg {
    int32_t tile_hi;   // last (highest) row tile of the segment: the first one issued
    int32_t n_tiles;
    int32_t n_split;   // pieces the key walk of each tile is cut into (>= 1)
    int32_t split_len; // keys per piece, a multiple of 64; the last piece runs to the end of the walk
    int32_t item0;     // first item of the segment inside a KV head's item list
    int32_t ws_row0;   // first partial row of the segment (n_split > 1)
    int32_t tok0;      // first token of the segment
    int32_t n_tok;     // tokens in the segment
};
#define TR_MAX_BD_SEG 64
struct TrBlockDiagArgs {
    const void* q;
    const void* k; // rotated keys K'
    const void* v;
    const int32_t* tok_start; // [T] first row each token may attend (the start of its chunk)
    const int32_t* pos;       // [T] RoPE position ids, or NULL: position = t - tok_start[t]
    void* out;
    int32_t total_tokens;
    int32_t n_tiles;
    int32_t n_q_heads;
    int32_t n_kv_heads;
    int32_t group;
    int32_t tok_per_tile;
    float scale_log2e;
    float scale;
    int32_t rope_half;
    int32_t n_seg;
    int32_t items_per_head;
    int32_t group_magic;
    _Float16* ws_o; // partial outputs and statistics of split tiles, laid out as in TrPrefixArgs
    float* ws_ml;
    double theta_rev[64];
    double theta[64];
    TrBdSeg seg[TR_MAX_BD_SEG];
};

static_assert(sizeof(TrAssembleArgs) <= 4096 && sizeof(TrAppendArgs) <= 4096 && sizeof(TrPrefixArgs) <= 4096 &&
                  sizeof(TrGatherArgs) <= 4096 && sizeof(TrBlockDiagArgs) <= 4096,
              "kernel argument blocks must fit the 4 KB kernarg segment");

// ---- launchers implemented in the .hip files --------------------------------------------------------------
int tr_launch_assemble(const TrAssembleArgs& a, int dtype, int n_blocks, hipStream_t s);
int tr_launch_append(const TrAppendArgs& a, int dtype, hipStream_t s);
int tr_launch_prefix_attn(const TrPrefixArgs& a, int head_dim, int wg_rows, bool any_split, int total_rows, hipStream_t s);
int tr_launch_prefix_attn_f32(const TrPrefixArgs& a, int head_dim, int total_rows, hipStream_t s);
int tr_launch_rope_table(double* table, int n_pos, int half_dim, const double* theta, hipStream_t s);
// table == NULL: the kernel works out the angles itself; table_rows bounds the positions either way
int tr_launch_rope_rows(const void* k, void* k_rot, const int32_t* cu, int n_chunks, int max_chunk_len, int32_t* tok_start,
                        const double* table, int table_rows, int64_t total_tokens, const tr_shape* shape, hipStream_t s);
static inline int tr_rope_half(const tr_shape* s) { return s->rope_layout == TR_ROPE_HALF ? 1 : 0; }
// combine: NULL, or the arguments of the merge over the split tiles' tokens (combine_rows = tokens x query heads)
int tr_launch_blockdiag_attn(const TrBlockDiagArgs& a, const TrPrefixArgs* combine, int combine_rows, int head_dim, int wg_rows,
                             hipStream_t s);
int tr_launch_gather_attn(const TrGatherArgs& a, const TrPrefixArgs& combine_args, int head_dim, hipStream_t s);
// longest: most keys that a row sees, as far as the host knows it; it decides how a row is shared out, not the result
int tr_launch_blockdiag_attn_f32(const TrBlockDiagArgs& a, int64_t longest, int head_dim, hipStream_t s);
// y_j = x w_j^T for at most 128 rows of x and up to TR_LINEAR_MAX_OUT weights that share x; N = sum of the feature
// counts; partial: fp32 [tr_linear_splits(M, N, K), M, N] when that count exceeds 1
#define TR_LINEAR_MAX_OUT 4
int tr_linear_splits(int32_t M, int32_t N, int32_t K);
// Which kernel a product takes under the overrides in force, for tests: 16 xb + wb where workgroups keep all of k for a tile of
// 16 xb rows of x by 16 wb features, 0 where k is cut into slices.  Not part of the public interface.
extern "C" int tr_linear_direct_tile(int32_t M, int32_t N, int32_t K);
// sink: 256 * 512 floats.  *flops receives the multiply-add count x 2 of the launch.
int tr_launch_mfma_loop_probe(int iters, int random_operands, float* sink, hipStream_t s, double* flops);
int tr_launch_linear(const void* x, int32_t n_out, const void* const* w, void* const* y, const int32_t* n_features, void* partial,
                     int32_t M, int32_t K, hipStream_t s);
