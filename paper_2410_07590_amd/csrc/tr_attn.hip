// bf16 MFMA attention kernels for gfx950: query prefill over an assembled cache (Sec. 3.4 step 6) and the
// offline block-diagonal chunk prefill (Sec. 3.4 step 2, independent attention of Sec. 3.2).
//
// Work decomposition.  A "packed row" is one (query token, query head of a GQA group) pair: the g query heads
// that share a KV head are stacked along the MFMA M dimension, so one K/V tile fetched from HBM serves all of
// them.  A workgroup of NW wavefronts owns 32*NW packed rows of one KV head; each wavefront owns 32 rows and
// walks the visible keys in tiles of 64.
//
// Transposed products.  S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16: A = K rows / V^T rows
// from LDS, B = rotated queries / P^T from registers.  Each lane then owns ONE query column, so the softmax
// statistics are per-lane scalars, and the S^T accumulator layout already is the B-operand layout of the
// second product, up to a permutation of the 16 keys inside a k-step that the V^T reads apply as well.
// V^T operands come from row-major V tiles through the transposing LDS read (ds_read_b64_tr_b16).
//
// Data movement.  K/V tiles go global -> LDS directly (global_load_lds_dwordx4, no staging registers) into a
// ring of NS stages; rows are stored unpadded and XOR-swizzled per 16-byte chunk so that the MFMA operand
// reads are bank-conflict free.  One s_barrier per tile; s_waitcnt vmcnt counts are managed by hand because
// the loads are asynchronous with respect to the wave that issued them.
//
// Softmax works in the log2 domain with a lazily updated reference maximum: the accumulators are rescaled
// only when the running maximum grew by more than 2^8, which is exact (softmax is invariant to the reference)
// and keeps P <= 256.
#include "tr_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

#define LDS_AS __attribute__((address_space(3)))
#define GLB_AS __attribute__((address_space(1)))

constexpr int KT = 64;               // keys per tile
constexpr float RESCALE_SLACK = 8.f; // log2 units a tile maximum may exceed the reference before a rescale
constexpr int K_PREFETCH = 2;        // k-steps the K operand reads run ahead of the score products
constexpr float REREF_BELOW = -32.f; // a row's first visible tile re-references when its maximum is below this

template <int D> struct Geo {
    static constexpr int CPR = D / 8;            // 16-byte chunks per row of one head
    static constexpr int RPI = 64 / CPR;         // rows moved by one wave-wide 1 KB load
    static constexpr int NI = KT / RPI;          // such loads per K (or V) tile
    static constexpr int TILE_BYTES = KT * D * 2;
    static constexpr int STAGE_BYTES = 2 * TILE_BYTES; // one K tile and one V tile
    static constexpr int GPR = CPR / 4;          // 64-byte groups per row
    // K: chunk c of row r sits at chunk c ^ kswz(r): 16 consecutive rows of one logical chunk cover all banks
    __device__ static __forceinline__ int kswz(int r) { return (r / (16 / CPR)) & (CPR - 1); }
    // V: 64-byte group q of row r sits at group q ^ vswz(r): 4 consecutive rows of one group cover all banks
    __device__ static __forceinline__ int vswz(int r) { return (r / (4 / GPR)) & (GPR - 1); }
};

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
template <int N> __device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(vmcnt_imm(N)); }

// Waits until this wave's LDS reads have delivered: what they read may be overwritten behind it.
__device__ __forceinline__ void wait_lds()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

struct RowCtx {
    bool valid;
    int orow;    // q_tok * n_q_heads + head: row of q / out in units of head vectors
    int key_lo;  // first visible cache row
    int key_hi;  // last visible cache row
};

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// x / g for the rows of a workgroup (x < 256, g <= 256): exact, as x * (tr_group_magic(g) * g - 2^16) < 2^16.  A division by a
// number that is not known when the code is compiled takes some twenty instructions, and a wave's rows ask for five.
__device__ __forceinline__ int by_group(int x, int magic) { return (int)(((uint32_t)x * (uint32_t)magic) >> 16); }

__device__ __forceinline__ int xcd_remap(int bid, int n)
{
    // Blocks are dealt round-robin to the 8 XCDs; give each XCD one contiguous range of items so that
    // items sharing K/V tiles meet in the same L2.
    const int x = bid & 7, idx = bid >> 3;
    const int q = n >> 3, r = n & 7;
    return x * q + (x < r ? x : r) + idx;
}

// Maximum and sum over the two lanes c and c + 32, which hold the two key halves of one query column, through the
// cross-half swap of the vector unit.  These exchanges sit on the critical path of every tile: an LDS permute would put
// an LDS round trip there, and its wait would also wait for every operand read in flight.
// permlane32_swap(u, u): result[0] = lanes 0..31 of u in both halves, result[1] = lanes 32..63 of u in both halves.
__device__ __forceinline__ float column_max(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float column_sum(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Maximum / minimum of an int over the wave, as a uniform value.  Four cross-lane steps inside each row of 16 lanes on
// the vector unit's data-parallel path (pairs, quads, the mirrored half-row, the mirrored row: max and min do not care
// which lanes meet, only that all do), then the four rows' results through scalar registers.  Every lane of the wave must
// be active.  (A butterfly of six LDS permutes does the same with six dependent LDS round trips; a workgroup of the
// offline kernel needs four such reductions before its first tile load can go out.)
template <bool MAX> __device__ __forceinline__ int wave_reduce_i(int v)
{
    auto op = [](int a, int b) { return MAX ? max(a, b) : min(a, b); };
    v = op(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, false));  // quad_perm [1,0,3,2]
    v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, false));  // quad_perm [2,3,0,1]
    v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false)); // row_half_mirror
    v = op(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false)); // row_mirror
    const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    return op(op(r0, r1), op(r2, r3));
}
__device__ __forceinline__ int wave_max_i(int v) { return wave_reduce_i<true>(v); }
__device__ __forceinline__ int wave_min_i(int v) { return wave_reduce_i<false>(v); }

// ---- rotated queries (Eq. 3 at the token's position id) -------------------------------------------------------
// Lane (c = lane & 31, h = lane >> 5) ends up holding Q'[row c][16 ks + 8 h .. +7] for ks < D/16, scaled by
// log2(e)/sqrt(d) before its single rounding to bf16.  Angles are reduced in fp64 to [-1/2, 1/2] revolutions and
// then go through v_sin/v_cos, which take revolutions.

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int ROT_SLOTS = 8; // token slots per rotation pass; covers a wave's 32 packed rows when the GQA group is >= 4

// theta_rev[m] of a kernel whose one argument is an Args block, by a load that is issued where it stands.  A plain load of an
// argument is free to move, and did: to its first use, behind the tile loads, with which it was then waited for.
template <class Args> __device__ __forceinline__ double load_theta(int m)
{
    uintptr_t args = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    return ((const GLB_AS double*)(args + offsetof(Args, theta_rev)))[m];
}

// Issue the loads of this lane's raw fragments; rows that do not exist read row 0 and are zeroed later.
template <int D>
__device__ __forceinline__ void load_q_raw(const __bf16* __restrict__ q, const RowCtx& rc, int h, u32x4 (&raw)[D / 16])
{
    const __bf16* qrow = q + (int64_t)(rc.valid ? rc.orow : 0) * D + 8 * h;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) raw[ks] = *(const u32x4*)(qrow + 16 * ks);
}

// cn, sn: cosine and sine of the pair's angle, already multiplied by the score scale.  Rows that do not exist are
// rotated like any other (they hold row 0's values and are never stored).
__device__ __forceinline__ void rot_pair(uint32_t w, float cn, float sn, bf16x8& f, int p)
{
    const float xa = bf_lo(w), xb = bf_hi(w);
    f[2 * p] = (__bf16)(xa * cn - xb * sn);
    f[2 * p + 1] = (__bf16)(xb * cn + xa * sn);
}

// The g query heads of a token share its angles, so a wave's 32 rows need at most ROT_SLOTS x D/2 distinct
// (cos, sin) pairs instead of 32 x D/2: the wave computes them once into a private LDS table, lane -> pair index,
// one token slot (two for D = 64) per step.  pos_lane: position id of slot (lane & 7).
// Table layout: slot j, pair m at byte j * 4 D + (((m >> 1) ^ 2 j) * 16) + (m & 1) * 8.
template <int D>
__device__ __forceinline__ void build_rot_table(LDS_AS char* tab, double th /* theta_rev[lane % (D/2)] */, int lane, int pos_lane,
                                                float sl2e /* log2(e) / sqrt(d): folded into the table */)
{
    constexpr int PAIRS = D / 2, LPS = 64 / PAIRS;
    const int m = lane % PAIRS;
#pragma unroll
    for (int pass = 0; pass < ROT_SLOTS / LPS; ++pass) {
        const int j = pass * LPS + lane / PAIRS;
        int pos = __builtin_amdgcn_readlane(pos_lane, pass * LPS);
        if (LPS == 2) pos = lane < PAIRS ? pos : __builtin_amdgcn_readlane(pos_lane, pass * LPS + 1);
        double rev = (double)pos * th;
        rev -= rint(rev);
        const float x = (float)rev;
        f32x2 cs;
        cs[0] = __builtin_amdgcn_cosf(x) * sl2e;
        cs[1] = __builtin_amdgcn_sinf(x) * sl2e;
        *(LDS_AS f32x2*)(tab + j * (4 * D) + (((m >> 1) ^ (2 * j)) * 16) + (m & 1) * 8) = cs;
    }
}

template <int D>
__device__ __forceinline__ void rotate_q_shared(const u32x4 (&raw)[D / 16], LDS_AS const char* tab, int slot, int h,
                                                bf16x8 (&qf)[D / 16])
{
    LDS_AS const char* row = tab + slot * (4 * D);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        // pairs 8 ks + 4 h .. +3 = 16-byte chunks 2 u, 2 u + 1 with u = 2 ks + h
        const int ch = (2 * (2 * ks + h)) ^ (2 * slot);
        const f32x4 cs0 = *(LDS_AS const f32x4*)(row + ch * 16);
        const f32x4 cs1 = *(LDS_AS const f32x4*)(row + ch * 16 + 16);
        bf16x8 f;
        rot_pair(raw[ks][0], cs0[0], cs0[1], f, 0);
        rot_pair(raw[ks][1], cs0[2], cs0[3], f, 1);
        rot_pair(raw[ks][2], cs1[0], cs1[1], f, 2);
        rot_pair(raw[ks][3], cs1[2], cs1[3], f, 3);
        qf[ks] = f;
    }
}

// Half-split layout: channel c < D/2 pairs with c + D/2, i.e. fragment ks (channels 16 ks + 8 h .. +7) pairs element by
// element with fragment ks + D/32, and the pair index of element e is 16 ks + 8 h + e.  row: the token slot's table
// row, sw: twice the slot (the swizzle of its 16-byte chunks).
template <int D>
__device__ __forceinline__ void rot_frag_half(const u32x4& lo, const u32x4& hi, LDS_AS const char* row, int ks, int h, int sw,
                                              bf16x8& flo, bf16x8& fhi)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) { // two pairs (one 16-byte table chunk) at a time
        const int ch = (8 * ks + 4 * h + q) ^ sw;
        const f32x4 cs = *(LDS_AS const f32x4*)(row + ch * 16);
        const float la = bf_lo(lo[q]), lb = bf_hi(lo[q]);
        const float ha = bf_lo(hi[q]), hb = bf_hi(hi[q]);
        flo[2 * q] = (__bf16)(la * cs[0] - ha * cs[1]);
        fhi[2 * q] = (__bf16)(ha * cs[0] + la * cs[1]);
        flo[2 * q + 1] = (__bf16)(lb * cs[2] - hb * cs[3]);
        fhi[2 * q + 1] = (__bf16)(hb * cs[2] + lb * cs[3]);
    }
}

template <int D>
__device__ __forceinline__ void rotate_q_shared_half(const u32x4 (&raw)[D / 16], LDS_AS const char* tab, int slot, int h,
                                                     bf16x8 (&qf)[D / 16])
{
    LDS_AS const char* row = tab + slot * (4 * D);
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) rot_frag_half<D>(raw[ks], raw[ks + D / 32], row, ks, h, 2 * slot, qf[ks], qf[ks + D / 32]);
}

// Rotated, scaled queries of a wave from their raw fragments.  slot: which of the wave's tokens this lane's row
// belongs to (0 .. n_slots-1, n_slots wave-uniform); pos_of_slot(s): position id of the wave's token slot s (any
// value for slots past the wave's last token).  Tokens go through the table ROT_SLOTS at a time: one pass when the
// GQA group is >= 4, up to four for smaller groups.
// LATER: vector-memory loads that this wave has issued behind the raw rows.  With a tile load in flight the compiler would
// wait for everything before it touches a loaded register, so the waits by count are written out: theta and the position ids
// (in front of the rows) first, the rows once the table is built.
// (us before / after, with the table's position ids from scalar lanes instead of an LDS permute each and the divisions by the
// group as products: one token for each of 64 requests of 4096 rows 95.5 / 94.1, for 5 ragged ones 18.5 / 17.8; 64 x 512
// offline tokens 283 / 276, one pass over 32 x 1024 + 256 tokens 536 / 528.)
template <int D, bool HALF, int LATER, class PosFn>
__device__ __forceinline__ void rotate_queries(u32x4 (&raw)[D / 16], LDS_AS char* tab, double th, int pos_lane, int lane, int h,
                                               int slot, int n_slots, float sl2e, PosFn pos_of_slot, bf16x8 (&qf)[D / 16])
{
    n_slots = __builtin_amdgcn_readfirstlane(n_slots);
    __builtin_amdgcn_sched_barrier(0);
    wait_vm<LATER + D / 16>();
    asm volatile("s_nop 0"); // the wait takes effect with the next instruction: that must not be one that needs it
    asm volatile("" : "+v"(th), "+v"(pos_lane));
    __builtin_amdgcn_sched_barrier(0);
    for (int p0 = 0; p0 < n_slots; p0 += ROT_SLOTS) {
        build_rot_table<D>(tab, th, lane, p0 == 0 ? pos_lane : pos_of_slot(p0 + (lane & (ROT_SLOTS - 1))), sl2e);
        if (p0 == 0) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<LATER>();
            asm volatile("s_nop 0");
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) asm volatile("" : "+v"(raw[ks]));
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool mine = (slot >= p0) && (slot < p0 + ROT_SLOTS);
        bf16x8 f[D / 16];
        if (HALF) rotate_q_shared_half<D>(raw, tab, mine ? slot - p0 : 0, h, f);
        else rotate_q_shared<D>(raw, tab, mine ? slot - p0 : 0, h, f);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            if (mine || p0 == 0) qf[ks] = f[ks]; // the first pass initialises every lane's fragments
        __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): the table is read before the next pass (or a tile load) overwrites it
    }
}

// Per-wave state of the tile loop.
template <int D> struct Acc {
    f32x16 o[D / 32]; // O^T: element e of block db is channel 32 db + 8 (e >> 2) + 4 h + (e & 3) of query column c
    // The negated reference maximum (log2 domain, score * log2(e)/sqrt(d)) of the lane's query column, in every element: the
    // addend of a tile's first score products.  Kept as a register block of its own, a tile starts its scores with no moves
    // (32 of some 130 vector instructions of a 64-key tile when they were written from a scalar each time).  With the test
    // for a new reference reduced to one comparison and the masks to constants, 89 are left, and one set of LDS offsets for
    // the whole ring frees the registers that the block takes (eight waves: 245 -> 206).  us before / after: one pass over
    // 32 x 1024 + 256 tokens 562 / 549, 256 query tokens over 32 x 1024 rows 177.8 / 175.7, 64 over 8 x 512 23.35 / 22.61.
    f32x16 nref;
    float l;          // this half-wave's share of the softmax denominator

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[db][e] = 0.0f;
        l = 0.0f;
        move_ref(0.0f);
    }
    __device__ __forceinline__ float mref() const { return -nref[0]; }
    __device__ __forceinline__ void move_ref(float neg)
    {
#pragma unroll
        for (int e = 0; e < 16; ++e) nref[e] = neg;
        asm volatile("" : "+v"(nref)); // a block of registers from here on, not a value to be spread again at each use
    }
};

// Issue this wave's share of the direct global->LDS loads of tile [kt, kt+KT): K rows to kdst, V rows to vdst.
// AUX is the cache policy of the loads: 0 where other workgroups read the same tile soon (the row tiles of a long
// query), DMA_STREAM (non-temporal) where every key is read exactly once (decode: 114 -> 100 us for 64 x 4096 rows;
// the same hint on the long-query kernels, whose row tiles share keys through L2, cost 5-8 %).
constexpr int DMA_STREAM = 2;
template <int D, int NW, int AUX = 0>
__device__ __forceinline__ void issue_tile(const __bf16* __restrict__ k, const __bf16* __restrict__ v, int64_t row_elems,
                                           int head_off, int kt, int key_clamp, LDS_AS char* kdst, LDS_AS char* vdst, int wave, int lane)
{
    using G = Geo<D>;
    constexpr int NI = KT / G::RPI;
    static_assert(NI % NW == 0, "tile loads must divide evenly over the waves");
    const int r_in = lane / G::CPR, pc = lane % G::CPR;
#pragma unroll
    for (int ii = 0; ii < NI / NW; ++ii) {
        const int i = wave + NW * ii;
        const int row = i * G::RPI + r_in;
        int key = kt + row;
        key = key > key_clamp ? key_clamp : key;
        const int ck = pc ^ G::kswz(row);
        const int cv = 4 * ((pc >> 2) ^ G::vswz(row)) + (pc & 3);
        const int64_t base = (int64_t)key * row_elems + head_off;
        __builtin_amdgcn_global_load_lds((const GLB_AS void*)(k + base + ck * 8), (LDS_AS void*)(kdst + i * 1024), 16, 0, AUX);
        __builtin_amdgcn_global_load_lds((const GLB_AS void*)(v + base + cv * 8), (LDS_AS void*)(vdst + i * 1024), 16, 0, AUX);
    }
}

// One tile of 32 KB keys in two phases.  Phase A: S^T = K Q^T and the online softmax, leaving P^T packed as bf16 B
// operands.  Phase B: O^T += V^T P^T.  krows / vrows point at the tile's first K / V row in LDS, kt is its first key.
struct NoHook {
    __device__ __forceinline__ void operator()(int) const {}
};

// between(ks) runs after the products of k-step ks have been issued: the tile loop puts its loads of a later tile
// there, so that their issue falls into the shadow of the matrix instructions instead of in front of them.
template <int D, int KB, class Between = NoHook>
__device__ __forceinline__ void scores_softmax(LDS_AS const char* krows, const bf16x8 (&qf)[D / 16], const RowCtx& rc, int kt,
                                               bool need_mask, bool need_lo, const int (&koff)[D / 16], int h, Acc<D>& acc, bf16x8 (&bpk)[KB][2],
                                               Between between = Between())
{
    // scores relative to the row reference, in the log2 domain (the queries carry log2(e)/sqrt(d)): the first products add
    // the negated reference, so P = exp2(S) needs no further arithmetic
    f32x16 s[KB];
    // operand reads run K_PREFETCH k-steps ahead of the products that use them (the compiler, left alone, reads one
    // step ahead and waits out the full LDS latency before every pair of products)
    constexpr int PD = K_PREFETCH, STEPS = D / 16;
    bf16x8 a[PD][KB];
#pragma unroll
    for (int ks = 0; ks < PD; ++ks)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) a[ks][kb] = *(LDS_AS const bf16x8*)(krows + koff[ks] + kb * 32 * D * 2);
#pragma unroll
    for (int ks = 0; ks < STEPS; ++ks) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks % PD][kb], qf[ks], ks == 0 ? acc.nref : s[kb], 0, 0, 0);
        if (ks + PD < STEPS) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) a[ks % PD][kb] = *(LDS_AS const bf16x8*)(krows + koff[ks + PD] + kb * 32 * D * 2);
        }
        between(ks);
        __builtin_amdgcn_sched_barrier(0);
    }
    // accumulator element e of block kb is key kt + 32 kb + 8 (e >> 2) + 4 h + (e & 3), query column c; the lane's share of
    // that sum goes into the bound, so that an element is tested against a constant
    if (need_mask) { // workgroup-uniform: only tiles that straddle a mask edge
        const int hi = rc.key_hi - kt - 4 * h;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (32 * kb + 8 * (e >> 2) + (e & 3) > hi) s[kb][e] = -INFINITY;
        if (need_lo) {
            const int lo = rc.key_lo - kt - 4 * h;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (32 * kb + 8 * (e >> 2) + (e & 3) < lo) s[kb][e] = -INFINITY;
        }
    }
    float part[4]; // four short chains instead of one long one
#pragma unroll
    for (int i = 0; i < 4; ++i) part[i] = s[0][i];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = kb == 0 ? 4 : 0; e < 16; ++e) part[e & 3] = fmaxf(part[e & 3], s[kb][e]);
    float mx = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    // Lazy reference update (exact: any reference gives the same softmax).  A lane whose scores stay below the slack and
    // that has accumulated something cannot ask for one, so the tiles after the first nearly always go on with this one
    // comparison; what the column decides is worked out only where some lane might.
    if (__any(mx > RESCALE_SLACK || acc.l == 0.0f)) {
        mx = column_max(mx); // both half-waves hold keys of the same query column
        // `first`: nothing accumulated yet and the tile sits far below the reference - move the reference down so that exp2
        // does not underflow.  Lanes c and c + 32 hold the two key halves of ONE query column and share its reference, so
        // the decision is taken on the column's denominator: a row whose first visible keys all fell into one half must not
        // move the other half's reference alone.
        const float l_col = column_sum(acc.l);
        const bool first = (l_col == 0.0f) && (mx < REREF_BELOW) && (mx > -INFINITY);
        const bool grow = (mx > RESCALE_SLACK) || first;
        if (__any(grow)) { // rare
            const float delta = grow ? mx : 0.0f;
            const float alpha = first ? 1.0f : __builtin_amdgcn_exp2f(-delta); // first: accumulators are still zero
            acc.move_ref(acc.nref[0] - delta);
            acc.l *= alpha;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc.o[db][e] *= alpha;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int e = 0; e < 16; ++e) s[kb][e] -= delta;
        }
    }
    // P = exp2(S), packed to bf16 B-operands; the denominator sums the rounded weights the product uses
    {
        bf16x2 ones;
        ones[0] = (__bf16)1.0f;
        ones[1] = (__bf16)1.0f;
        float l = acc.l;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                bf16x2 pr;
                pr[0] = (__bf16)__builtin_amdgcn_exp2f(s[kb][2 * i]);
                pr[1] = (__bf16)__builtin_amdgcn_exp2f(s[kb][2 * i + 1]);
                bpk[kb][i / 4][2 * (i % 4)] = pr[0];
                bpk[kb][i / 4][2 * (i % 4) + 1] = pr[1];
                l = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l, false);
            }
        acc.l = l;
    }
}

// O^T += V^T P^T.  k-slot j of k-step (kb, t) is key 32 kb + 16 t + 8 (j >> 2) + 4 h + (j & 3).
// between(i) runs behind product i.
template <int D, int KB, class Between = NoHook>
__device__ __forceinline__ void weighted_values(LDS_AS const char* vrows, const bf16x8 (&bpk)[KB][2], const int (&voff)[D / 32],
                                                Acc<D>& acc, Between between = Between())
{
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16x8 bp = bpk[kb][t];
            const int rbase = (32 * kb + 16 * t) * D * 2;
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
                LDS_AS const char* p0 = vrows + rbase + voff[db];
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(p0));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(p0 + 8 * D * 2));
                const s16x8 av = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                acc.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), bp, acc.o[db], 0, 0, 0);
                between((kb * 2 + t) * (D / 32) + db);
            }
        }
}

// The rows of K/V one workgroup walks: tiles of 64 keys from kt_begin, n_tiles of them; key_clamp is the last row
// that may be loaded (rows past it are never visible and read that row instead).
struct Walk {
    int kt_begin;
    int n_tiles;
    bool half_tail; // the last tile holds at most 32 of the walk's keys
    int key_clamp;
    int head_off;
    int64_t row_elems;
};

__device__ __forceinline__ Walk make_walk(int kt_begin, int kt_end, int key_clamp, int n_kv_heads, int kvh, int d)
{
    Walk w;
    w.kt_begin = kt_begin;
    w.n_tiles = kt_end > kt_begin ? (kt_end - kt_begin + KT - 1) / KT : 0;
    w.half_tail = kt_end > kt_begin && (kt_end - kt_begin - 1) % KT < KT / 2;
    w.key_clamp = key_clamp;
    w.head_off = kvh * d;
    w.row_elems = (int64_t)n_kv_heads * d;
    return w;
}

// The ring: NS K tiles, then NS V tiles.  K and V lie apart so that every stage of either is within reach of the 16-bit
// offset field of an LDS instruction (64 KB) and one set of lane offsets serves all stages.
template <int D> constexpr int ring_k(int stage) { return stage * Geo<D>::TILE_BYTES; }
template <int D, int NS> constexpr int ring_v(int stage) { return (NS + stage) * Geo<D>::TILE_BYTES; }

// This wave's loads of one whole tile whose 64 rows all exist (no clamping): the lane's byte offsets inside the tile
// are computed once, the tile's first row is a uniform base, so a load costs no vector arithmetic.
template <int D, int NW> constexpr int tile_loads() { return 2 * Geo<D>::NI / NW; } // load instructions of a wave for a tile
template <int D, int NW> struct TileLoads {
    uint32_t dk[Geo<D>::NI / NW], dv[Geo<D>::NI / NW]; // byte offsets of this lane's 16 bytes from the tile's first row
    uint32_t lds_wave; // LDS address of this wave's first 1 KB slot in K stage 0 (uniform)

    __device__ __forceinline__ TileLoads(const Walk& w, LDS_AS char* smem, int wave, int lane)
    {
        using G = Geo<D>;
        lds_wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)smem + wave * 1024);
        const int r_in = lane / G::CPR, pc = lane % G::CPR;
        const uint32_t row_bytes = (uint32_t)w.row_elems * 2u;
#pragma unroll
        for (int ii = 0; ii < G::NI / NW; ++ii) {
            const int row = (wave + NW * ii) * G::RPI + r_in;
            const int ck = pc ^ G::kswz(row);
            const int cv = 4 * ((pc >> 2) ^ G::vswz(row)) + (pc & 3);
            dk[ii] = (uint32_t)row * row_bytes + (uint32_t)(w.head_off + ck * 8) * 2u;
            dv[ii] = (uint32_t)row * row_bytes + (uint32_t)(w.head_off + cv * 8) * 2u;
        }
    }
    // load pair ii of this wave: 1 KB of the K tile and 1 KB of the V tile; stage: a constant
    template <int NS, int AUX>
    __device__ __forceinline__ void pair(const char* __restrict__ ktile, const char* __restrict__ vtile, int stage, int ii) const
    {
        const uint32_t dst = lds_wave + (uint32_t)(NW * ii * 1024);
        __builtin_amdgcn_global_load_lds((const GLB_AS void*)(ktile + dk[ii]), (LDS_AS void*)(uintptr_t)(dst + ring_k<D>(stage)), 16, 0, AUX);
        __builtin_amdgcn_global_load_lds((const GLB_AS void*)(vtile + dv[ii]), (LDS_AS void*)(uintptr_t)(dst + ring_v<D, NS>(stage)), 16, 0, AUX);
    }
    template <int NS, int AUX>
    __device__ __forceinline__ void tile(const char* __restrict__ ktile, const char* __restrict__ vtile, int stage) const
    {
#pragma unroll
        for (int ii = 0; ii < Geo<D>::NI / NW; ++ii) pair<NS, AUX>(ktile, vtile, stage, ii);
    }
};

// The loads of the tile whose first key is kt; a tile that lacks rows takes the clamping path.
template <int D, int NW, int NS, int AUX>
__device__ __forceinline__ void issue_any(const __bf16* __restrict__ k, const __bf16* __restrict__ v, const Walk& w,
                                          const TileLoads<D, NW>& tl, int kt, int stage, LDS_AS char* smem, int wave, int lane)
{
    const int64_t off = (int64_t)kt * w.row_elems;
    if (kt + KT - 1 <= w.key_clamp) tl.template tile<NS, AUX>((const char*)(k + off), (const char*)(v + off), stage);
    else issue_tile<D, NW, AUX>(k, v, w.row_elems, w.head_off, kt, w.key_clamp, smem + ring_k<D>(stage), smem + ring_v<D, NS>(stage), wave, lane);
}

// Tiles 0 .. NS-2 in flight.  Stage NS-1 stays free until the tile loop's first iteration has passed its barrier.  Tiles that
// the walk does not have are requested all the same (rows past the last one read that row, and nothing looks at them), so
// that the number of loads in flight is a constant and what was requested before them can be waited for by count.
template <int D, int NW, int NS, int AUX = 0>
__device__ __forceinline__ void issue_prologue(const __bf16* __restrict__ k, const __bf16* __restrict__ v, const Walk& w,
                                               const TileLoads<D, NW>& tl, LDS_AS char* smem, int wave, int lane)
{
    using G = Geo<D>;
    static_assert(2 * G::NI / NW == tile_loads<D, NW>(), "");
#pragma unroll
    for (int p = 0; p < NS - 1; ++p) {
        // a branch around the offsets, not around the loads
        const int kt = min(w.kt_begin + p * KT, w.key_clamp), last = w.key_clamp - kt; // last: row of the tile, if below KT
        TileLoads<D, NW> t = tl;
        if (last < KT - 1) {
            const uint32_t row_bytes = (uint32_t)w.row_elems * 2u;
#pragma unroll
            for (int ii = 0; ii < G::NI / NW; ++ii) {
                const int row = (wave + NW * ii) * G::RPI + lane / G::CPR;
                const uint32_t back = (uint32_t)max(row - last, 0) * row_bytes;
                t.dk[ii] -= back;
                t.dv[ii] -= back;
            }
        }
        const int64_t off = (int64_t)kt * w.row_elems;
        t.template tile<NS, AUX>((const char*)(k + off), (const char*)(v + off), p);
    }
}

// The tile loop shared by both kernels (issue_prologue has run).  Tile [kt, kt+64) needs per-element masking iff
// kt+63 > mask_hi_min or kt < mask_lo_max.  The loop is unrolled over the ring so that the stage of every LDS
// access is a constant of the instruction: the operand reads then need no address arithmetic at all (the lane's
// offsets inside a stage are loop constants, the stage goes into the instruction's offset field).
template <int D, int NW, int NS, int AUX = 0>
__device__ __forceinline__ void attn_tiles(const __bf16* __restrict__ k, const __bf16* __restrict__ v, const Walk& w,
                                           const TileLoads<D, NW>& tl, const RowCtx& rc, const bf16x8 (&qf)[D / 16], int mask_hi_min,
                                           int mask_lo_max, LDS_AS char* smem, Acc<D>& acc)
{
    using G = Geo<D>;
    constexpr int IPW = 2 * G::NI / NW; // loads each wave issues per tile
    static_assert(G::NI % NW == 0, "tile loads must divide evenly over the waves");
    static_assert(NS == 2 || NS == 4, "the ring has two or four stages");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int i16 = lane & 15, colhalf = (lane >> 4) & 1;

    const int wave_hi_max = wave_max_i(rc.valid ? rc.key_hi : INT32_MIN);
    const int wave_lo_min = wave_min_i(rc.valid ? rc.key_lo : INT32_MAX);

    // LDS addresses of this lane's operands in stage 0: whole addresses, the ring's base included, so that what an access
    // adds is a constant that fits its offset field
    const int lds0 = (int)(uintptr_t)smem;
    int koff[D / 16];
    int voff[D / 32];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) koff[ks] = lds0 + c * D * 2 + (((2 * ks + h) ^ G::kswz(c)) * 16);
    const int r = 4 * h + (i16 >> 2); // row inside an 8-row k-slot block; rows 8 apart share the swizzle
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
        voff[db] = lds0 + ring_v<D, NS>(0) + r * D * 2 + (4 * (db ^ G::vswz(r)) + 2 * colhalf + ((i16 & 3) >> 1)) * 16 + (i16 & 1) * 8;
    const int64_t row_bytes64 = w.row_elems * 2;

    const int n_tiles = w.n_tiles, n_whole = n_tiles - (w.half_tail ? 1 : 0);
    bf16x8 bpk[2][2];
    // Interior tiles first, a ring-full at a time, in a loop with nothing to decide: every row of the workgroup sees
    // every key of the tile (no mask, every wave that has rows computes), the tile requested behind each barrier
    // exists and has all its rows (the plain loads), so the wait counts are constants.  A long document prefix is almost all interior; the general loop below takes over wherever this stops.
    // Only the eight-wave kernel has it (2 % at the long-query configuration): in the four-wave kernels it would have to
    // give up the loads issued between the score products (with them the compiler spills), and measured 2 % slower.
    int t0 = 0;
    if (NW == 8) {
        // tiles [0, t_b) lie wholly below the first row's causal edge; the lower edge must not cut into the walk at all
        const int t_b = mask_lo_max <= w.kt_begin ? (mask_hi_min - (KT - 1) - w.kt_begin >= 0 ? (mask_hi_min - (KT - 1) - w.kt_begin) / KT + 1 : 0) : 0;
        const bool wave_has_rows = wave_hi_max != INT32_MIN;
        // a group of NS tiles from t0: all interior (t0 + NS <= t_b), all requested tiles t0 + NS - 1 .. t0 + 2 NS - 2 exist
        // and are not the walk's last tile, the only one that may lack rows (t0 + 2 NS <= n_tiles)
        for (; t0 + NS <= t_b && t0 + 2 * NS <= n_tiles; t0 += NS) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                wait_vm<(NS - 2) * IPW>();
                __builtin_amdgcn_s_barrier();
                const int ktn = w.kt_begin + (t0 + s + NS - 1) * KT;
                const char* ktile = (const char*)k + (int64_t)ktn * row_bytes64;
                const char* vtile = (const char*)v + (int64_t)ktn * row_bytes64;
                LDS_AS const char* stage = (LDS_AS const char*)(uintptr_t)(s * G::TILE_BYTES);
                tl.template tile<NS, AUX>(ktile, vtile, (s + NS - 1) % NS);
                if (wave_has_rows) {
                    scores_softmax<D, 2>(stage, qf, rc, 0, false, false, koff, h, acc, bpk);
                    weighted_values<D, 2>(stage, bpk, voff, acc);
                }
            }
        }
    }
    for (; t0 < n_whole; t0 += NS) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int t = t0 + s;
            if (t >= n_whole) break;
            const int kt = w.kt_begin + t * KT;
            // tile t has landed once at most the loads of the tiles issued after it are outstanding
            const int later = min(NS - 2, n_tiles - 1 - t);
            if (NS >= 4 && later >= 2) wait_vm<2 * IPW>();
            else if (NS >= 3 && later >= 1) wait_vm<IPW>();
            else wait_vm<0>();
            __builtin_amdgcn_s_barrier(); // every wave's share of tile t is in LDS; everyone is done with tile t-1
            const bool active = (kt <= wave_hi_max) && (kt + KT - 1 >= wave_lo_min); // wave-uniform
            const int ktn = kt + (NS - 1) * KT;
            const int dst = (s + NS - 1) % NS; // a constant once the loop is unrolled
            const bool more = t + NS - 1 < n_tiles;
            const bool whole = ktn + KT - 1 <= w.key_clamp;
            const char* ktile = (const char*)k + (int64_t)ktn * row_bytes64;
            const char* vtile = (const char*)v + (int64_t)ktn * row_bytes64;
            // the loads of tile t + NS - 1: a wave that computes this tile issues them between its first score products
            // (below); a wave that skips the tile, or a tile with clamped rows, issues them here
            // (measured: the four-wave kernels, whose waves issue twice as many loads per tile, gain 2-5 %; the
            // eight-wave kernel loses the 2 % the unrolled ring gave it, so it keeps its loads in front)
            const bool defer = (NW == 4) && more && whole && active;
            if (more && !defer) issue_any<D, NW, NS, AUX>(k, v, w, tl, ktn, dst, smem, wave, lane);
            if (active) {
                // the stage is a constant of each access, of the K and of the V reads alike (their offsets include the base)
                LDS_AS const char* stage = (LDS_AS const char*)(uintptr_t)(s * G::TILE_BYTES);
                const bool need_lo = kt < mask_lo_max;
                const bool need_mask = (kt + KT - 1 > mask_hi_min) || need_lo;
                scores_softmax<D, 2>(stage, qf, rc, kt, need_mask, need_lo, koff, h, acc, bpk, [&](int ks) {
                    if (ks < G::NI / NW && defer) tl.template pair<NS, AUX>(ktile, vtile, dst, ks);
                });
                weighted_values<D, 2>(stage, bpk, voff, acc);
            }
        }
    }
    // A last tile of at most 32 keys takes its lower half alone: half the products, weights and operand reads.  Under a causal
    // mask that is every other row tile of 32 tokens (group 4).  Offline ingest of 64 chunks of 512 tokens, 32 / 8 heads:
    // 280.4 -> 275.6 us; one pass over 33024 tokens: 538.0 -> 535.7 us.  Behind the loop, not a branch in it: with both forms
    // in the unrolled loop the compiler spills.
    if (w.half_tail) {
        const int kt = w.kt_begin + n_whole * KT;
        wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        if (kt <= wave_hi_max && kt + KT / 2 - 1 >= wave_lo_min) {
            LDS_AS const char* stage = (LDS_AS const char*)(uintptr_t)((n_whole % NS) * G::TILE_BYTES);
            bf16x8 bph[1][2];
            scores_softmax<D, 1>(stage, qf, rc, kt, true, kt < mask_lo_max, koff, h, acc, bph);
            weighted_values<D, 1>(stage, bph, voff, acc);
        }
    }
}

// The ordinary loads of a workgroup's start, issued as one batch before anything waits: the position id of the lane's
// token slot and whatever indices the caller needs (issued by the caller, first), theta, then the raw query rows.
// Loads return in order, so the small ones in front are back after one L2 round trip while the query rows are
// still on their way from HBM.
template <int D> struct QLoads {
    double th;          // theta_rev[lane % (D/2)]
    u32x4 raw[D / 16];  // this lane's raw query fragments
};

// The order is fixed: the waits in front of the rotation count on it.
template <int D, class Args>
__device__ __forceinline__ void issue_q_loads(const __bf16* __restrict__ q, const RowCtx& rc, QLoads<D>& ql)
{
    const int lane = threadIdx.x & 63, h = lane >> 5;
    ql.th = load_theta<Args>(lane % (D / 2));
    __builtin_amdgcn_sched_barrier(0);
    load_q_raw<D>(q, rc, h, ql.raw);
    __builtin_amdgcn_sched_barrier(0);
}

// The first K/V tiles, then the rotation: the tile loads fly while the angles are computed.  Their addresses need no loaded
// value, so they go out behind the query rows without a wait.  theta and pos_lane (the position id of token slot (lane & 7) of
// this wave, which the caller loaded first) are touched next, the query rows after the angle table is built; pos_of_slot
// serves the later passes of small GQA groups.  The rotation table sits in stage NS-1, which no tile load targets before the
// first barrier of the tile loop.
template <int D, int NW, int NS, bool HALF, int AUX = 0, class PosFn>
__device__ __forceinline__ void prologue(const __bf16* __restrict__ k, const __bf16* __restrict__ v, const Walk& w,
                                         const TileLoads<D, NW>& tl, QLoads<D>& ql,
                                         int pos_lane, int slot, int n_slots, PosFn pos_of_slot, float sl2e, LDS_AS char* smem,
                                         bf16x8 (&qf)[D / 16])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5;
    issue_prologue<D, NW, NS, AUX>(k, v, w, tl, smem, wave, lane);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int TAB = ROT_SLOTS * 4 * D, PER_TILE = Geo<D>::TILE_BYTES / TAB; // tables that fit a K or V tile
    static_assert(NW <= 2 * PER_TILE, "the waves' tables fit one stage");
    LDS_AS char* tab = smem + (wave < PER_TILE ? ring_k<D>(NS - 1) + wave * TAB : ring_v<D, NS>(NS - 1) + (wave - PER_TILE) * TAB);
    rotate_queries<D, HALF, (NS - 1) * tile_loads<D, NW>()>(ql.raw, tab, ql.th, pos_lane, lane, h, slot, n_slots, sl2e, pos_of_slot, qf);
}

// Write the wave's 32 x D accumulator as rows, straight from registers.
//   PARTIAL = false: out[dst_row][:] = bf16(O / l)       PARTIAL = true: ws_o[dst_row][:] = fp16(O / l)
// A partial is normalised by its own denominator, so it is a convex combination of V rows and fp16 (11 bits,
// 8 times finer than the bf16 result) holds it where V is in fp16's range, above some 1e-4 and below 65504; the merge weighs it
// with l again.
// Lanes c and c + 32 hold alternate groups of four channels of row c.  Two swaps of the vector unit give each of them
// eight neighbouring channels, so a lane stores 16 bytes and a row receives 32 contiguous bytes per instruction.  An
// epilogue is pure latency at the end of a workgroup, so what counts is how short its dependent chain is: staging the rows
// through LDS for whole-line stores, with two lane permutes per four rows, took 2.4 us of the 12.4 us of a workgroup that
// walks five key tiles; without it the request over 8 x 512 rows went from 25.6 to 24.1 us, 64 x 512 offline tokens from
// 296 to 284 us.  Partials too are ordinary stores: 64-byte pieces (a third swap) that bypass the L2 are faster where a call
// is repeated on one workspace that the caches still hold (8 MB of partials 22.6 -> 20.7 us, and whole lines through LDS 21.7),
// but in every call on a workspace that other work has displaced, slower than the above by 4 to 9 % from 4 MB on
// (16 heads, 100 tokens over 5000 keys 21.8 -> 23.8 us; through LDS 23.0); 64-byte pieces through the L2 make no difference.
// The caller's rows may start at any multiple of an element: unaligned 16-byte stores are one instruction all the same.
typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef bf16x4 bf16x4_any __attribute__((aligned(2)));
template <int D, bool PARTIAL>
__device__ __forceinline__ void store_rows(const Acc<D>& acc, float l_tot, bool valid, int64_t dst_row, void* dst, int lane)
{
    const int h = lane >> 5;
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    auto pack = [&](int db, int q4, int i) { // channels 32 db + 8 q4 + 4 h + 2 i, + 1
        const float x = acc.o[db][4 * q4 + 2 * i] * inv, y = acc.o[db][4 * q4 + 2 * i + 1] * inv;
        if (PARTIAL) {
            f16x2 t;
            t[0] = (_Float16)x;
            t[1] = (_Float16)y;
            return __builtin_bit_cast(uint32_t, t);
        }
        bf16x2 t;
        t[0] = (__bf16)x;
        t[1] = (__bf16)y;
        return __builtin_bit_cast(uint32_t, t);
    };
    char* row = (char*)dst + (dst_row * D + 8 * h) * 2;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                // lanes below 32 keep group 2 p of both halves, lanes from 32 on group 2 p + 1
                const auto r = __builtin_amdgcn_permlane32_swap(pack(db, 2 * p, i), pack(db, 2 * p + 1, i), false, false);
                w[i] = r[0];
                w[2 + i] = r[1];
            }
            if (valid) *(u32x4_any*)(row + (32 * db + 16 * p) * 2) = w;
        }
}

// ---- step 6: query prefill over the assembled cache -------------------------------------------------------------
// AUX: cache policy of the K/V tile loads; DMA_STREAM when no request of the launch has more than one row tile, so
// that every key is read by exactly one workgroup (a few query tokens over a long context: 24.0 -> 22.5 us for
// 16 tokens over 12288 rows, Qwen2-7B heads).
template <int D, int NW, int NS, bool HALF, int AUX>
__global__ __launch_bounds__(64 * NW, 2) void prefix_attn_kernel(const TrPrefixArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
    LDS_AS char* smem = (LDS_AS char*)smem_raw;
    const int item = xcd_remap(blockIdx.x, a.n_items);
    const TrSeqDesc sd = a.seq[last_not_above(a.n_seq, item, [&](int i) { return a.seq[i].item0; })];
    const int local = item - sd.item0;
    const int tile = local % sd.n_tiles;
    const int rest = local / sd.n_tiles;
    const int split = rest % sd.n_split;
    const int kvh = rest / sd.n_split;
    const int g = a.group, tpt = a.tok_per_tile;
    const int n_doc = sd.kv_len - sd.n_q;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int rl = 32 * wave + c;
    const int tok_in = by_group(rl, a.group_magic), head_in = rl - tok_in * g; // token and head inside the tile
    const int tok_local = tile * tpt + tok_in;
    RowCtx rc;
    rc.valid = (rl < tpt * g) && (tok_local < sd.n_q);
    rc.orow = (sd.q_row0 + tok_local) * a.n_q_heads + kvh * g + head_in;
    rc.key_lo = sd.kv_row0;
    rc.key_hi = sd.kv_row0 + n_doc + tok_local;
    // position ids per token slot of the wave
    const int wave_in = by_group(32 * wave, a.group_magic); // first token of the wave
    const int wave_tok0 = tile * tpt + wave_in;
    const int slot = min(tok_in - wave_in, 31);
    const int n_slots = by_group(32 * wave + 31, a.group_magic) - wave_in + 1;
    auto pos_of_slot = [&](int s) { return a.q_pos[sd.q_row0 + min(wave_tok0 + s, sd.n_q - 1)]; };
    const int pos_lane = pos_of_slot(lane & (ROT_SLOTS - 1));
    QLoads<D> ql;
    issue_q_loads<D, TrPrefixArgs>((const __bf16*)a.q, rc, ql);

    const int first_tok = tile * tpt;
    const int last_tok = min(first_tok + tpt, sd.n_q) - 1;
    const int sb = sd.kv_row0 + split * sd.split_len;
    const int se = min(sb + sd.split_len, sd.kv_row0 + sd.kv_len);
    const Walk w = make_walk(sb, min(se, sd.kv_row0 + n_doc + last_tok + 1), sd.kv_row0 + sd.kv_len - 1, a.n_kv_heads, kvh, D);

    const TileLoads<D, NW> tl(w, smem, wave, lane);
    bf16x8 qf[D / 16];
    prologue<D, NW, NS, HALF, AUX>((const __bf16*)a.k, (const __bf16*)a.v, w, tl, ql, pos_lane, slot, n_slots, pos_of_slot, a.scale_log2e, smem, qf);

    Acc<D> acc;
    acc.clear();

    attn_tiles<D, NW, NS, AUX>((const __bf16*)a.k, (const __bf16*)a.v, w, tl, rc, qf, sd.kv_row0 + n_doc + first_tok, sd.kv_row0, smem, acc);

    const float l_tot = acc.l + __shfl_xor(acc.l, 32);
    if (sd.n_split == 1) {
        store_rows<D, false>(acc, l_tot, rc.valid, (int64_t)rc.orow, a.out, lane);
    } else {
        const int rows_s = sd.n_q * g;
        const int64_t prow = (int64_t)sd.ws_row0 + (int64_t)(split * a.n_kv_heads + kvh) * rows_s + tok_local * g + head_in;
        store_rows<D, true>(acc, l_tot, rc.valid, prow, a.ws_o, lane);
        // a split in which the row saw no key reports m = -inf so that the merge ignores it
        if (rc.valid && h == 0) *(float2*)(a.ws_ml + prow * 2) = make_float2(l_tot > 0.0f ? acc.mref() : -INFINITY, l_tot);
    }
}

// ---- step 6 without a materialised cache: attention that gathers the chunks itself --------------------------------
// The document keys are read straight from the store, where they are rotated at chunk-local positions.  Under
// reordered positions the score needs R(off + t) k; since <R(p) q, R(off + t) k> = <R(p - off) q, R(t) k> (the
// relative-position property behind Eq. 3), the kernel turns the QUERY by -off once per chunk instead of turning
// every key.  The request's own query tokens are read from the cache rows that tr_kv_append wrote.  The walk is a
// list of 64-key tiles, chunk by chunk; the last tile of a chunk may be partial (its missing keys are masked).
constexpr int GATHER_NW = 4, GATHER_NS = 2;
template <int D> constexpr int gather_lds_bytes() { return GATHER_NS * Geo<D>::STAGE_BYTES + GATHER_NW * ROT_SLOTS * 4 * D; }

template <int D, bool HALF>
__global__ __launch_bounds__(64 * GATHER_NW, 2) void gather_attn_kernel(const TrGatherArgs a)
{
    using G = Geo<D>;
    constexpr int NW = GATHER_NW, NS = GATHER_NS;
    extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
    LDS_AS char* smem = (LDS_AS char*)smem_raw;
    const int item = xcd_remap(blockIdx.x, a.n_items);
    const int tile = item % a.row_tiles;
    const int rest = item / a.row_tiles;
    const int split = rest % a.n_split;
    const int kvh = rest / a.n_split;
    const int g = a.group, tpt = a.tok_per_tile;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int i16 = lane & 15, colhalf = (lane >> 4) & 1;
    const int rl = 32 * wave + c;
    const int tok_in = by_group(rl, a.group_magic), head_in = rl - tok_in * g; // token and head inside the tile
    const int tok_local = tile * tpt + tok_in;
    RowCtx rc;
    rc.valid = (rl < tpt * g) && (tok_local < a.n_q);
    rc.orow = tok_local * a.n_q_heads + kvh * g + head_in;
    rc.key_lo = 0;
    rc.key_hi = a.n_doc + tok_local;
    const int wave_in = by_group(32 * wave, a.group_magic); // first token of the wave
    const int wave_tok0 = tile * tpt + wave_in;
    const int slot = min(tok_in - wave_in, 31);
    const int n_slots = by_group(32 * wave + 31, a.group_magic) - wave_in + 1;
    const int first_tok = tile * tpt;
    const int last_tok = min(first_tok + tpt, a.n_q) - 1;

    // this workgroup's tiles: a contiguous range of the request's tile list, cut at the causal end of its rows
    const int tail = a.n_seg - 1;
    const int g0 = split * a.tiles_per_split;
    int g1 = min(g0 + a.tiles_per_split, a.n_tiles_total);
    g1 = min(g1, a.seg[tail].tile0 + last_tok / KT + 1);
    const int n_tiles = g1 > g0 ? g1 - g0 : 0;
    int s_issue = last_not_above(a.n_seg, g0, [&](int i) { return a.seg[i].tile0; });
    int s_comp = s_issue;

    const int64_t row_elems = (int64_t)a.n_kv_heads * D;
    const int head_off = kvh * D;
    auto issue = [&](int gt, int sg, LDS_AS char* stage) {
        const TrGatherSeg e = a.seg[sg];
        const int first = e.src_row + (gt - e.tile0) * KT;
        const bool from_cache = sg == tail;
        issue_tile<D, NW>((const __bf16*)(from_cache ? a.k_cache : a.k_store), (const __bf16*)(from_cache ? a.v_cache : a.v_store),
                          row_elems, head_off, first, e.src_row + e.n_rows - 1, stage, stage + G::TILE_BYTES, wave, lane);
    };

    if (n_tiles > 0) issue(g0, s_issue, smem);
    // The queries are rotated at the top of the tile loop whenever the chunk (hence the offset) changes, the first
    // tile included.  The raw rows are fetched again each time rather than held in 32 registers through the loop:
    // the change is rare (once per chunk) and the rows are in L2.
    LDS_AS char* tab = smem + NS * G::STAGE_BYTES + wave * (ROT_SLOTS * 4 * D); // private to the wave, outside the ring
    bf16x8 qf[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) qf[ks] = bf16x8{};
    int cur_delta = INT32_MIN;

    Acc<D> acc;
    acc.clear();

    const int wave_hi_max = wave_max_i(rc.valid ? rc.key_hi : INT32_MIN);
    const int mask_hi_min = a.n_doc + first_tok;
    int koff[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) koff[ks] = c * D * 2 + (((2 * ks + h) ^ G::kswz(c)) * 16);
    int voff[D / 32];
    {
        const int r = 4 * h + (i16 >> 2);
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
            voff[db] = r * D * 2 + (4 * (db ^ G::vswz(r)) + 2 * colhalf + ((i16 & 3) >> 1)) * 16 + (i16 & 1) * 8;
    }

    bf16x8 bpk[2][2];
    for (int t = 0; t < n_tiles; ++t) {
        const int gt = g0 + t;
        while (s_comp + 1 < a.n_seg && a.seg[s_comp + 1].tile0 <= gt) ++s_comp;
        const TrGatherSeg e = a.seg[s_comp];
        if (e.delta != cur_delta) { // a new chunk: the queries turn to its offset
            cur_delta = e.delta;
            const double th = a.theta_rev[lane % (D / 2)];
            const __bf16* qrow = (const __bf16*)a.q + (int64_t)(rc.valid ? rc.orow : 0) * D + 8 * h;
            const int ns = __builtin_amdgcn_readfirstlane(n_slots);
            for (int p0 = 0; p0 < ns; p0 += ROT_SLOTS) { // one pass when the GQA group is >= 4
                build_rot_table<D>(tab, th, lane, a.q_pos[min(wave_tok0 + p0 + (lane & (ROT_SLOTS - 1)), a.n_q - 1)] - cur_delta, a.scale_log2e);
                const bool mine = (slot >= p0) && (slot < p0 + ROT_SLOTS);
                LDS_AS const char* row = tab + (mine ? slot - p0 : 0) * (4 * D);
                const int sw = 2 * (mine ? slot - p0 : 0);
                // the raw fragments come in two parts so that they never hold more than 16 registers
                if (HALF) {
#pragma unroll
                    for (int part = 0; part < 2; ++part) {
                        u32x4 qlo[D / 64], qhi[D / 64];
#pragma unroll
                        for (int i = 0; i < D / 64; ++i) {
                            qlo[i] = *(const u32x4*)(qrow + 16 * (part * (D / 64) + i));
                            qhi[i] = *(const u32x4*)(qrow + 16 * (part * (D / 64) + i + D / 32));
                        }
#pragma unroll
                        for (int i = 0; i < D / 64; ++i) {
                            const int ks = part * (D / 64) + i;
                            bf16x8 flo, fhi;
                            rot_frag_half<D>(qlo[i], qhi[i], row, ks, h, sw, flo, fhi);
                            if (mine || p0 == 0) { qf[ks] = flo; qf[ks + D / 32] = fhi; }
                        }
                    }
                } else {
#pragma unroll
                    for (int part = 0; part < 2; ++part) {
                        u32x4 raw[D / 32];
#pragma unroll
                        for (int i = 0; i < D / 32; ++i) raw[i] = *(const u32x4*)(qrow + 16 * (part * (D / 32) + i));
#pragma unroll
                        for (int i = 0; i < D / 32; ++i) {
                            const int ks = part * (D / 32) + i;
                            const int ch = (2 * (2 * ks + h)) ^ sw;
                            const f32x4 cs0 = *(LDS_AS const f32x4*)(row + ch * 16);
                            const f32x4 cs1 = *(LDS_AS const f32x4*)(row + ch * 16 + 16);
                            bf16x8 f;
                            rot_pair(raw[i][0], cs0[0], cs0[1], f, 0);
                            rot_pair(raw[i][1], cs0[2], cs0[3], f, 1);
                            rot_pair(raw[i][2], cs1[0], cs1[1], f, 2);
                            rot_pair(raw[i][3], cs1[2], cs1[3], f, 3);
                            if (mine || p0 == 0) qf[ks] = f;
                        }
                    }
                }
                __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): the table is read before the next pass rewrites it
            }
        }
        wait_vm<0>(); // two stages: tile t is the only load in flight here
        __builtin_amdgcn_s_barrier();
        if (t + 1 < n_tiles) {
            while (s_issue + 1 < a.n_seg && a.seg[s_issue + 1].tile0 <= gt + 1) ++s_issue;
            issue(gt + 1, s_issue, smem + ((t + 1) % NS) * G::STAGE_BYTES);
        }
        const int j = gt - e.tile0;
        const int kt = e.cache_row + j * KT;                      // cache row the tile's first key stands for
        const int last_valid = e.cache_row + min(e.n_rows, (j + 1) * KT) - 1;
        if (kt <= wave_hi_max) {
            LDS_AS const char* stage = smem + (t % NS) * G::STAGE_BYTES;
            RowCtx rct = rc;
            rct.key_hi = min(rc.key_hi, last_valid);
            const bool need_mask = (kt + KT - 1 > mask_hi_min) || (last_valid < kt + KT - 1);
            scores_softmax<D, 2>(stage, qf, rct, kt, need_mask, false, koff, h, acc, bpk);
            weighted_values<D, 2>(stage + G::TILE_BYTES, bpk, voff, acc);
        }
    }

    const float l_tot = acc.l + __shfl_xor(acc.l, 32);
    if (a.n_split == 1) {
        store_rows<D, false>(acc, l_tot, rc.valid, (int64_t)rc.orow, a.out, lane);
    } else {
        const int rows_s = a.n_q * g;
        const int64_t prow = (int64_t)(split * a.n_kv_heads + kvh) * rows_s + tok_local * g + head_in;
        store_rows<D, true>(acc, l_tot, rc.valid, prow, a.ws_o, lane);
        if (rc.valid && h == 0) *(float2*)(a.ws_ml + prow * 2) = make_float2(l_tot > 0.0f ? acc.mref() : -INFINITY, l_tot);
    }
}

// ---- step 6 / step 7 for very short queries (decode: one new token per request) --------------------------------
// When the packed rows of a (request, KV head) fit one 32-row MFMA block, giving each wave its own rows would
// leave three of four waves idle.  Here all four waves hold the SAME rows and split the keys instead: wave w owns
// keys [32 w, 32 w + 32) of every 128, and the four partial results are merged through LDS at the end.
//
// Bound by the stream of keys and values, whose rate depends on how much of it is on its way: a bare ring of loads over 537 MB in
// these rows' order reads 5.6 / 6.7 / 7.1 / 6.8 / 6.4 TB/s with 12 / 16 / 20 / 24 / 32 KB and more in flight per CU
// (profiles/load_rates.md).  So a wave refills its own units as soon as their operands are read, with at most SHORT_FLIGHT loads of
// 1 KB on their way: no barrier, and no stretch in which nothing is on its way.  (The first units, 2 D / 16 loads, leave together:
// nothing else would be asked for while the queries are rotated.  Two stages of a tile shared by the waves, a barrier
// each: the values' reads waited for every load of the next tile.)  With one unit of K and one of V per wave two workgroups
// fit a CU, and one reads while the other starts or merges.
// us with 5 / 6 / 7 / 8 loads: 64 tokens over 4096 keys each (539 MB; 94.3 with the shared stages) 82.5 / 84.4 / 86.5 / 90.6, 32
// over 8192 (8 heads) 154.5 / 158.3 / 162.0 / 170.2, but 32 over 1000 to 3000 56.5 / 53.7 / 53.7 / 54.2, 12 over 600 to 6000 40.2 /
// 38.9 / 39.3 / 40.4, and no clear difference where launch and prologue are most of the call or the pieces many.  Six is within
// 2.5 % of the best at these, five and seven are not.
constexpr int SHORT_NW = 4, SHORT_KT = 32 * SHORT_NW;
constexpr int SHORT_FLIGHT = 6;
template <int D> constexpr int short_unit_bytes() { return 32 * D * 2; }
template <int D> constexpr int short_ring_bytes() { return SHORT_NW * 2 * short_unit_bytes<D>(); }
template <int D> constexpr int short_tables_bytes() { return SHORT_NW * ROT_SLOTS * 4 * D; }
template <int D> constexpr int short_merge_row_bytes() { return D * 4 + 16; }

// A wave's loads of a unit.  Load i fills rows RPI i .. of it; the lane's byte offsets from the unit's first row are kept.
template <int D> struct UnitLoads {
    using G = Geo<D>;
    static constexpr int LPU = D / 16;
    uint32_t dk[LPU], dv[LPU], lds;

    __device__ __forceinline__ UnitLoads(uint32_t ring, uint32_t row_bytes, uint32_t head_bytes, int lane)
    {
        lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)ring);
        const int r_in = lane / G::CPR, pc = lane % G::CPR;
#pragma unroll
        for (int i = 0; i < LPU; ++i) {
            const int row = i * G::RPI + r_in;
            dk[i] = (uint32_t)row * row_bytes + head_bytes + (uint32_t)(pc ^ G::kswz(row)) * 16u;
            dv[i] = (uint32_t)row * row_bytes + head_bytes + (uint32_t)(4 * ((pc >> 2) ^ G::vswz(row)) + (pc & 3)) * 16u;
        }
    }
    // The unit has rows 0 .. last: rows past them read that one, and nothing looks at them.  For a walk's last unit.
    __device__ __forceinline__ void stay_within(int last, uint32_t row_bytes, int lane)
    {
        if (last >= 31) return;
#pragma unroll
        for (int i = 0; i < LPU; ++i) {
            const uint32_t back = (uint32_t)max(i * G::RPI + lane / G::CPR - last, 0) * row_bytes;
            dk[i] -= back;
            dv[i] -= back;
        }
    }
    __device__ __forceinline__ void k(const char* __restrict__ unit, int i) const
    {
        __builtin_amdgcn_global_load_lds((const GLB_AS void*)(unit + dk[i]), (LDS_AS void*)(uintptr_t)(lds + i * 1024), 16, 0, DMA_STREAM);
    }
    __device__ __forceinline__ void v(const char* __restrict__ unit, int i) const
    {
        __builtin_amdgcn_global_load_lds((const GLB_AS void*)(unit + dv[i]), (LDS_AS void*)(uintptr_t)(lds + short_unit_bytes<D>() + i * 1024), 16, 0, DMA_STREAM);
    }
};

// One wave's walk over n_own units, 128 keys apart, the first of them on its way.  Loads return in order, so the counts below
// say which of them have: unit t's keys once no more than the LPU loads of its values are left, its values once no more than
// those of unit t + 1's keys are.  Nothing is shared between waves.  k and v are restricted pointers of a function of its own
// and LDS is reached by whole addresses because the compiler otherwise waits for every load before each read of V.
template <int D>
__device__ __forceinline__ void short_units(const char* __restrict__ k, const char* __restrict__ v, UnitLoads<D>& ul, const RowCtx& rc,
                                            const bf16x8 (&qf)[D / 16], int own_begin, int n_own, int key_clamp, int mask_hi_min,
                                            uint32_t row_bytes, int lane, Acc<D>& acc)
{
    using G = Geo<D>;
    constexpr int LPU = D / 16, UNIT = short_unit_bytes<D>();
    constexpr int FLIGHT = SHORT_FLIGHT;
    static_assert(FLIGHT <= 2 * LPU, "a unit of each is all there is room for");
    const int c = lane & 31, h = lane >> 5;
    const int i16 = lane & 15, colhalf = (lane >> 4) & 1;
    const int ring0 = (int)ul.lds; // whole addresses: see attn_tiles
    int koff[D / 16], voff[D / 32];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) koff[ks] = ring0 + c * D * 2 + (((2 * ks + h) ^ G::kswz(c)) * 16);
    const int r = 4 * h + (i16 >> 2);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
        voff[db] = ring0 + UNIT + r * D * 2 + (4 * (db ^ G::vswz(r)) + 2 * colhalf + ((i16 & 3) >> 1)) * 16 + (i16 & 1) * 8;

    bf16x8 bpk[1][2];
    for (int t = 0; t < n_own; ++t) {
        const int kt = own_begin + t * SHORT_KT;
        const int next = kt + SHORT_KT;
        const bool more = t + 1 < n_own;
        const char* const knext = k + (int64_t)next * row_bytes;
        const char* const vnext = v + (int64_t)next * row_bytes;
        if (more) ul.stay_within(key_clamp - next, row_bytes, lane);
        wait_vm<LPU>(); // K(t)
        asm volatile("" ::: "memory");
        LDS_AS const char* unit = (LDS_AS const char*)(uintptr_t)0;
        scores_softmax<D, 1>(unit, qf, rc, kt, kt + 31 > mask_hi_min, false, koff, h, acc, bpk, [&](int ks) {
            if (ks == LPU - 1 && more) {
                wait_lds(); // the unit's keys are read
#pragma unroll
                for (int i = 0; i < LPU; ++i) {
                    if (i + LPU >= FLIGHT) wait_vm<FLIGHT - 1>();
                    ul.k(knext, i);
                }
            }
        });
        if (!more) wait_vm<0>(); // V(t)
        else wait_vm<LPU>();
        asm volatile("" ::: "memory");
        weighted_values<D, 1>(unit, bpk, voff, acc, [&](int i) {
            if (more && i % (LPU / 2) == LPU / 2 - 1) {
                wait_lds(); // this half of the unit's values is read
#pragma unroll
                for (int j = i - LPU / 2 + 1; j <= i; ++j) {
                    if (j + LPU >= FLIGHT) wait_vm<FLIGHT - 1>();
                    ul.v(vnext, j);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    }
}

// What a workgroup of the short-query kernel reads before its first request, in one batch of scalar loads: the arguments, the first
// request's descriptor, and, where there are more requests, the item's own.  Left alone, the loads came one after the other, each
// where its value was needed, with two divisions between them: nine round trips in front of the first keys.  us: 2 tokens over
// 1.3 k rows 16.7 / 16.3, 57 over 650 keys each 33.6 / 33.4.  The kernel for longer queries gains nothing by it (64 tokens over 4096 rows
// 22.2 / 22.3, batches of four requests 36.9 / 37.2).
struct ItemArgs {
    const __bf16 *q, *k, *v;
    const int32_t* q_pos;
    void* out;
    _Float16* ws_o;
    float* ws_ml;
    int n_q_heads, n_kv_heads, group, tok_per_tile, group_magic, partial_f32;
    float scale_log2e;
    TrSeqDesc sd;
    int tile, split, kvh;
};
__device__ __forceinline__ ItemArgs item_args(const TrPrefixArgs& a)
{
    ItemArgs r;
    r.n_q_heads = a.n_q_heads, r.n_kv_heads = a.n_kv_heads, r.group = a.group, r.tok_per_tile = a.tok_per_tile, r.group_magic = a.group_magic;
    r.scale_log2e = a.scale_log2e;
    r.partial_f32 = a.partial_f32;
    r.sd = a.seq[0];
    int n_seq = a.n_seq;
    // as pointers to global memory: out of the assembler they are pointers to anything, and flat accesses count twice
    auto q = (const GLB_AS __bf16*)a.q, k = (const GLB_AS __bf16*)a.k, v = (const GLB_AS __bf16*)a.v;
    auto q_pos = (const GLB_AS int32_t*)a.q_pos;
    auto out = (GLB_AS char*)a.out;
    auto ws_o = (GLB_AS _Float16*)a.ws_o;
    auto ws_ml = (GLB_AS float*)a.ws_ml;
    asm volatile("" : "+s"(q), "+s"(k), "+s"(v), "+s"(q_pos), "+s"(r.n_q_heads), "+s"(r.n_kv_heads), "+s"(r.group), "+s"(r.tok_per_tile),
                 "+s"(r.group_magic), "+s"(r.scale_log2e), "+s"(r.partial_f32), "+s"(n_seq));
    asm volatile("" : "+s"(r.sd.q_row0), "+s"(r.sd.n_q), "+s"(r.sd.kv_row0), "+s"(r.sd.kv_len), "+s"(r.sd.item0), "+s"(r.sd.n_tiles),
                 "+s"(r.sd.n_split), "+s"(r.sd.split_len), "+s"(r.sd.ws_row0), "+s"(r.sd.split_magic), "+s"(out), "+s"(ws_o), "+s"(ws_ml));
    r.q = (const __bf16*)q, r.k = (const __bf16*)k, r.v = (const __bf16*)v, r.q_pos = (const int32_t*)q_pos;
    r.out = (void*)out, r.ws_o = (_Float16*)ws_o, r.ws_ml = (float*)ws_ml;
    // Not by XCD: a workgroup shares no keys with another, and dealt out in turn the heads of a long request spread over the
    // chip (18 requests of 1.6 k to 5.8 k keys 49.4 / 40.4 us).
    const int item = blockIdx.x;
    if (n_seq > 1) r.sd = a.seq[last_not_above(n_seq, item, [&](int i) { return a.seq[i].item0; })];
    const int local = item - r.sd.item0;
    const int rest = r.sd.n_tiles == 1 ? local : local / r.sd.n_tiles;
    r.tile = local - rest * r.sd.n_tiles;
    r.kvh = r.sd.n_split == 1 ? rest : (int)(((uint64_t)(uint32_t)rest * r.sd.split_magic) >> 32);
    r.split = rest - r.kvh * r.sd.n_split;
    return r;
}

template <int D, bool HALF>
__global__ __launch_bounds__(64 * SHORT_NW, 2) void short_attn_kernel(const TrPrefixArgs args)
{
    constexpr int NW = SHORT_NW;
    constexpr int UNIT = short_unit_bytes<D>(), LPU = D / 16; // LPU: loads of a unit, as many as a unit has products
    extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
    LDS_AS char* smem = (LDS_AS char*)smem_raw;
    const ItemArgs a = item_args(args);
    const TrSeqDesc sd = a.sd;
    const int tile = a.tile, split = a.split, kvh = a.kvh, g = a.group, tpt = a.tok_per_tile;
    const int n_doc = sd.kv_len - sd.n_q;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;
    const int tok_in = by_group(c, a.group_magic), head_in = c - tok_in * g; // token and head inside the tile
    const int tok_local = tile * tpt + tok_in;
    RowCtx rc;
    rc.valid = (c < tpt * g) && (tok_local < sd.n_q);
    rc.orow = (sd.q_row0 + tok_local) * a.n_q_heads + kvh * g + head_in;
    rc.key_lo = sd.kv_row0;
    rc.key_hi = sd.kv_row0 + n_doc + tok_local;
    const int slot = min(tok_in, 31);
    const int n_slots = by_group(31, a.group_magic) + 1;
    auto pos_of_slot = [&](int s) { return a.q_pos[sd.q_row0 + min(tile * tpt + s, sd.n_q - 1)]; };
    const int pos_lane = pos_of_slot(lane & (ROT_SLOTS - 1));

    const int first_tok = tile * tpt;
    const int last_tok = min(first_tok + tpt, sd.n_q) - 1;
    const int sb = sd.kv_row0 + split * sd.split_len;
    const int se = min(sb + sd.split_len, sd.kv_row0 + sd.kv_len);
    const int kt_begin = sb;
    const int kt_end = min(se, sd.kv_row0 + n_doc + last_tok + 1);
    const int key_clamp = sd.kv_row0 + sd.kv_len - 1;
    const int64_t row_elems = (int64_t)a.n_kv_heads * D;
    const int head_off = kvh * D;
    const __bf16* kp = (const __bf16*)a.k;
    const __bf16* vp = (const __bf16*)a.v;

    LDS_AS char* ring = smem + wave * (2 * UNIT); // this wave's unit of K, then its unit of V
    const uint32_t row_bytes = (uint32_t)row_elems * 2u;
    UnitLoads<D> ul((uint32_t)(uintptr_t)ring, row_bytes, (uint32_t)head_off * 2u, lane);
    auto unit_base = [&](const __bf16* base, int kt) { return (const char*)base + (int64_t)min(kt, key_clamp) * row_bytes; };
    const int own_begin = kt_begin + 32 * wave; // this wave's keys: 32 of every 128
    const int n_own = own_begin < kt_end ? (kt_end - own_begin + SHORT_KT - 1) / SHORT_KT : 0;

    ul.stay_within(key_clamp - min(own_begin, key_clamp), row_bytes, lane);
    // prologue: ordinary loads, then the first units, then the rotation (every wave rotates the same rows)
    double th = load_theta<TrPrefixArgs>(lane % (D / 2));
    __builtin_amdgcn_sched_barrier(0);
    u32x4 raw[D / 16];
    load_q_raw<D>((const __bf16*)a.q, rc, h, raw);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < LPU; ++i) ul.k(unit_base(kp, own_begin), i);
#pragma unroll
    for (int i = 0; i < LPU; ++i) ul.v(unit_base(vp, own_begin), i);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 qf[D / 16];
    {
        LDS_AS char* tab = smem + short_ring_bytes<D>() + wave * (ROT_SLOTS * 4 * D);
        rotate_queries<D, HALF, 2 * LPU>(raw, tab, th, pos_lane, lane, h, slot, n_slots, a.scale_log2e, pos_of_slot, qf);
    }

    Acc<D> acc;
    acc.clear();

    short_units<D>((const char*)kp, (const char*)vp, ul, rc, qf, own_begin, n_own, key_clamp, sd.kv_row0 + n_doc + first_tok, row_bytes, lane, acc);

    // merge the four key slices: every wave parks (m, l) and its unnormalised O in LDS
    constexpr int ROWB = short_merge_row_bytes<D>();
    const float l_tot = acc.l + __shfl_xor(acc.l, 32);
    // All waves are done with their units, and nothing is on its way to them: a wave whose keys lie behind its tokens' causal
    // end walks none, and its first unit, requested all the same, must not land on the rows parked here.
    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    LDS_AS char* obuf = smem + wave * (32 * ROWB);
    LDS_AS float* mlbuf = (LDS_AS float*)(smem + NW * 32 * ROWB);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            f32x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = acc.o[db][4 * q4 + e];
            *(LDS_AS f32x4*)(obuf + c * ROWB + (32 * db + 8 * q4 + 4 * h) * 4) = x;
        }
    if (h == 0) {
        mlbuf[(wave * 32 + c) * 2] = l_tot > 0.0f ? acc.mref() : -INFINITY;
        mlbuf[(wave * 32 + c) * 2 + 1] = l_tot;
    }
    __syncthreads();
    // thread -> (row r, D/8 consecutive channels)
    constexpr int CPT = D / 8;
    const int r = tid >> 3, j = tid & 7;
    float mw[NW], lw[NW], M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        mw[w] = mlbuf[(w * 32 + r) * 2];
        lw[w] = mlbuf[(w * 32 + r) * 2 + 1];
        M = fmaxf(M, mw[w]);
    }
    float L = 0.0f, ww[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        ww[w] = (mw[w] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mw[w] - M);
        L += ww[w] * lw[w];
    }
    float o[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) o[e] = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int e4 = 0; e4 < CPT / 4; ++e4) {
            const f32x4 x = *(LDS_AS const f32x4*)(smem + w * (32 * ROWB) + r * ROWB + (CPT * j + 4 * e4) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[4 * e4 + e] += ww[w] * x[e];
        }
    const int r_in = by_group(r, a.group_magic), r_head = r - r_in * g;
    const int r_tok = tile * tpt + r_in;
    const bool r_valid = (r < tpt * g) && (r_tok < sd.n_q);
    if (!r_valid) return;
    const float inv = L > 0.0f ? 1.0f / L : 0.0f;
    if (sd.n_split == 1) {
        __bf16* op = (__bf16*)a.out + ((int64_t)(sd.q_row0 + r_tok) * a.n_q_heads + kvh * g + r_head) * D + CPT * j;
#pragma unroll
        for (int e4 = 0; e4 < CPT / 4; ++e4) {
            bf16x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (__bf16)(o[4 * e4 + e] * inv);
            *(bf16x4_any*)(op + 4 * e4) = y;
        }
    } else {
        const int rows_s = sd.n_q * g;
        const int64_t prow = (int64_t)sd.ws_row0 + (int64_t)(split * a.n_kv_heads + kvh) * rows_s + r_tok * g + r_head;
        const int64_t at = prow * D + CPT * j;
        f32x4 x[CPT / 4];
#pragma unroll
        for (int e4 = 0; e4 < CPT / 4; ++e4)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e4][e] = o[4 * e4 + e] * inv;
        if (a.partial_f32) {
#pragma unroll
            for (int e4 = 0; e4 < CPT / 4; ++e4) *(f32x4*)((float*)a.ws_o + at + 4 * e4) = x[e4];
        } else {
#pragma unroll
            for (int e4 = 0; e4 < CPT / 4; ++e4) *(f16x4*)(a.ws_o + at + 4 * e4) = __builtin_convertvector(x[e4], f16x4);
        }
        if (j == 0) *(float2*)(a.ws_ml + prow * 2) = make_float2(L > 0.0f ? M : -INFINITY, L);
    }
}

// Merge the split-KV partial results: out = sum_s w_s l_s P_s / sum_s w_s l_s with w_s = 2^(m_s - max_s m_s) and
// P_s = O_s / l_s the normalised partial of split s.
// A lane owns eight channels of a row (one 16-byte piece of each partial, 16 or 8 lanes per row) and the statistics of every
// LPR-th split.  A merge is a chain of latencies, so the first round of partials is requested together with the statistics
// and before the reductions over the row, which run on the vector unit's cross-lane path.  (Half a wave per row, the
// reductions as LDS permutes with the partials behind them, and a 64-bit division took 15.4 us for 39.8 k
// rows of a serving batch, now 11.1; 6.4 for 8.2 k rows, now 5.6; 4.2 for 1.8 k, now 4.0.)
// SPLITS: statistics a row's lanes hold; 32 unless some request of the launch has more key splits.
// GROUPS: sets of D/8 lanes that share a row, each merging every GROUPS-th split.  A lane spends sixteen vector instructions
// on a partial, so one group walks 64 splits in some 2 us of issue alone (49 splits of 32 rows: 7.3 us, with half a wave of
// four-channel lanes 7.8, with a whole wave of four groups 4.9).
// F32: the partials are fp32, not fp16.
template <bool MAX, int LANES> __device__ __forceinline__ float row_reduce(float x)
{
    static_assert(LANES == 8 || LANES == 16 || LANES == 64, "");
    auto step = [&](int y) { return MAX ? fmaxf(x, __builtin_bit_cast(float, y)) : x + __builtin_bit_cast(float, y); };
    auto bits = [&]() { return __builtin_bit_cast(int, x); };
    x = step(__builtin_amdgcn_update_dpp(bits(), bits(), 0xB1, 0xf, 0xf, false));  // quad_perm [1,0,3,2]
    x = step(__builtin_amdgcn_update_dpp(bits(), bits(), 0x4E, 0xf, 0xf, false));  // quad_perm [2,3,0,1]
    x = step(__builtin_amdgcn_update_dpp(bits(), bits(), 0x141, 0xf, 0xf, false)); // row_half_mirror
    if (LANES >= 16) x = step(__builtin_amdgcn_update_dpp(bits(), bits(), 0x140, 0xf, 0xf, false)); // row_mirror
    if (LANES == 64) {
        x = step(__shfl_xor(bits(), 16));
        x = step(__shfl_xor(bits(), 32));
    }
    return x;
}
constexpr int COMBINE_THREADS = 128; // two waves: the few thousand rows of one request then reach every compute unit
template <int D, int GROUPS> constexpr int combine_rows() { return COMBINE_THREADS / (D / 8 * GROUPS); } // output rows per workgroup

template <int D, int SPLITS, int GROUPS, bool F32>
__global__ __launch_bounds__(COMBINE_THREADS) void combine_kernel(const TrPrefixArgs a, int total_rows)
{
    constexpr int LPG = D / 8, LPR = LPG * GROUPS; // lanes per group and per row
    constexpr int NK = SPLITS / LPR;               // statistics per lane
    constexpr int PER_ROUND = 8;                   // partials in flight per lane
    static_assert(LPR <= 64 && NK >= 1 && SPLITS / GROUPS % PER_ROUND == 0, "");
    const int lane = threadIdx.x & 63, lane_r = lane % LPR, grp = lane_r / LPG, piece = lane % LPG;
    const uint32_t R = blockIdx.x * combine_rows<D, GROUPS>() + threadIdx.x / LPR;
    const int tq = a.seq[0].q_row0 + (int)(R / (uint32_t)a.n_q_heads);
    const int hq = (int)(R % (uint32_t)a.n_q_heads);
    // the wave's rows ascend, so they belong to the requests from s0 to s1, nearly always one
    int s0 = 0, s1 = 0;
    if (a.n_seq > 1) {
        auto first = [&](int i) { return a.seq[i].q_row0; };
        s0 = last_not_above(a.n_seq, __builtin_amdgcn_readlane(tq, 0), first);
        s1 = last_not_above(a.n_seq, __builtin_amdgcn_readlane(tq, 63), first);
    }
    if (R >= (uint32_t)total_rows) return;
    int n_split = a.seq[s0].n_split, ws_row0 = a.seq[s0].ws_row0, n_q = a.seq[s0].n_q, q_row0 = a.seq[s0].q_row0;
    if (s0 != s1) {
        int sq = s0;
        while (sq < s1 && a.seq[sq + 1].q_row0 <= tq) ++sq;
        n_split = a.seq[sq].n_split;
        ws_row0 = a.seq[sq].ws_row0;
        n_q = a.seq[sq].n_q;
        q_row0 = a.seq[sq].q_row0;
    }
    if (n_split == 1) return;
    const int g = a.group;
    const int kvh = hq / g;
    const int64_t rows_s = (int64_t)n_q * g;
    const int64_t prow0 = (int64_t)ws_row0 + kvh * rows_s + (tq - q_row0) * g + hq % g;
    const int64_t pstride = (int64_t)a.n_kv_heads * rows_s; // partial rows between consecutive splits
    float2 ml[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        ml[k] = make_float2(-INFINITY, 0.0f);
        if (lane_r + LPR * k < n_split) ml[k] = *(const float2*)(a.ws_ml + (prow0 + (lane_r + LPR * k) * pstride) * 2);
    }
    typedef std::conditional_t<F32, float, _Float16> PART;
    typedef PART Piece __attribute__((ext_vector_type(8)));
    const PART* base = (const PART*)a.ws_o + prow0 * D + 8 * piece;
    Piece x[PER_ROUND];
    auto load = [&](int j0) { // the group's j-th split is GROUPS j + grp; splits past the last one give zeros
#pragma unroll
        for (int u = 0; u < PER_ROUND; ++u) {
            const int sp = GROUPS * (j0 + u) + grp;
            x[u] = Piece{};
            if (sp < n_split) x[u] = *(const Piece*)(base + sp * pstride * D);
        }
    };
    load(0);
    float M = ml[0].x;
#pragma unroll
    for (int k = 1; k < NK; ++k) M = fmaxf(M, ml[k].x);
    M = row_reduce<true, LPR>(M);
    float w[NK], L = 0.0f;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        w[k] = ml[k].x == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(ml[k].x - M) * ml[k].y;
        L += w[k];
    }
    L = row_reduce<false, LPR>(L);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    const int row_lane0 = lane - lane_r; // first lane of this row
#pragma unroll
    for (int j0 = 0; j0 < SPLITS / GROUPS; j0 += PER_ROUND) {
        if (GROUPS * j0 >= n_split) break;
        if (j0 > 0) load(j0);
#pragma unroll
        for (int u = 0; u < PER_ROUND; ++u) {
            const int sp = GROUPS * (j0 + u); // + grp, which stays below LPR: the same statistics register for all groups
            const float ws = __shfl(w[sp / LPR], row_lane0 + sp % LPR + grp); // zero past the last split
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += ws * (float)x[u][e];
        }
    }
    if (GROUPS > 1) {
#pragma unroll
        for (int o = LPG; o < LPR; o <<= 1)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], o);
        if (grp != 0) return;
    }
    const float inv = L > 0.0f ? 1.0f / L : 0.0f; // a row without any weight is zero, as in a launch that is not cut
    bf16x8 y;
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = (__bf16)(acc[e] * inv);
    *(u32x4_any*)((__bf16*)a.out + ((int64_t)tq * a.n_q_heads + hq) * D + 8 * piece) = __builtin_bit_cast(u32x4, y);
}

// ---- step 2 (offline): block-diagonal causal attention over packed chunks --------------------------------------
// First row of the chunk that owns token t.  Clamped into [0, t] so that a cu_chunk_lens array that does not cover
// every token can only give wrong numbers, never an access outside the tensors.
__device__ __forceinline__ int chunk_start(const int32_t* tok_start, int t) { return min(max(tok_start[t], 0), t); }

template <int D, int NW, int NS, bool HALF>
__global__ __launch_bounds__(64 * NW, 2) void blockdiag_attn_kernel(const TrBlockDiagArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) char smem_raw[];
    LDS_AS char* smem = (LDS_AS char*)smem_raw;
    const int item = xcd_remap(blockIdx.x, a.items_per_head * a.n_kv_heads);
    const int kvh = item / a.items_per_head;
    const int j = item % a.items_per_head;
    const TrBdSeg sg = a.seg[last_not_above(a.n_seg, j, [&](int i) { return a.seg[i].item0; })];
    // last row tiles first: under a causal mask they walk the most keys (a query behind the documents walks all of
    // them), so they must not be the ones that start last
    const int tile = sg.tile_hi - (j - sg.item0) / sg.n_split;
    const int split = (j - sg.item0) % sg.n_split;
    const int g = a.group, tpt = a.tok_per_tile;
    const int T = a.total_tokens;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31;
    const int rl = 32 * wave + c;
    const int tok_in = by_group(rl, a.group_magic), head_in = rl - tok_in * g; // token and head inside the tile
    const int t = tile * tpt + tok_in;
    RowCtx rc;
    rc.valid = (rl < tpt * g) && (t < T);
    rc.orow = t * a.n_q_heads + kvh * g + head_in;
    rc.key_hi = t;
    const int wave_in = by_group(32 * wave, a.group_magic); // first token of the wave
    const int wave_t0 = tile * tpt + wave_in;
    const int slot = min(tok_in - wave_in, 31);
    const int n_slots = by_group(32 * wave + 31, a.group_magic) - wave_in + 1;
    const int t_first = tile * tpt;
    const int t_last = min(t_first + tpt, T) - 1;
    // One batch of loads, nothing waited for in between: this row's chunk start, the position id (or chunk start) of
    // the lane's token slot, the chunk start of the tile's token `lane` (tokens 64 and up of a tile, which only small
    // GQA groups have, follow below), then theta and the raw query rows.  Indices are clamped instead of branched on.
    const int ts_lane = min(wave_t0 + (lane & (ROT_SLOTS - 1)), T - 1);
    const int start_row_raw = a.tok_start[min(t, T - 1)];
    const int slot_raw = a.pos ? a.pos[ts_lane] : a.tok_start[ts_lane];
    const int start_tile_raw = a.tok_start[min(t_first + lane, t_last)];
    __builtin_amdgcn_sched_barrier(0);
    QLoads<D> ql;
    issue_q_loads<D, TrBlockDiagArgs>((const __bf16*)a.q, rc, ql);

    rc.key_lo = rc.valid ? min(max(start_row_raw, 0), t) : 0;
    // position id of each token slot of this wave: given, or chunk-local
    auto pos_of_slot = [&](int s) {
        const int ts = min(wave_t0 + s, T - 1);
        return a.pos ? a.pos[ts] : ts - chunk_start(a.tok_start, ts);
    };
    const int pos_lane = a.pos ? slot_raw : ts_lane - min(max(slot_raw, 0), ts_lane);

    // first row any token of the tile attends, and the largest such start (tiles below it need the lower mask);
    // the starts need not be monotone: a query token behind the documents starts at row 0 again
    int lo_first = INT32_MAX, lo_last = 0;
    if (t_first + lane <= t_last) lo_first = lo_last = min(max(start_tile_raw, 0), t_first + lane);
    for (int tt = t_first + 64 + lane; tt <= t_last; tt += 64) {
        const int st = chunk_start(a.tok_start, tt);
        lo_first = min(lo_first, st);
        lo_last = max(lo_last, st);
    }
    lo_first = wave_min_i(lo_first);
    lo_last = wave_max_i(lo_last);
    // this item's piece of the walk [lo_first, t_last]: pieces of split_len keys, the last one open-ended
    int kb = lo_first, ke = t_last + 1;
    if (sg.n_split > 1) {
        const int64_t kb64 = (int64_t)lo_first + (int64_t)split * sg.split_len;
        kb = (int)(kb64 < ke ? kb64 : ke);
        if (split + 1 < sg.n_split && (int64_t)kb + sg.split_len < ke) ke = kb + sg.split_len;
    }
    const Walk w = make_walk(kb, ke, T - 1, a.n_kv_heads, kvh, D);

    const TileLoads<D, NW> tl(w, smem, wave, lane);
    bf16x8 qf[D / 16];
    prologue<D, NW, NS, HALF>((const __bf16*)a.k, (const __bf16*)a.v, w, tl, ql, pos_lane, slot, n_slots, pos_of_slot, a.scale_log2e, smem, qf);

    Acc<D> acc;
    acc.clear();

    attn_tiles<D, NW, NS>((const __bf16*)a.k, (const __bf16*)a.v, w, tl, rc, qf, t_first, lo_last, smem, acc);

    const float l_tot = acc.l + __shfl_xor(acc.l, 32);
    if (sg.n_split == 1) {
        store_rows<D, false>(acc, l_tot, rc.valid, (int64_t)rc.orow, a.out, lane);
    } else { // the layout the merge kernel reads: [split][KV head][token of the segment x group]
        const int64_t rows_s = (int64_t)sg.n_tok * g;
        const int64_t prow = (int64_t)sg.ws_row0 + ((int64_t)split * a.n_kv_heads + kvh) * rows_s + (int64_t)(t - sg.tok0) * g + head_in;
        store_rows<D, true>(acc, l_tot, rc.valid, prow, a.ws_o, lane);
        if (rc.valid && lane < 32) *(float2*)(a.ws_ml + prow * 2) = make_float2(l_tot > 0.0f ? acc.mref() : -INFINITY, l_tot);
    }
}

template <int D, int NW, int NS> constexpr int smem_bytes()
{
    return NS * Geo<D>::STAGE_BYTES;
}

template <int D, int NW, int NS, bool HALF, int AUX = 0>
int launch_prefix(const TrPrefixArgs& a, hipStream_t s)
{
    auto kern = prefix_attn_kernel<D, NW, NS, HALF, AUX>;
    constexpr int lds = smem_bytes<D, NW, NS>();
    static std::atomic<uint64_t> configured{0};
    if (int rc = tr_raise_lds_limit((const void*)kern, lds, &configured)) return rc;
    hipLaunchKernelGGL(kern, dim3(a.n_items), dim3(64 * NW), lds, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

template <int D, bool HALF>
int launch_short(const TrPrefixArgs& a, hipStream_t s)
{
    auto kern = short_attn_kernel<D, HALF>;
    constexpr int ring = short_ring_bytes<D>() + short_tables_bytes<D>();
    constexpr int merge = SHORT_NW * 32 * short_merge_row_bytes<D>() + SHORT_NW * 32 * 8;
    constexpr int lds = ring > merge ? ring : merge;
    static std::atomic<uint64_t> configured{0};
    static_assert(2 * lds <= 160 * 1024, "two workgroups fit a CU");
    if (int rc = tr_raise_lds_limit((const void*)kern, lds, &configured)) return rc;
    hipLaunchKernelGGL(kern, dim3(a.n_items), dim3(64 * SHORT_NW), lds, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

template <int D, bool HALF>
int launch_gather(const TrGatherArgs& a, hipStream_t s)
{
    auto kern = gather_attn_kernel<D, HALF>;
    constexpr int lds = gather_lds_bytes<D>();
    static std::atomic<uint64_t> configured{0};
    if (int rc = tr_raise_lds_limit((const void*)kern, lds, &configured)) return rc;
    hipLaunchKernelGGL(kern, dim3(a.n_items), dim3(64 * GATHER_NW), lds, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

template <int D, int NW, int NS, bool HALF>
int launch_blockdiag(const TrBlockDiagArgs& a, hipStream_t s)
{
    auto kern = blockdiag_attn_kernel<D, NW, NS, HALF>;
    constexpr int lds = smem_bytes<D, NW, NS>();
    static std::atomic<uint64_t> configured{0};
    if (int rc = tr_raise_lds_limit((const void*)kern, lds, &configured)) return rc;
    hipLaunchKernelGGL(kern, dim3(a.items_per_head * a.n_kv_heads), dim3(64 * NW), lds, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

template <bool HALF>
int prefix_dispatch(const TrPrefixArgs& a, int head_dim, int wg_rows, hipStream_t s)
{
    if (wg_rows == 32) return head_dim == 128 ? launch_short<128, HALF>(a, s) : launch_short<64, HALF>(a, s);
    if (wg_rows == 128) {
        bool one_tile = true; // every request fits one row tile: its keys are read once
        for (int i = 0; i < a.n_seq; ++i) one_tile = one_tile && a.seq[i].n_tiles == 1;
        if (one_tile)
            return head_dim == 128 ? launch_prefix<128, 4, 2, HALF, DMA_STREAM>(a, s) : launch_prefix<64, 4, 2, HALF, DMA_STREAM>(a, s);
    }
    if (head_dim == 128) return wg_rows == 256 ? launch_prefix<128, 8, 4, HALF>(a, s) : launch_prefix<128, 4, 2, HALF>(a, s);
    return wg_rows == 256 ? launch_prefix<64, 8, 4, HALF>(a, s) : launch_prefix<64, 4, 2, HALF>(a, s);
}

template <bool HALF>
int blockdiag_dispatch(const TrBlockDiagArgs& a, int head_dim, int wg_rows, hipStream_t s)
{
    if (head_dim == 128) return wg_rows == 256 ? launch_blockdiag<128, 8, 4, HALF>(a, s) : launch_blockdiag<128, 4, 2, HALF>(a, s);
    return wg_rows == 256 ? launch_blockdiag<64, 8, 4, HALF>(a, s) : launch_blockdiag<64, 4, 2, HALF>(a, s);
}

} // namespace

// the merge kernel for a launch of total_rows output rows
template <int D, int SPLITS, int GROUPS> static void launch_combine_d(const TrPrefixArgs& a, int total_rows, hipStream_t s)
{
    constexpr int per_block = combine_rows<D, GROUPS>();
    auto kern = a.partial_f32 ? combine_kernel<D, SPLITS, GROUPS, true> : combine_kernel<D, SPLITS, GROUPS, false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(((int64_t)total_rows + per_block - 1) / per_block)), dim3(COMBINE_THREADS), 0, s, a, total_rows);
}
// A wave for each row where lanes of one group would walk the splits in more than one round of eight, one after the other,
// while most of the chip is idle; D/8 lanes per row elsewhere.  A wave for each row against lanes, difference of the whole
// attention call in us on a fresh cache and workspace (mean over heads and layouts of rows): 6 .. 8 splits +0.04 .. +0.28 at
// any count of rows, 10 splits -0.28 .. -0.63 up to 1024 rows, 16 splits -0.36 .. -0.69, 20 splits -0.8 .. -1.1.  Of more
// rows the lanes fill the chip: merge alone, lanes / wave, 12 splits of 2048 rows 4.7 / 4.8, 16 splits of 2048 rows of 64
// 4.1 / 4.9, 17 splits 5.0 / 5.0, 24 splits 5.4 / 5.1; 24 splits of 3584 rows 6.0 / 6.0, 49 splits 10.6 / 11.2.
static bool combine_by_waves(int splits, int rows) { return splits > 8 && rows <= (splits > 16 ? 2048 : 1024); }
static int launch_combine(const TrPrefixArgs& a, int head_dim, int total_rows, hipStream_t s)
{
    int max_split = 1;
    for (int i = 0; i < a.n_seq; ++i) max_split = a.seq[i].n_split > max_split ? a.seq[i].n_split : max_split;
    if (combine_by_waves(max_split, total_rows)) {
        if (head_dim == 128) launch_combine_d<128, 64, 4>(a, total_rows, s);
        else launch_combine_d<64, 64, 8>(a, total_rows, s);
    } else if (max_split > 32) {
        if (head_dim == 128) launch_combine_d<128, 64, 1>(a, total_rows, s);
        else launch_combine_d<64, 64, 1>(a, total_rows, s);
    } else {
        if (head_dim == 128) launch_combine_d<128, 32, 1>(a, total_rows, s);
        else launch_combine_d<64, 32, 1>(a, total_rows, s);
    }
    TR_HIP(hipGetLastError());
    return TR_OK;
}

// wg_rows: 128 (4 waves, 2-stage ring, two workgroups per CU), 256 (8 waves, 4-stage ring, one per CU) or 32 (the
// short-query kernel: 4 waves share 32 rows and split the keys)
int tr_launch_prefix_attn(const TrPrefixArgs& a, int head_dim, int wg_rows, bool any_split, int total_rows, hipStream_t s)
{
    if (a.n_items <= 0) return TR_OK;
    const int rc = a.rope_half ? prefix_dispatch<true>(a, head_dim, wg_rows, s) : prefix_dispatch<false>(a, head_dim, wg_rows, s);
    if (rc) return rc;
    if (any_split) {
        if (int rc2 = launch_combine(a, head_dim, total_rows, s)) return rc2;
    }
    return TR_OK;
}

int tr_launch_gather_attn(const TrGatherArgs& a, const TrPrefixArgs& combine_args, int head_dim, hipStream_t s)
{
    if (a.n_items <= 0) return TR_OK;
    int rc;
    if (a.rope_half) rc = head_dim == 128 ? launch_gather<128, true>(a, s) : launch_gather<64, true>(a, s);
    else rc = head_dim == 128 ? launch_gather<128, false>(a, s) : launch_gather<64, false>(a, s);
    if (rc) return rc;
    if (a.n_split > 1) {
        const int total_rows = a.n_q * a.n_q_heads;
        if (int rc2 = launch_combine(combine_args, head_dim, total_rows, s)) return rc2;
    }
    return TR_OK;
}

int tr_launch_blockdiag_attn(const TrBlockDiagArgs& a, const TrPrefixArgs* combine, int combine_rows, int head_dim, int wg_rows,
                             hipStream_t s)
{
    if (a.total_tokens <= 0) return TR_OK;
    const int rc = a.rope_half ? blockdiag_dispatch<true>(a, head_dim, wg_rows, s) : blockdiag_dispatch<false>(a, head_dim, wg_rows, s);
    if (rc) return rc;
    if (combine && combine_rows > 0) {
        if (int rc2 = launch_combine(*combine, head_dim, combine_rows, s)) return rc2;
    }
    return TR_OK;
}
