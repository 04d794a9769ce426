// Bandwidth-bound kernels: KV-cache formation (gather + per-chunk RoPE re-rotation), query append,
// and the offline key rotation.  All key rotations are computed in fp64 and rounded once to the
// storage type, so the rotated keys are reproducible to the last bit against an fp64 definition.
#include "tr_internal.h"
#include <type_traits>

namespace {

// ---- storage helpers ------------------------------------------------------------------------------------

__device__ __forceinline__ double bf16_bits_to_double(uint32_t b16)
{
    return (double)__uint_as_float(b16 << 16);
}

// double -> bf16 with a single rounding (nearest, ties to even).  By way of fp32 a value is rounded twice, and that goes wrong
// only where the first step lands on a tie of the second: bf16's ties are fp32 numbers, so the first step moves no value past
// one.  Ties, subnormals and NaN (which becomes 0x7fc0) are therefore left to the slow form: truncate to fp32, sticky bit, round.
// A lane that meets one redoes its unit, about one in 8000.  us with integer arithmetic on every value's bit pattern (some 14
// instructions each instead of 4) / this: five appended tokens and attention 17.4 / 16.7, 6200 rows of un-rotated keys and
// 37 query tokens 28.0 / 27.7, 32 x 1024 + 256 tokens in one pass 505 / 500.
__device__ __forceinline__ uint32_t double_to_bf16_bits_slow(double y)
{
    float f = __double2float_rz(y);
    uint32_t u = __float_as_uint(f);
    u |= ((double)f != y) ? 1u : 0u;
    if (y != y) return 0x7fc0u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
struct Bf16Fast { // two values to a word; `redo` is set where the slow form has to
    bool redo = false;
    __device__ __forceinline__ float to_f32(double y)
    {
        const float f = __double2float_rn(y);
        redo |= (uint16_t)__float_as_uint(f) == 0x8000u || __builtin_isfpclass(f, 0x0003 | 0x0010 | 0x0080); // NaN, subnormal
        return f;
    }
    __device__ __forceinline__ uint32_t pack(double lo, double hi)
    {
        bf16x2 t;
        t[0] = (__bf16)to_f32(lo);
        t[1] = (__bf16)to_f32(hi);
        return __builtin_bit_cast(uint32_t, t);
    }
};
struct Bf16Slow {
    __device__ __forceinline__ uint32_t pack(double lo, double hi) { return double_to_bf16_bits_slow(lo) | (double_to_bf16_bits_slow(hi) << 16); }
};

// y = R(angle) x on one pair, unfused multiplies and adds (the order Eq. 3 is written in)
__device__ __forceinline__ void rotate_pair(double xa, double xb, double c, double s, double& ya, double& yb)
{
    ya = __dsub_rn(__dmul_rn(xa, c), __dmul_rn(xb, s));
    yb = __dadd_rn(__dmul_rn(xb, c), __dmul_rn(xa, s));
}

template <int DTYPE> struct Unit; // one 16-byte unit of a row

template <> struct Unit<TR_BF16> {
    static constexpr int PAIRS = 4;
    template <class Round> __device__ static __forceinline__ uint4 rotate_by(Round& round, uint4 x, const double* c, const double* s)
    {
        uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            double xa = bf16_bits_to_double(w[p] & 0xffffu), xb = bf16_bits_to_double(w[p] >> 16);
            double ya, yb;
            rotate_pair(xa, xb, c[p], s[p], ya, yb);
            w[p] = round.pack(ya, yb);
        }
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
    __device__ static __forceinline__ uint4 rotate(uint4 x, const double* c, const double* s)
    {
        Bf16Fast fast;
        uint4 y = rotate_by(fast, x, c, s);
        if (__builtin_expect(fast.redo, 0)) {
            Bf16Slow slow;
            y = rotate_by(slow, x, c, s);
        }
        return y;
    }
};

// Half-split layout: channel c < d/2 pairs with c + d/2, so a unit of the low half pairs element by element with
// the unit d/2 channels further on.  me / partner: the two units, low: whether `me` is the low half; c, s: the
// (cos, sin) of the ELEMS pair indices the unit covers.  y_lo = x_lo c - x_hi s, y_hi = x_hi c + x_lo s.
template <int DTYPE> struct UnitHalf;
template <> struct UnitHalf<TR_BF16> {
    static constexpr int ELEMS = 8;
    template <class Round>
    __device__ static __forceinline__ uint4 rotate_by(Round& round, uint4 me, uint4 partner, bool low, const double* c, const double* s)
    {
        uint32_t a[4] = {me.x, me.y, me.z, me.w}, b[4] = {partner.x, partner.y, partner.z, partner.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            double r[2];
#pragma unroll
            for (int hw = 0; hw < 2; ++hw) {
                const double xm = bf16_bits_to_double(hw ? a[p] >> 16 : a[p] & 0xffffu);
                const double xp = bf16_bits_to_double(hw ? b[p] >> 16 : b[p] & 0xffffu);
                const double t0 = __dmul_rn(xm, c[2 * p + hw]), t1 = __dmul_rn(xp, s[2 * p + hw]);
                r[hw] = low ? __dsub_rn(t0, t1) : __dadd_rn(t0, t1);
            }
            a[p] = round.pack(r[0], r[1]);
        }
        return make_uint4(a[0], a[1], a[2], a[3]);
    }
    __device__ static __forceinline__ uint4 rotate(uint4 me, uint4 partner, bool low, const double* c, const double* s)
    {
        Bf16Fast fast;
        uint4 y = rotate_by(fast, me, partner, low, c, s);
        if (__builtin_expect(fast.redo, 0)) {
            Bf16Slow slow;
            y = rotate_by(slow, me, partner, low, c, s);
        }
        return y;
    }
};
template <> struct UnitHalf<TR_F32> {
    static constexpr int ELEMS = 4;
    __device__ static __forceinline__ uint4 rotate(uint4 me, uint4 partner, bool low, const double* c, const double* s)
    {
        uint32_t a[4] = {me.x, me.y, me.z, me.w}, b[4] = {partner.x, partner.y, partner.z, partner.w};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double t0 = __dmul_rn((double)__uint_as_float(a[p]), c[p]), t1 = __dmul_rn((double)__uint_as_float(b[p]), s[p]);
            a[p] = __float_as_uint(__double2float_rn(low ? __dsub_rn(t0, t1) : __dadd_rn(t0, t1)));
        }
        return make_uint4(a[0], a[1], a[2], a[3]);
    }
};
__device__ __forceinline__ uint4 shfl_xor_u4(uint4 x, int mask)
{
    return make_uint4(__shfl_xor(x.x, mask), __shfl_xor(x.y, mask), __shfl_xor(x.z, mask), __shfl_xor(x.w, mask));
}

template <> struct Unit<TR_F32> {
    static constexpr int PAIRS = 2;
    __device__ static __forceinline__ uint4 rotate(uint4 x, const double* c, const double* s)
    {
        uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            double xa = (double)__uint_as_float(w[2 * p]), xb = (double)__uint_as_float(w[2 * p + 1]);
            double ya, yb;
            rotate_pair(xa, xb, c[p], s[p], ya, yb);
            w[2 * p] = __float_as_uint(__double2float_rn(ya));
            w[2 * p + 1] = __float_as_uint(__double2float_rn(yb));
        }
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// streaming (read-once) 16-byte load
__device__ __forceinline__ uint4 ld_stream(const uint4* p)
{
    const u32x4 r = __builtin_nontemporal_load((const u32x4*)p);
    return make_uint4(r[0], r[1], r[2], r[3]);
}

// The append's 16-byte accesses, for rows that start at any multiple of an element: the caller's tensors may be views.  The
// vector memory path serves such an address with one instruction (the target's unaligned access mode, which lets the
// compiler emit the same wide accesses as for aligned rows).
typedef u32x4 u32x4_any __attribute__((aligned(2)));
__device__ __forceinline__ uint4 ld_stream_any(const uint4* p)
{
    const u32x4 r = __builtin_nontemporal_load((const u32x4_any*)p);
    return make_uint4(r[0], r[1], r[2], r[3]);
}
__device__ __forceinline__ void st_any(uint4* p, uint4 x) { *(u32x4_any*)p = u32x4{x.x, x.y, x.z, x.w}; }

// ---- one row of the query append: K' rotated at its position id, V copied, for every KV head -----------------
// A group of half_dim lanes (a wave at 128 channels, half of one at 64) owns two 16-byte units per lane of a token's row; a
// longer row has several groups.  Lane m computes (cos, sin) of pair m once, with the loads on their way, parks it in LDS, and
// the lanes rotate their units.  half_dim is a multiple of the units per head, so a lane keeps its unit position, hence its pairs.  Nothing is
// shared between groups, so there is no barrier: the only dependent chain is load, angle, rotate, store, and its length
// does not grow with the row: the angles a long row computes again cost less than a second trip.
// Measured, every call on fresh rows (us, one group per row with four units per lane and as many trips as the row needs /
// this): bf16, 8 heads of 128, 30000 rows 53.8 (a thread per unit position) / 47.0; replayed on the same rows: 40 heads of
// 128, 64 rows 10.1 / 4.6, 1024 rows 13.7 / 9.4; fp32, 40 heads of 128, 1024 rows 25.4 / 14.6; bf16, one head of 64, 256
// rows (a whole wave per token) 4.25 / 3.9.
constexpr int APPEND_WAVES = TR_APPEND_WAVES_PER_BLOCK;
constexpr int APPEND_UNITS = TR_APPEND_UNITS; // 16-byte units of K (and of V) a lane has in flight

template <int DTYPE, bool HALF>
__device__ __forceinline__ void append_token(const void* k_new, const void* v_new, int pos, void* cache_k, void* cache_v, int row_units,
                                             int head_units, int half_dim, const double* theta, int64_t src_row, int64_t dst_row, int part,
                                             double2* cs /* LDS, this group's half_dim entries */, int lane /* in the group */)
{
    const uint4* ks = (const uint4*)k_new + src_row * row_units;
    const uint4* vs = (const uint4*)v_new + src_row * row_units;
    uint4* kd = (uint4*)cache_k + dst_row * row_units;
    uint4* vd = (uint4*)cache_v + dst_row * row_units;
    constexpr int N_CS = HALF ? UnitHalf<DTYPE>::ELEMS : Unit<DTYPE>::PAIRS; // pairs a unit takes part in
    const int hu = lane % head_units, hmask = head_units >> 1;
    const bool low = hu < hmask;
    const int m0 = (HALF && !low ? hu - hmask : hu) * N_CS;
    const int u0 = part * APPEND_UNITS * half_dim + lane;
    uint4 kx[APPEND_UNITS], vx[APPEND_UNITS];
#pragma unroll
    for (int i = 0; i < APPEND_UNITS; ++i)
        if (u0 + half_dim * i < row_units) {
            kx[i] = ld_stream_any(ks + u0 + half_dim * i);
            if (v_new) vx[i] = ld_stream_any(vs + u0 + half_dim * i);
        }
    double sn, cn;
    tr_sincos((double)pos * theta[lane], &sn, &cn);
    cs[lane] = make_double2(cn, sn);
    // LDS serves a wave's accesses in order; only the compiler has to keep them so
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    double c[N_CS], s[N_CS];
#pragma unroll
    for (int p = 0; p < N_CS; ++p) {
        const double2 e = cs[m0 + p];
        c[p] = e.x;
        s[p] = e.y;
    }
#pragma unroll
    for (int i = 0; i < APPEND_UNITS; ++i)
        if (u0 + half_dim * i < row_units) { // rows are whole heads, so a lane and its partner's lane are here together
            uint4 y;
            if constexpr (HALF) y = UnitHalf<DTYPE>::rotate(kx[i], shfl_xor_u4(kx[i], hmask), low, c, s);
            else y = Unit<DTYPE>::rotate(kx[i], c, s);
            st_any(kd + u0 + half_dim * i, y);
            if (v_new) st_any(vd + u0 + half_dim * i, vx[i]); // v_new == NULL: keys only
        }
}

// ---- KV-cache formation: Sec. 3.4 step 5 with the reordered-position rotation of Sec. 3.2 -------------------
// A run of rows is contiguous in the store and in the cache, so a block moves a flat span of 16-byte
// units.  A thread's unit index modulo the units-per-head never changes while it strides by 256, hence
// the (cos, sin) of "its" pairs for this chunk's offset are loop constants.
constexpr int ASM_UNROLL = 4;

// How the rows that a launch forms are stored.  Ordinary stores leave their lines dirty in the L2s, which write them back when
// they need the room or when the kernel ends; device-scope stores go through at once, which shortens a launch that forms more
// than the L2s hold, but the attention behind it then finds none of the rows there.  us of whole requests on fresh stores and
// caches, ordinary / through, by MB of K and V: 8.4 MB 22.6 / 22.3, 16.8 MB 30.7 / 30.3, 21 MB 33.6 / 33.9, 25 MB 30.0 / 30.2,
// 34 MB 35.0 / 35.3, 67 MB 68.8 / 68.8, 134 MB 178.9 / 172.7, batches of 300 MB 237.9 / 230.6 and of 403 MB 223.2 / 204.0.
// So: through from 96 MB on.  Streamed stores make the copy alone fastest, and the requests slower on the whole: 2 tokens
// over 256 to 2048 rows 14.6 / 15.2 .. 17.5 / 18.1, over 8.4 MB from -0.7 us (128 tokens and more) to +0.3 (16 and fewer),
// over 34 MB 35.0 / 38.0.
enum StorePolicy { ST_CACHED, ST_THROUGH };
constexpr int64_t THROUGH_MIN_BYTES = 96ll << 20;

// One 16-byte unit, `unit` (at most a block's span) behind a base that is the same in every lane.
template <int POLICY> __device__ __forceinline__ void st_unit(uint4* base, int unit, uint4 x)
{
    const u32x4 w = {x.x, x.y, x.z, x.w};
    if constexpr (POLICY == ST_THROUGH)
        __builtin_amdgcn_raw_buffer_store_b128(w, __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00020000), unit * 16, 0, 16 /* sc1 */);
    else *(u32x4*)(base + unit) = w;
}

template <int DTYPE, bool HALF, int POLICY>
__global__ __launch_bounds__(256) void assemble_kernel(const TrAssembleArgs a)
{
    __shared__ double2 cs[64 * APPEND_WAVES]; // a copy block uses the first 64
    const int b = blockIdx.x;
    if (a.app.n_q > 0 && b >= a.app.first_block) {
        // tail blocks: the request's own query tokens
        const uint32_t grp = ((uint32_t)(b - a.app.first_block) * 256 + threadIdx.x) >> tr_append_shift(a.half_dim);
        const uint32_t parts = (uint32_t)tr_append_groups(a.row_units, a.half_dim);
        const int tok = (int)(parts == 1 ? grp : grp / parts), lane = threadIdx.x & (a.half_dim - 1);
        if (tok < a.app.n_q)
            append_token<DTYPE, HALF>(a.app.k_new, a.app.v_new, a.app.q_pos[tok], a.k_dst, a.v_dst, a.row_units, a.head_units, a.half_dim,
                                      a.theta, tok, (int64_t)a.app.dst_row0 + tok, (int)(grp - tok * parts), cs + (threadIdx.x - lane), lane);
        return;
    }
    int lo = 0, hi = a.n_desc - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (a.desc[mid].blk_start <= b) lo = mid; else hi = mid - 1;
    }
    const TrCopyDesc d = a.desc[lo];
    const int64_t run_units = (int64_t)d.n_rows * a.row_units;
    const int64_t u0 = (int64_t)(b - d.blk_start) * a.span_units;
    int64_t u1 = u0 + a.span_units;
    if (u1 > run_units) u1 = run_units;
    const int tid = threadIdx.x;

    const uint4* ks = (const uint4*)a.k_src + (int64_t)d.src_row * a.row_units;
    const uint4* vs = (const uint4*)a.v_src + (int64_t)d.src_row * a.row_units;
    uint4* kd = (uint4*)a.k_dst + (int64_t)d.dst_row * a.row_units;
    uint4* vd = (uint4*)a.v_dst + (int64_t)d.dst_row * a.row_units;

    // the first round of loads goes out before the angle work, which needs no data
    uint4 kx[ASM_UNROLL], vx[ASM_UNROLL];
    int64_t u = u0 + tid;
#pragma unroll
    for (int i = 0; i < ASM_UNROLL; ++i) {
        const int64_t uu = u + 256 * i;
        if (uu < u1) { kx[i] = ld_stream(ks + uu); vx[i] = ld_stream(vs + uu); }
    }

    constexpr int P = Unit<DTYPE>::PAIRS, E = UnitHalf<DTYPE>::ELEMS;
    double c[HALF ? E : P], s[HALF ? E : P];
    const bool rot = d.delta != 0;
    const int hu = (int)((u0 + tid) % a.head_units); // unit inside its head: the same for every unit this thread moves
    const int hmask = a.head_units >> 1;             // lane distance to the unit d/2 channels away
    const bool low = hu < hmask;
    if (rot) {
        if (tid < a.half_dim) {
            double sn, cn;
            tr_sincos((double)d.delta * a.theta[tid], &sn, &cn);
            cs[tid] = make_double2(cn, sn);
        }
        __syncthreads();
        if constexpr (HALF) {
            const int m0 = (low ? hu : hu - hmask) * E;
#pragma unroll
            for (int p = 0; p < E; ++p) { c[p] = cs[m0 + p].x; s[p] = cs[m0 + p].y; }
        } else {
            const int m0 = hu * P;
#pragma unroll
            for (int p = 0; p < P; ++p) { c[p] = cs[m0 + p].x; s[p] = cs[m0 + p].y; }
        }
    }

    while (u < u1) {
#pragma unroll
        for (int i = 0; i < ASM_UNROLL; ++i) {
            const int64_t uu = u + 256 * i;
            // the 16-byte units of one head sit in neighbouring lanes and runs are whole rows, so a lane and the lane
            // that holds its partner unit are always in this branch together
            if (uu < u1) {
                uint4 y = kx[i];
                if (rot) {
                    if constexpr (HALF) y = UnitHalf<DTYPE>::rotate(kx[i], shfl_xor_u4(kx[i], hmask), low, c, s);
                    else y = Unit<DTYPE>::rotate(kx[i], c, s);
                }
                st_unit<POLICY>(kd + u0, (int)(uu - u0), y);
                st_unit<POLICY>(vd + u0, (int)(uu - u0), vx[i]);
            }
        }
        u += 256 * ASM_UNROLL;
#pragma unroll
        for (int i = 0; i < ASM_UNROLL; ++i) {
            const int64_t uu = u + 256 * i;
            if (uu < u1) { kx[i] = ld_stream(ks + uu); vx[i] = ld_stream(vs + uu); }
        }
    }
}

// ---- query append: cache rows of the query tokens (K' rotated at q_pos, V copied) -------------------------
template <int DTYPE, bool HALF>
__global__ __launch_bounds__(64 * APPEND_WAVES) void append_kernel(const TrAppendArgs a)
{
    __shared__ double2 cs[64 * APPEND_WAVES];
    const int half_dim = a.head_dim >> 1, shift = tr_append_shift(half_dim);
    const int head_units = a.head_dim * (DTYPE == TR_BF16 ? 2 : 4) / 16; // a power of two, at most 32
    const int row_units = a.n_kv_heads * head_units;
    const uint32_t parts = (uint32_t)tr_append_groups(row_units, half_dim);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // the wave's first group, whose token is wave-uniform, finds its run; a second group is in the same one or behind it
    const uint32_t grp0 = (blockIdx.x * APPEND_WAVES + wave) << (6 - shift), grp = grp0 + ((threadIdx.x & 63) >> shift);
    const int tok0 = (int)(parts == 1 ? grp0 : grp0 / parts);
    if (tok0 >= a.total_tokens) return;
    int r = last_not_above(a.n_desc, tok0, [&](int i) { return a.tok0[i]; }), tok = tok0;
    if (shift == 5) {
        tok = (int)(parts == 1 ? grp : grp / parts);
        if (tok >= a.total_tokens) return;
        if (r + 1 < a.n_desc && a.tok0[r + 1] <= tok) ++r; // tok is tok0 or the token behind it, and every run has one
    }
    const TrAppendDesc d = a.desc[r];
    const int i = tok - a.tok0[r];
    // position id: the caller's, or (raw-store assembly) the run's first position plus the row's index in the run
    const int pos = a.q_pos ? a.q_pos[d.q_row0 + i] : d.pos0 + i;
    const int lane = threadIdx.x & (half_dim - 1);
    append_token<DTYPE, HALF>(a.k_new, a.v_new, pos, a.cache_k, a.cache_v, row_units, head_units, half_dim, a.theta,
                              (int64_t)d.q_row0 + i, (int64_t)d.dst_row0 + i, (int)(grp - tok * parts), cs + (threadIdx.x - lane), lane);
}

// The same rows for launches of many short ones (a store of un-rotated keys, or the key rotation of the one-pass call, with
// one or two KV heads per device): the lanes of a head's units own a token, so a wave holds 64 / head_units tokens side by
// side, and a token's lanes walk its heads.  A group of half_dim lanes leaves at least half of them idle there through the
// whole load, rotate and store, and there are enough tokens to fill the chip without that.  Each lane computes the angles of
// its own pairs (in the half-split layout half of them, its partner lane the other half).  Same arithmetic, so the same bits.
constexpr int PACKED_HEADS = 2;
template <int DTYPE, bool HALF>
__global__ __launch_bounds__(64 * APPEND_WAVES) void append_packed_kernel(const TrAppendArgs a)
{
    constexpr int P = Unit<DTYPE>::PAIRS, N_CS = HALF ? 2 * P : P;
    static_assert(UnitHalf<DTYPE>::ELEMS == 2 * P, "partner lanes share the angles of their unit evenly");
    const int head_units = a.head_dim * (DTYPE == TR_BF16 ? 2 : 4) / 16; // a power of two, at most 32
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int per_wave = 64 / head_units, unit = lane % head_units;
    const int tok0 = ((int)blockIdx.x * APPEND_WAVES + wave) * per_wave, tok = tok0 + lane / head_units;
    int r = last_not_above(a.n_desc, tok0, [&](int i) { return a.tok0[i]; });
    if (tok >= a.total_tokens) return; // whole tokens leave together, so a partner lane stays
    while (r + 1 < a.n_desc && a.tok0[r + 1] <= tok) ++r;
    const TrAppendDesc d = a.desc[r];
    const int i = tok - a.tok0[r];
    const int pos = a.q_pos ? a.q_pos[d.q_row0 + i] : d.pos0 + i;
    const int64_t row_units = (int64_t)a.n_kv_heads * head_units;
    const uint4* ks = (const uint4*)a.k_new + ((int64_t)d.q_row0 + i) * row_units + unit;
    const uint4* vs = (const uint4*)a.v_new + ((int64_t)d.q_row0 + i) * row_units + unit;
    uint4* kd = (uint4*)a.cache_k + ((int64_t)d.dst_row0 + i) * row_units + unit;
    uint4* vd = (uint4*)a.cache_v + ((int64_t)d.dst_row0 + i) * row_units + unit;
    const int hmask = head_units >> 1;
    const bool low = unit < hmask;
    const int m0 = HALF ? (low ? unit : unit - hmask) * N_CS : unit * N_CS;
    double c[N_CS], s[N_CS];
    uint4 kx[PACKED_HEADS], vx[PACKED_HEADS];
#pragma unroll
    for (int j = 0; j < PACKED_HEADS; ++j)
        if (j < a.n_kv_heads) {
            kx[j] = ld_stream_any(ks + j * head_units);
            if (a.v_new) vx[j] = ld_stream_any(vs + j * head_units);
        }
    // the loads are on their way while the angles are computed
#pragma unroll
    for (int p = 0; p < P; ++p) {
        double sn, cn;
        tr_sincos((double)pos * a.theta[m0 + (HALF && !low ? P : 0) + p], &sn, &cn);
        if constexpr (HALF) {
            const double co = __shfl_xor(cn, hmask), so = __shfl_xor(sn, hmask);
            c[p] = low ? cn : co;
            s[p] = low ? sn : so;
            c[P + p] = low ? co : cn;
            s[P + p] = low ? so : sn;
        } else {
            c[p] = cn;
            s[p] = sn;
        }
    }
#pragma unroll
    for (int j = 0; j < PACKED_HEADS; ++j)
        if (j < a.n_kv_heads) {
            uint4 y;
            if constexpr (HALF) y = UnitHalf<DTYPE>::rotate(kx[j], shfl_xor_u4(kx[j], hmask), low, c, s);
            else y = Unit<DTYPE>::rotate(kx[j], c, s);
            st_any(kd + j * head_units, y);
            if (a.v_new) st_any(vd + j * head_units, vx[j]); // v_new == NULL: keys only
        }
}

// ---- offline key rotation (Sec. 3.4 step 2): K' = R(t - cu[c]) k -------------------------------------------
// table[pos][m] = (cos, sin)(pos * theta_m) in fp64, positions 0 .. n_pos-1
struct ThetaArg { double v[64]; };
__global__ __launch_bounds__(256) void rope_table_kernel(double2* table, int n_pos, int half_dim, const ThetaArg theta_arg)
{
    const double* theta = theta_arg.v;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= (int64_t)n_pos * half_dim) return;
    const int pos = (int)(gid / half_dim), m = (int)(gid % half_dim);
    double sn, cn;
    tr_sincos((double)pos * theta[m], &sn, &cn);
    table[gid] = make_double2(cn, sn);
}

// Grid (row blocks, chunks); a thread owns one 16-byte unit position inside a head for one token and walks the
// KV heads, so the (cos, sin) of its pairs serve every head.  Row blocks stride over the chunk, so
// every token of [cu[c], cu[c+1]) is covered whatever the chunk's length.  Also records, per token, the first
// row of its chunk.
// TABLE: the angles come from rope_table_kernel's table, which serves every chunk.  Otherwise each thread works out the
// angles of one unit's pairs, the first heads' loads being on their way (in the half-split layout partner lanes have half each):
// no launch in front and no table to wait for, but tokens x half_dim fp64 sincos in all, which a long call does not hide.
constexpr int ROPE_ROWS_HEADS = 8; // KV heads in flight per thread

template <int DTYPE, bool HALF, bool TABLE>
__global__ __launch_bounds__(256) void rope_rows_kernel(const uint4* k, uint4* k_rot, const int32_t* cu, int32_t* tok_start,
                                                        const double2* table, int table_rows, const ThetaArg theta, int64_t total_tokens,
                                                        int n_kv_heads, int head_units, int half_dim)
{
    constexpr int P = Unit<DTYPE>::PAIRS, N_CS = HALF ? UnitHalf<DTYPE>::ELEMS : P; // N_CS: pairs this thread's unit takes part in
    static_assert(UnitHalf<DTYPE>::ELEMS == 2 * P, "partner lanes share the angles of a unit evenly");
    const int hmask = head_units >> 1;
    const int chunk = blockIdx.y;
    int start = cu[chunk], end = cu[chunk + 1];
    if (start < 0) start = 0;
    if (end > total_tokens) end = (int)total_tokens;
    const int tpb = 256 / head_units; // tokens per block
    const int unit = threadIdx.x % head_units;
    const int row_units = n_kv_heads * head_units;
    const bool low = unit < hmask;
    const int m0 = (HALF && !low ? unit - hmask : unit) * N_CS;
    for (int t = start + blockIdx.x * tpb + threadIdx.x / head_units; t < end; t += gridDim.x * tpb) {
        if (unit == 0) tok_start[t] = start;
        int pos = t - start;
        if (pos > table_rows - 1) pos = table_rows - 1; // caller promised max_chunk_len; never read past the table
        const uint4* src = k + (int64_t)t * row_units + unit;
        uint4* dst = k_rot + (int64_t)t * row_units + unit;
        double c[N_CS], s[N_CS];
        for (int h0 = 0; h0 < n_kv_heads; h0 += ROPE_ROWS_HEADS) {
            uint4 x[ROPE_ROWS_HEADS];
#pragma unroll
            for (int j = 0; j < ROPE_ROWS_HEADS; ++j)
                if (h0 + j < n_kv_heads) x[j] = ld_stream(src + (h0 + j) * head_units);
            // a token's units sit in neighbouring lanes (head_units of them, a power of two), so the partner lane of the
            // half-split layout is in this iteration too
            if constexpr (TABLE) {
#pragma unroll
                for (int p = 0; p < N_CS; ++p) {
                    const double2 e = table[(int64_t)pos * half_dim + m0 + p];
                    c[p] = e.x;
                    s[p] = e.y;
                }
            } else if (h0 == 0) {
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    double sn, cn;
                    tr_sincos((double)pos * theta.v[m0 + (HALF && !low ? P : 0) + p], &sn, &cn);
                    if constexpr (HALF) {
                        const double co = __shfl_xor(cn, hmask), so = __shfl_xor(sn, hmask);
                        c[p] = low ? cn : co;
                        s[p] = low ? sn : so;
                        c[P + p] = low ? co : cn;
                        s[P + p] = low ? so : sn;
                    } else {
                        c[p] = cn;
                        s[p] = sn;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < ROPE_ROWS_HEADS; ++j)
                if (h0 + j < n_kv_heads) {
                    uint4 y = x[j];
                    if constexpr (HALF) y = UnitHalf<DTYPE>::rotate(x[j], shfl_xor_u4(x[j], hmask), low, c, s);
                    else if (pos != 0) y = Unit<DTYPE>::rotate(x[j], c, s);
                    dst[(h0 + j) * head_units] = y;
                }
        }
    }
}

} // namespace

int tr_launch_assemble(const TrAssembleArgs& a, int dtype, int n_blocks, hipStream_t s)
{
    if (n_blocks <= 0) return TR_OK;
    auto pick = [&](auto policy) {
        constexpr int P = decltype(policy)::value;
        return dtype == TR_BF16 ? (a.rope_half ? assemble_kernel<TR_BF16, true, P> : assemble_kernel<TR_BF16, false, P>)
                                : (a.rope_half ? assemble_kernel<TR_F32, true, P> : assemble_kernel<TR_F32, false, P>);
    };
    auto kern = a.formed_bytes >= THROUGH_MIN_BYTES ? pick(std::integral_constant<int, ST_THROUGH>())
                                                    : pick(std::integral_constant<int, ST_CACHED>());
    hipLaunchKernelGGL(kern, dim3(n_blocks), dim3(256), 0, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

// Tokens share the lanes of a group where a row leaves at least half of them idle and there are enough tokens to fill the
// chip all the same.  us, a group to a token / several, fresh rows, interleaved layout, bf16: one head of 64 (a quarter of
// the lanes) 4.5 / 4.7 at 6000 tokens, 5.1 / 5.0 at 8192, 11.2 / 8.1 at 30000; one head of 128 4.5 / 4.7 at 3000, 5.2 / 4.9 at
// 4096; two heads of 64 (half of them) 7.0 / 7.1 at 12000, 8.2 / 7.9 at 16384; two heads of 128 6.9 / 7.2 at 6000, 8.0 / 7.9 at
// 8192, 62 / 48 at 100000; three heads of 64 14.8 / 14.6 at 30000, 36.6 / 36.9 at 100000; four heads of 128 26.4 / 29.9 at
// 30000.  fp32 has half the angles per unit: one head of 64 (half of the lanes) 4.6 / 4.6 at 8192, 5.9 / 5.3 at 12000.
static bool append_packed(int tokens, int n_kv_heads, int head_units, int half_dim, int dtype)
{
    const int row_units = n_kv_heads * head_units;
    if (n_kv_heads > PACKED_HEADS || head_units > 16 || row_units * 2 > half_dim) return false;
    const int waves = row_units * 4 <= half_dim || dtype == TR_F32 ? 4096 : 8192; // of a group to a token
    return tokens >= waves * (64 / half_dim);
}

int tr_launch_append(const TrAppendArgs& a, int dtype, hipStream_t s)
{
    if (a.total_tokens <= 0) return TR_OK;
    const int head_units = a.head_dim * (dtype == TR_BF16 ? 2 : 4) / 16;
    const int row_units = a.n_kv_heads * head_units;
    const bool packed = append_packed(a.total_tokens, a.n_kv_heads, head_units, a.head_dim / 2, dtype);
    const int64_t blocks = packed ? ((int64_t)a.total_tokens * head_units + 64 * APPEND_WAVES - 1) / (64 * APPEND_WAVES) : tr_append_blocks(a.total_tokens, row_units, a.head_dim / 2);
    auto kern = dtype == TR_BF16 ? (a.rope_half ? append_kernel<TR_BF16, true> : append_kernel<TR_BF16, false>)
                                 : (a.rope_half ? append_kernel<TR_F32, true> : append_kernel<TR_F32, false>);
    if (packed)
        kern = dtype == TR_BF16 ? (a.rope_half ? append_packed_kernel<TR_BF16, true> : append_packed_kernel<TR_BF16, false>)
                                : (a.rope_half ? append_packed_kernel<TR_F32, true> : append_packed_kernel<TR_F32, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * APPEND_WAVES), 0, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

int tr_launch_rope_table(double* table, int n_pos, int half_dim, const double* theta, hipStream_t s)
{
    int64_t threads = (int64_t)n_pos * half_dim;
    if (threads <= 0) return TR_OK;
    ThetaArg th;
    for (int m = 0; m < 64; ++m) th.v[m] = theta[m];
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                       (double2*)table, n_pos, half_dim, th);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

int tr_launch_rope_rows(const void* k, void* k_rot, const int32_t* cu, int n_chunks, int max_chunk_len, int32_t* tok_start,
                        const double* table, int table_rows, int64_t total_tokens, const tr_shape* shape, hipStream_t s)
{
    const int eb = tr_elem_bytes(shape);
    const int head_units = shape->head_dim * eb / 16;
    if (total_tokens <= 0 || n_chunks <= 0) return TR_OK;
    ThetaArg th = {};
    tr_fill_theta(shape, th.v);
    const int tpb = 256 / head_units;
    int row_blocks = (max_chunk_len + tpb - 1) / tpb;
    if (row_blocks < 1) row_blocks = 1;
    if (row_blocks > 1024) row_blocks = 1024;
    // grid.y carries the chunk index: at most 65535 chunks per launch
    for (int c0 = 0; c0 < n_chunks; c0 += 65535) {
        const int nc = n_chunks - c0 < 65535 ? n_chunks - c0 : 65535;
        dim3 grid((unsigned)row_blocks, (unsigned)nc);
        const bool half = tr_rope_half(shape) != 0;
        auto kern = shape->dtype == TR_BF16 ? (half ? rope_rows_kernel<TR_BF16, true, true> : rope_rows_kernel<TR_BF16, false, true>)
                                            : (half ? rope_rows_kernel<TR_F32, true, true> : rope_rows_kernel<TR_F32, false, true>);
        if (!table)
            kern = shape->dtype == TR_BF16 ? (half ? rope_rows_kernel<TR_BF16, true, false> : rope_rows_kernel<TR_BF16, false, false>)
                                           : (half ? rope_rows_kernel<TR_F32, true, false> : rope_rows_kernel<TR_F32, false, false>);
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, (const uint4*)k, (uint4*)k_rot, cu + c0, tok_start, (const double2*)table,
                           table_rows, th, total_tokens, shape->n_kv_heads, head_units, shape->head_dim / 2);
        TR_HIP(hipGetLastError());
    }
    return TR_OK;
}
