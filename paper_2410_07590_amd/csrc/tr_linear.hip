// Projections around the attention (Eq. 1: Q, K, V = X W; the output projection is the same product) for the
// query tokens of a request: y[m, n] = sum_k x[m, k] w[n, k] with at most 128 rows of x.  With so few rows the
// product is bound by streaming the weights once from HBM, so the kernel is organised around that stream.
//   * A workgroup owns 128 output features (four waves x 32 rows of w, each row contiguous along k) and a slice of k.
//   * k is walked in chunks of 128 values.  Every wave fetches its 32 x 256-byte piece of w with direct global -> LDS
//     loads that read whole 256-byte runs (16-byte pieces XOR-swizzled by the row on the source side) and reads it
//     back in the matrix instruction's operand layout; reading w straight in operand layout would touch 32 rows x
//     32 bytes per instruction, which the memory system serves at a fraction of its rate.
//   * The chunk of x (all rows x 256 bytes) is fetched once per workgroup the same way and shared by the four waves:
//     x is re-read once per 128 features, not once per 32.
//   * v_mfma_f32_32x32x16_bf16 with w rows as the A operand and x rows as the B operand makes the arithmetic free,
//     provided its operand reads are batched ahead of it: read-wait-multiply per step left the products of a chunk
//     as one chain of LDS latencies, which showed as soon as x had more than 32 rows.
//   * Up to three chunks per workgroup are in flight in a ring of LDS slots while the current one is multiplied.
// Slices of k that live in different workgroups write fp32 partial sums that a second small kernel adds in a fixed
// order: no atomics, same inputs, same bits.
// An attention projection is over before such a stream is long enough to pay for that second launch, so weights up to a size
// go through linear_direct_kernel, whose workgroups keep all of k (see there and direct_plan).
#include "tr_internal.h"

#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <cmath>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Up to TR_LINEAR_MAX_OUT weights share x in one launch (query, key and value): output j owns the 32-feature tiles
// [tile0[j], tile0[j+1]) and the columns [32 tile0[j], 32 tile0[j+1]) of the partial sums.
struct TrLinearArgs {
    const __bf16* x;                    // [M, K]
    const __bf16* w[TR_LINEAR_MAX_OUT]; // [N_j, K]
    __bf16* y[TR_LINEAR_MAX_OUT];       // [M, N_j]
    float* partial;                     // [n_split, M, N] when n_split > 1, N = sum of the N_j
    int32_t tile0[TR_LINEAR_MAX_OUT + 1];
    int32_t n_out;
    int32_t M, N, K;
    int32_t n_split;
    int32_t m_split;                    // 1, or 2: rows [0, 64) and [64, M) of x go to two workgroups of the same XCD
    int32_t row_tiles;                  // of 16 XB rows (linear_direct_kernel)
    int32_t row_magic;                  // 65536 / row_tiles + 1: x / row_tiles = x row_magic >> 16 for x < 256
};

constexpr int LIN_CK = 128;           // values of k per chunk: 256 bytes of every row
constexpr int LIN_PPR = LIN_CK / 8;   // 16-byte pieces per row of a chunk: 16
constexpr int LIN_ROW = LIN_CK * 2;   // bytes per parked row
constexpr int LIN_MAX_SPLIT = 16;     // k-slices across workgroups, at most

#define LDS_AS __attribute__((address_space(3)))
#define GLB_AS __attribute__((address_space(1)))

__device__ __forceinline__ int lin_piece_off(int row, int piece) { return row * LIN_ROW + ((piece ^ (row & (LIN_PPR - 1))) * 16); }

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
constexpr int lin_vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
template <int N> __device__ __forceinline__ void lin_wait_vm() { __builtin_amdgcn_s_waitcnt(lin_vmcnt_imm(N)); }

template <int MT> constexpr int lin_slot_bytes() { return (4 + MT) * 32 * LIN_ROW; }    // four waves' w pieces, then x
// Chunks in flight per workgroup.  A small weight (the attention projections) is over within a few round trips, so
// one workgroup per CU requests its whole slice at once (DEEP: three chunks, two from 96 rows of x on, <= 144 KB of
// LDS).  A large weight (an MLP's) streams better with one chunk per workgroup and three workgroups per CU.
template <int MT, bool DEEP> constexpr int lin_slots() { return !DEEP ? 1 : (MT <= 2 ? 3 : 2); }
constexpr int64_t LIN_LARGE_WEIGHT_BYTES = 64ll << 20;

// MT: 32-row blocks of x (ceil(M / 32), 1..4)
template <int MT, bool DEEP>
__global__ __launch_bounds__(256) void linear_kernel(const TrLinearArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    LDS_AS char* lds = (LDS_AS char*)lds_raw;
    constexpr int NSLOT = lin_slots<MT, DEEP>(), SLOT = lin_slot_bytes<MT>();
    constexpr int IPC = 8 + 2 * MT; // load instructions per wave and chunk: its 8 KB of w, its quarter of x
    // all arguments in one batch of scalar loads, and selects between them: see linear_direct_kernel
    static_assert(TR_LINEAR_MAX_OUT == 4, "");
    const __bf16 *x = a.x, *w0 = a.w[0], *w1 = a.w[1], *w2 = a.w[2], *w3 = a.w[3];
    auto y0 = (GLB_AS __bf16*)a.y[0], y1 = (GLB_AS __bf16*)a.y[1], y2 = (GLB_AS __bf16*)a.y[2], y3 = (GLB_AS __bf16*)a.y[3]; // else flat stores
    auto partial = (GLB_AS float*)a.partial;
    int rows = a.M, N = a.N, K = a.K, n_split = a.n_split, m_split = a.m_split, t1 = a.tile0[1], t2 = a.tile0[2], t3 = a.tile0[3];
    asm volatile("" : "+s"(x), "+s"(w0), "+s"(w1), "+s"(w2), "+s"(w3), "+s"(rows), "+s"(N), "+s"(K), "+s"(n_split), "+s"(m_split), "+s"(t1),
                 "+s"(t2), "+s"(t3));
    asm volatile("" : "+s"(y0), "+s"(y1), "+s"(y2), "+s"(y3), "+s"(partial));
    // what belongs to the output of a tile; tile0 of outputs that are not there is the end
    auto of_output = [&](int tile, auto v0, auto v1, auto v2, auto v3) { return tile >= t3 ? v3 : tile >= t2 ? v2 : tile >= t1 ? v1 : v0; };
    const int groups = (N / 32 + 3) / 4;                        // workgroups along the features
    // With two row halves, blocks b and b + 8 (same XCD, dispatched together) take the two halves of one
    // (features, k-slice) item, so that the second read of its weights is served by that XCD's L2.
    int item = blockIdx.x, m0 = 0;
    if (m_split == 2) {
        item = ((blockIdx.x >> 4) << 3) | (blockIdx.x & 7);
        m0 = ((blockIdx.x >> 3) & 1) * (32 * MT);
        if (item >= groups * n_split) return;                   // padding of the grid to a multiple of 16 (whole workgroup)
    }
    const int M = min(rows - m0, 32 * MT);                      // rows of x this workgroup multiplies
    const __bf16* xrows = x + (int64_t)m0 * K;
    const int split = (int)((uint32_t)item / (uint32_t)groups), group = item - split * groups;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int tile = min(4 * group + wave, N / 32 - 1);         // a wave past the last tile redoes it and stores nothing
    const bool tile_mine = 4 * group + wave < N / 32;
    const int first_tile = of_output(tile, 0, t1, t2, t3), ltile = tile - first_tile; // inside the output this tile belongs to
    // chunks of this workgroup: a contiguous range; the last chunk of a row may be short
    const uint32_t total_chunks = (uint32_t)(K + LIN_CK - 1) / LIN_CK; // times LIN_MAX_SPLIT fits 32 bits
    const int c0 = (int)(total_chunks * (uint32_t)split / (uint32_t)n_split), c1 = (int)(total_chunks * (uint32_t)(split + 1) / (uint32_t)n_split);
    const int n_chunks = c1 - c0;

    // Direct global -> LDS loads: instruction i of a wave fills 1 KB, lane l the 16-byte piece 64 i + l of the
    // destination, i.e. row (64 i + l) / 16, parked piece (64 i + l) % 16; it therefore fetches the logical piece
    // parked there (the XOR swizzle is applied on the source side).  Four rows x 256 contiguous bytes per instruction.
    const int lrow = lane / LIN_PPR, ppiece = lane % LIN_PPR;
    const int last_piece = K / 8 - 1; // pieces past the end of a row are read from its last piece and never used
    const __bf16* wbase = of_output(tile, w0, w1, w2, w3) + (int64_t)(ltile * 32) * K;
    auto issue_chunk = [&](int c, LDS_AS char* slot) {
        LDS_AS char* wdst = slot + wave * (32 * LIN_ROW);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = 4 * i + lrow;
            const int piece = min(c * LIN_PPR + (ppiece ^ (row & (LIN_PPR - 1))), last_piece);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(wbase + (int64_t)row * K + 8 * piece),
                                             (LDS_AS void*)(wdst + i * 1024), 16, 0, 0);
        }
        LDS_AS char* xdst = slot + 4 * 32 * LIN_ROW;
#pragma unroll
        for (int i = 0; i < 2 * MT; ++i) {
            const int row = 4 * (wave * 2 * MT + i) + lrow; // this wave's quarter of the 32 MT rows
            const int piece = min(c * LIN_PPR + (ppiece ^ (row & (LIN_PPR - 1))), last_piece);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xrows + (int64_t)min(row, M - 1) * K + 8 * piece),
                                             (LDS_AS void*)(xdst + (wave * 2 * MT + i) * 1024), 16, 0, 0);
        }
    };

    f32x16 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[mt][e] = 0.0f;

#pragma unroll
    for (int p = 0; p < NSLOT; ++p)
        if (p < n_chunks) issue_chunk(c0 + p, lds + p * SLOT);
    for (int t = 0; t < n_chunks; ++t) {
        // chunk t has landed once only the loads of the chunks issued after it are outstanding
        const int later = min(NSLOT - 1, n_chunks - 1 - t);
        if (later >= 2) lin_wait_vm<2 * IPC>();
        else if (later == 1) lin_wait_vm<IPC>();
        else lin_wait_vm<0>();
        __builtin_amdgcn_s_barrier(); // every wave's part of chunk t (its share of x included) is in LDS
        LDS_AS const char* slot = lds + (t % NSLOT) * SLOT;
        LDS_AS const char* wb = slot + wave * (32 * LIN_ROW);
        LDS_AS const char* xb0 = slot + 4 * 32 * LIN_ROW;
        const int steps = min(LIN_CK, K - (c0 + t) * LIN_CK) / 16;
        auto step = [&](int s) {
            const bf16x8 wa = *(LDS_AS const bf16x8*)(wb + lin_piece_off(r, 2 * s + h));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const bf16x8 xb = *(LDS_AS const bf16x8*)(xb0 + lin_piece_off(32 * mt + r, 2 * s + h));
                acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, xb, acc[mt], 0, 0, 0);
            }
        };
        if (steps == LIN_CK / 16) { // a whole chunk: the operands of SB steps are read before their products start
            constexpr int SB = 2; // deeper batches measured the same and cost registers
#pragma unroll
            for (int s0 = 0; s0 < LIN_CK / 16; s0 += SB) {
                bf16x8 wa[SB], xb[MT][SB];
#pragma unroll
                for (int s = 0; s < SB; ++s) {
                    wa[s] = *(LDS_AS const bf16x8*)(wb + lin_piece_off(r, 2 * (s0 + s) + h));
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) xb[mt][s] = *(LDS_AS const bf16x8*)(xb0 + lin_piece_off(32 * mt + r, 2 * (s0 + s) + h));
                }
                __builtin_amdgcn_sched_barrier(0); // keep the reads above: the scheduler would sink each to its use
#pragma unroll
                for (int s = 0; s < SB; ++s)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[s], xb[mt][s], acc[mt], 0, 0, 0);
            }
        } else {                    // the short last chunk of a row (workgroup-uniform)
#pragma unroll
            for (int s = 0; s < LIN_CK / 16; ++s)
                if (s < steps) step(s);
        }
        if (t + NSLOT < n_chunks) {
            __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): this wave's operand reads of the slot are done
            __builtin_amdgcn_s_barrier();        // ... and everyone else's: the slot can be refilled
            issue_chunk(c0 + t + NSLOT, lds + (t % NSLOT) * SLOT);
        }
    }
    if (!tile_mine) return;
    auto y = of_output(tile, y0, y1, y2, y3);
    const int Nj = 32 * (of_output(tile, t1, t2, t3, N / 32) - first_tile);

    // element e of acc[mt] is y_j[32 mt + r][32 ltile + 8 (e >> 2) + 4 h + (e & 3)]
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (32 * mt + r >= M) continue;
        const int m = m0 + 32 * mt + r;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int n = 32 * tile + 8 * q4 + 4 * h; // column among all outputs
            if (n_split == 1) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)acc[mt][4 * q4 + e];
                *(GLB_AS bf16x4*)(y + (int64_t)m * Nj + (n - 32 * first_tile)) = o;
            } else {
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = acc[mt][4 * q4 + e];
                *(GLB_AS f32x4*)(partial + ((int64_t)split * rows + m) * N + n) = o;
            }
        }
    }
}

// y = bf16(sum over the k-slices, in slice order); four outputs per thread
__global__ __launch_bounds__(256) void linear_combine_kernel(const TrLinearArgs a)
{
    const int64_t total4 = (int64_t)a.M * a.N / 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total4) return;
    const int m = (int)(4 * i / a.N), n = (int)(4 * i % a.N);
    int j = 0;
    while (j + 1 < a.n_out && n >= 32 * a.tile0[j + 1]) ++j;
    // every slice's load is issued before the first sum needs one: the latencies overlap instead of adding up
    f32x4 t[LIN_MAX_SPLIT];
#pragma unroll
    for (int sp = 0; sp < LIN_MAX_SPLIT; ++sp)
        if (sp < a.n_split) t[sp] = *(const f32x4*)(a.partial + (int64_t)sp * a.M * a.N + 4 * i);
    f32x4 s = t[0];
#pragma unroll
    for (int sp = 1; sp < LIN_MAX_SPLIT; ++sp)
        if (sp < a.n_split) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += t[sp][e];
        }
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (__bf16)s[e];
    *(bf16x4*)(a.y[j] + (int64_t)m * (32 * (a.tile0[j + 1] - a.tile0[j])) + (n - 32 * a.tile0[j])) = o;
}

// All of k in one workgroup, so that no partial sums are left over: a tile of 16 XB rows of x and 16 WB features.  What bounds it
// is how fast a CU takes bytes in through the direct loads, from HBM or L2 alike: with nothing but the loads and the exchange left
// (profiles/load_rates.md) 4608 x 3584 and 3584 x 3584 at 64 rows take 13.5 and 11.2 us of their 14.2 and 11.9, 41 .. 43 GB/s
// per CU, some 50 without an empty launch.  A workgroup asks for (XB + WB) * 16 rows of K
// values, and the best tile is the one that keeps the largest share per CU small.  The row tiles of one feature tile run on the same
// XCD, whose L2 serves the weights to all but the first of them.
// k is walked in chunks of 128 values through a ring of LDS slots; of a chunk each of the four waves multiplies 32 values (one
// k-step of v_mfma_f32_16x16x32_bf16: w rows = A, x rows = B), and the four sums meet in LDS at the end, added in wave order.
// Ten layers' projections of 64 rows (3584 -> 3584 + 512 + 512, 3584 -> 3584) take 269 us instead of 307.
// The rounding error of a chain through the matrix unit's accumulator grows with the chain's length, that of several chains with the
// root of their number, and a slice of linear_kernel may be as short as two chunks: 256 values in a row.  So after DIRECT_FOLD chunks, of each of which 32 values
// are a wave's own (224 in a row), the accumulator is added to a second one and starts again.  Error of the sums alone (operands
// whose exact results are zero), this kernel / the slices: 3584 x 3584 at 64 rows 5.2e-6 / 7.2e-6, 512 x 3584 at 128 rows 5.2e-6 /
// 5.4e-6, 2048 x 2048 at 64 rows 3.7e-6 / 3.9e-6; in one chain 9.1e-6, 9.1e-6 and 5.2e-6.  The additions run while the operand
// reads do; up to seven chunks there are none.  Cost: ten layers of 64 rows 267 -> 269 us, 6144 x 3072 at 17 rows 11.5 -> 11.75.
constexpr int DIRECT_FOLD = 7;
constexpr int DIRECT_MAX_SLOTS = 8, DIRECT_LDS = 128 * 1024;
template <int XB, int WB> constexpr int direct_slot_bytes() { return 16 * (XB + WB) * LIN_ROW; }
template <int XB, int WB> constexpr int direct_slots()
{
    return DIRECT_LDS / direct_slot_bytes<XB, WB>() < DIRECT_MAX_SLOTS ? DIRECT_LDS / direct_slot_bytes<XB, WB>() : DIRECT_MAX_SLOTS;
}
template <int XB, int WB> constexpr int direct_lds_bytes() { return direct_slots<XB, WB>() * direct_slot_bytes<XB, WB>(); }

// Two workgroups per CU in the bounds, though LDS leaves room for one of most tiles: with more registers the compiler keeps the accumulators in
// the other half of the file and moves them there and back in every chunk (3584 x 3584 at 64 rows 12.1 -> 14.8 us).
template <int XB, int WB>
__global__ __launch_bounds__(256, 2) void linear_direct_kernel(const TrLinearArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    LDS_AS char* lds = (LDS_AS char*)lds_raw;
    constexpr int SLOT = direct_slot_bytes<XB, WB>(), NSLOT = direct_slots<XB, WB>();
    constexpr int IPC = XB + WB; // load instructions of a wave for a chunk, four rows x 256 bytes each
    static_assert(NSLOT >= 3 && (NSLOT - 2) * IPC < 63 && 4 * XB * WB * 1024 <= NSLOT * SLOT, "");
    // All arguments in one batch of scalar loads, and selects between them: indexed by the output, each load address waited for two
    // more scalar loads, and with the division seven round trips lay in front of the first request.  Ten layers of 64 rows:
    // 268 -> 261 us.
    const __bf16* x = a.x;
    const __bf16 *w0 = a.w[0], *w1 = a.w[1], *w2 = a.w[2], *w3 = a.w[3];
    auto y0 = (GLB_AS __bf16*)a.y[0], y1 = (GLB_AS __bf16*)a.y[1], y2 = (GLB_AS __bf16*)a.y[2], y3 = (GLB_AS __bf16*)a.y[3]; // else flat stores
    int M = a.M, N = a.N, K = a.K, row_tiles = a.row_tiles, row_magic = a.row_magic, t1 = a.tile0[1], t2 = a.tile0[2], t3 = a.tile0[3];
    asm volatile("" : "+s"(x), "+s"(w0), "+s"(w1), "+s"(w2), "+s"(w3), "+s"(M), "+s"(N), "+s"(K), "+s"(row_tiles), "+s"(row_magic), "+s"(t1),
                 "+s"(t2), "+s"(t3));
    asm volatile("" : "+s"(y0), "+s"(y1), "+s"(y2), "+s"(y3));
    const int place = blockIdx.x >> 3, group = (int)(((uint32_t)place * (uint32_t)row_magic) >> 16);
    const int item = group * 8 + (blockIdx.x & 7); // feature tile
    const int m0 = (place - group * row_tiles) * (16 * XB);
    const int blocks = N / 16;                     // of features
    if (item * WB >= blocks) return;                             // padding of the grid (whole workgroup)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    static_assert(TR_LINEAR_MAX_OUT == 4, "");
    // what belongs to the output of a block of features; tile0 of outputs that are not there is the end
    auto of_output = [&](int block, auto v0, auto v1, auto v2, auto v3) { return block >= 2 * t3 ? v3 : block >= 2 * t2 ? v2 : block >= 2 * t1 ? v1 : v0; };

    // Load i of this wave fills rows 4 g .. 4 g + 3 of a slot (x rows, then w rows), 16-byte pieces XOR-swizzled by the row on
    // the source side.  Rows of x past the last one and features past the last one read the last one's and are not stored.
    const int lrow = lane / LIN_PPR, ppiece = lane % LIN_PPR, last_piece = K / 8 - 1;
    const __bf16* src[IPC];
    int piece0[IPC];
#pragma unroll
    for (int i = 0; i < IPC; ++i) {
        const int g = wave * IPC + i, row = 4 * g + lrow;
        piece0[i] = ppiece ^ (row & (LIN_PPR - 1));
        if (g < 4 * XB) {
            src[i] = x + (int64_t)min(m0 + row, M - 1) * K;
        } else {
            const int block = min(item * WB + (g - 4 * XB) / 4, blocks - 1);
            src[i] = of_output(block, w0, w1, w2, w3) + (int64_t)(16 * (block - 2 * of_output(block, 0, t1, t2, t3)) + (row & 15)) * K;
        }
    }
    auto issue = [&](int c, int slot) {
        LDS_AS char* dst = lds + slot * SLOT + wave * (IPC * 1024);
#pragma unroll
        for (int i = 0; i < IPC; ++i) {
            const int piece = min(c * LIN_PPR + piece0[i], last_piece); // pieces past the end of a row are not used
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[i] + 8 * piece), (LDS_AS void*)(dst + i * 1024), 16, 0, 0);
        }
    };

    // acc: products of at most DIRECT_FOLD chunks, sum: of all before them
    f32x4 acc[WB][XB], sum[WB][XB];
#pragma unroll
    for (int wb = 0; wb < WB; ++wb)
#pragma unroll
        for (int xb = 0; xb < XB; ++xb) acc[wb][xb] = sum[wb][xb] = f32x4{};

    // rows that lie a multiple of 8 KB apart, or all but so, would all be asked for on the same few memory channels at the same time:
    // there every feature tile starts its walk somewhere else (4096 x 4096, 37 rows of x 15.1 -> 11.4 us; 8192 x 8192, 32 rows 35.6 ->
    // 26.5; 44 sizes within 64 bytes of 8 KB 1.09 times as fast, 63 of 16 KB 1.15; elsewhere it costs up to a tenth)
    const bool staggered = K > 32 && (K + 32) % 4096 <= 64;
    const int n_chunks = (K + LIN_CK - 1) / LIN_CK, first = staggered ? (int)((uint32_t)item * 5u % (uint32_t)n_chunks) : 0;
    auto chunk = [&](int c) { return c + first < n_chunks ? c + first : c + first - n_chunks; };
#pragma unroll
    for (int p = 0; p < NSLOT - 1; ++p)
        if (p < n_chunks) issue(chunk(p), p);
    const int r = lane & 15, piece = 4 * wave + (lane >> 4); // this lane's operand row of a block and its piece of a chunk
    const int off = lin_piece_off(r, piece);
    int slot = 0, chain = 0; // chain: chunks in acc
    for (int c = 0; c < n_chunks; ++c) {
        // chunk c has landed once at most the loads of the chunks requested after it are outstanding
        if (c + NSLOT - 1 <= n_chunks) lin_wait_vm<(NSLOT - 2) * IPC>();
        else lin_wait_vm<0>();
        __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): this wave's operand reads of chunk c - 1 are done
        __builtin_amdgcn_s_barrier();       // ... and everyone else's, so its slot is free; every wave's part of chunk c has landed
        if (c + NSLOT - 1 < n_chunks) issue(chunk(c + NSLOT - 1), slot == 0 ? NSLOT - 1 : slot - 1);
        LDS_AS const char* base = lds + slot * SLOT + off;
        bf16x8 xb_[XB], wb_[WB];
#pragma unroll
        for (int b = 0; b < XB; ++b) xb_[b] = *(LDS_AS const bf16x8*)(base + b * (16 * LIN_ROW));
#pragma unroll
        for (int b = 0; b < WB; ++b) wb_[b] = *(LDS_AS const bf16x8*)(base + (XB + b) * (16 * LIN_ROW));
        if (chain == DIRECT_FOLD) { // in the shadow of the operand reads
            asm volatile("");       // a branch, not selects in every iteration
#pragma unroll
            for (int w = 0; w < WB; ++w)
#pragma unroll
                for (int b = 0; b < XB; ++b) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[w][b][e] += acc[w][b][e];
                    acc[w][b] = f32x4{};
                }
            chain = 0;
        }
        ++chain;
        if (chunk(c) * LIN_PPR + piece > last_piece) { // past the end of a row, in its short last chunk
#pragma unroll
            for (int b = 0; b < XB; ++b) xb_[b] = bf16x8{};
#pragma unroll
            for (int b = 0; b < WB; ++b) wb_[b] = bf16x8{};
        }
#pragma unroll
        for (int w = 0; w < WB; ++w)
#pragma unroll
            for (int b = 0; b < XB; ++b) acc[w][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb_[w], xb_[b], acc[w][b], 0, 0, 0);
        slot = slot + 1 == NSLOT ? 0 : slot + 1;
    }
    if (n_chunks > DIRECT_FOLD) {
#pragma unroll
        for (int w = 0; w < WB; ++w)
#pragma unroll
            for (int b = 0; b < XB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[w][b][e] += sum[w][b][e];
    }

    // element e of lane l's acc[w][b]: row m0 + 16 b + (l & 15) of x, feature 4 (l >> 4) + e of block w
    __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0): this wave's operand reads are done
    __builtin_amdgcn_s_barrier();       // ... and everyone else's: the ring becomes the exchange
#pragma unroll
    for (int w = 0; w < WB; ++w)
#pragma unroll
        for (int b = 0; b < XB; ++b) *(LDS_AS f32x4*)(lds + ((wave * WB + w) * XB + b) * 1024 + lane * 16) = acc[w][b];
    __syncthreads();
#pragma unroll
    for (int t0 = 0; t0 < WB * XB; t0 += 4) {
        const int t = t0 + wave;
        if (t >= WB * XB) break;
        f32x4 s = *(LDS_AS const f32x4*)(lds + t * 1024 + lane * 16);
#pragma unroll
        for (int v = 1; v < 4; ++v) {
            const f32x4 q = *(LDS_AS const f32x4*)(lds + (v * WB * XB + t) * 1024 + lane * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += q[e];
        }
        const int block = item * WB + t / XB, m = m0 + 16 * (t % XB) + r;
        if (block >= blocks || m >= M) continue;
        const int first_tile = of_output(block, 0, t1, t2, t3);
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)s[e];
        *(GLB_AS bf16x4*)(of_output(block, y0, y1, y2, y3) + (int64_t)m * (32 * (of_output(block, t1, t2, t3, N / 32) - first_tile)) +
                   16 * (block - 2 * first_tile) + 4 * (lane >> 4)) = o;
    }
}

} // namespace

// k-slices across workgroups.  Small weights: one workgroup per CU, about 200 of them measured best (more slices
// cost more partial traffic and shorter streams than the last CUs gain).  Large weights: about 450 workgroups, up
// to three per CU.  At least two 128-value chunks of k in each.

static bool lin_large(int32_t N, int32_t K) { return (int64_t)N * K * 2 >= LIN_LARGE_WEIGHT_BYTES; }
// More than 96 rows of x against a small weight: two workgroups per item, one per 64 rows, each with the ring of
// three chunks that 64 rows leave room for (128 rows x 4608 x 3584: 20.7 -> 18.9 us; at 65..96 rows and for large
// weights one workgroup per item measured faster).  tr_set_tuning("lin_msplit", 1) keeps one.
static int lin_m_split(int32_t M, int32_t N, int32_t K)
{
    if (tr_knob(TR_KNOB_LIN_MSPLIT, 0) == 1) return 1;
    return (M > 96 && !lin_large(N, K)) ? 2 : 1;
}

int tr_linear_splits(int32_t M, int32_t N, int32_t K)
{
    const int groups = (N / 32 + 3) / 4 * lin_m_split(M, N, K), chunks = (K + LIN_CK - 1) / LIN_CK;
    int n_split = ((lin_large(N, K) ? 450 : 200) + groups / 2) / groups;
    if (n_split > chunks / 2) n_split = chunks / 2;
    if (n_split > LIN_MAX_SPLIT) n_split = LIN_MAX_SPLIT;
    if (const int forced = tr_knob(TR_KNOB_LIN_SPLIT, 0); forced >= 1 && forced <= chunks && forced <= LIN_MAX_SPLIT) n_split = forced;
    if (n_split < 1) n_split = 1;
    return n_split;
}

template <int XB, int WB> static int launch_direct(const TrLinearArgs& a, hipStream_t s)
{
    auto kern = linear_direct_kernel<XB, WB>;
    constexpr int lds = direct_lds_bytes<XB, WB>();
    static std::atomic<uint64_t> configured{0};
    if (int rc = tr_raise_lds_limit((const void*)kern, lds, &configured)) return rc;
    const int tiles = (a.N / 16 + WB - 1) / WB;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * a.row_tiles * ((tiles + 7) / 8))), dim3(256), lds, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}
// The tiles there are, in blocks of 16 rows of x and 16 features.  Tiles of two or more row blocks by one feature block and (4, 2) would
// never be taken: where one fits, so does one with fewer bytes or a squarer one of as many.
struct DirectTile {
    int xb, wb;
    int per_cu; // workgroups that the LDS of a CU holds
    int (*launch)(const TrLinearArgs& a, hipStream_t s);
};
template <int XB, int WB> constexpr DirectTile direct_tile() { return {XB, WB, 160 * 1024 / direct_lds_bytes<XB, WB>(), launch_direct<XB, WB>}; }
static constexpr DirectTile DIRECT_TILES[] = {
    direct_tile<1, 1>(), direct_tile<1, 2>(), direct_tile<1, 3>(), direct_tile<1, 4>(), direct_tile<2, 2>(), direct_tile<2, 3>(),
    direct_tile<2, 4>(), direct_tile<3, 2>(), direct_tile<3, 3>(), direct_tile<3, 4>(), direct_tile<4, 3>(), direct_tile<4, 4>(),
};

// The tile of linear_direct_kernel, or none: slices of k and a merge.
// Of the tiles whose workgroups all run at once, the one that asks for the fewest bytes per CU (of equal ones the squarest: fewer
// workgroups read the same weights or the same x).  Its time and that of the slices are estimated from fits to 19 shapes at 11
// row counts each (1 .. 128), weights not in the caches, on which they are right to 6 % (rms):
//   direct   launch + the larger of 0.1 + 0.058 (xb + wb) us a chunk of k and the weights at the HBM rate
//   slices   two launches + weights, partial sums, and rows of x (which the slices read once per 128 features)
// and the direct kernel is taken where it is the faster one by 7 %.  us, slices / direct: 3584 x 3584 14.8 / 12.5 at 64 rows,
// 10.4 / 10.0 at one, 16.9 / 15.6 at 128; 4608 x 3584 16.0 / 15.0 at 64; 6144 x 4096 19.4 / 19.1 at 64; 512 x 3584 6.6 / 8.9 at
// one and 9.8 / 9.3 at 128; 512 x 512 7.9 / 3.7; 8192 x 8192 38.0 / 34.5 at 64; 3584 x 18944 36.5 / 47.6 at 64; 2048 x 8192
// 15.6 / 22.7 at 64: with few features or a long k the slices have more CUs at work, or longer streams.
static const DirectTile* direct_plan(int32_t M, int32_t N, int32_t K, int n_split)
{
    if (tr_knob(TR_KNOB_LIN_SPLIT, 0) || tr_knob(TR_KNOB_LIN_MSPLIT, 0)) return nullptr; // a forced split is a split
    const int blocks = N / 16;
    const DirectTile* best = nullptr;
    for (const DirectTile& t : DIRECT_TILES) {
        const int row_tiles = (M + 16 * t.xb - 1) / (16 * t.xb), tiles = (blocks + t.wb - 1) / t.wb;
        // A feature tile's row tiles all go to one XCD, so they have to fit there too: a workgroup that waits for a CU doubles the
        // time (5408 x 8192 at 127 rows in tiles of 48 x 64, 33 workgroups for 32 CUs: 60.7 us, the slices 38.5).
        if ((int64_t)row_tiles * tiles > TrChip::CUS) continue;
        if (row_tiles * ((tiles + TrChip::XCDS - 1) / TrChip::XCDS) > t.per_cu * (TrChip::CUS / TrChip::XCDS)) continue;
        const int d = best ? t.xb + t.wb - best->xb - best->wb : -1;
        if (d < 0 || (d == 0 && abs(t.xb - t.wb) < abs(best->xb - best->wb))) best = &t;
    }
    if (!best) return nullptr;
    const double mb = 2e-6 * N * (double)K, chunks = (K + LIN_CK - 1) / LIN_CK;
    const double direct = 2.8 + std::max(chunks * (0.1 + 0.058 * (best->xb + best->wb)), mb / 5.3 + 1.5);
    const double slices = 6.3 + 0.146 * mb + (n_split > 1 ? 0.71e-6 * n_split * M * (double)N : 0.0) + (0.69 + 0.0314 * mb) * M / 32;
    if (direct > 0.93 * slices) return nullptr;
    if (K <= 4096 || K == 8192) return best;
    // Rows further apart than 8 KB take the direct kernel up to 1.4 times that estimate (8864 features x 8160 at 44 rows 58 us, the
    // slices 41; 6144 x 8224 at 59 rows 39 / 32), but for two whole 8 KB, where its tiles start their walks in different places (59
    // sizes of 8192 values: 1.02 .. 1.29 times as fast as the slices).  There both are estimated from fits to 560 sizes of 4112 ..
    // 20000 values as well, and the line is a tenth: none of the 86 that it sends to the direct kernel is slower by more than 2 %.
    const double far_direct = 2.6 + chunks * (0.10 + 0.06 * (best->xb + best->wb)) + 0.054 * mb;
    const double far_slices = 3.0 + 0.127 * mb + (n_split > 1 ? 2.3 + 2.0e-6 * n_split * M * (double)N : 0.0) + (0.75 + 0.0097 * mb) * M / 32 +
                              0.55 * ceil(chunks / n_split);
    return far_direct <= 0.9 * far_slices ? best : nullptr;
}

extern "C" int tr_linear_direct_tile(int32_t M, int32_t N, int32_t K)
{
    const DirectTile* t = M > 0 ? direct_plan(M, N, K, tr_linear_splits(M, N, K)) : nullptr;
    return t ? 16 * t->xb + t->wb : 0;
}

template <int MT, bool DEEP>
static int launch_linear_mt(const TrLinearArgs& a, hipStream_t s)
{
    auto kern = linear_kernel<MT, DEEP>;
    constexpr int lds = lin_slots<MT, DEEP>() * lin_slot_bytes<MT>();
    static std::atomic<uint64_t> configured{0};
    if (int rc = tr_raise_lds_limit((const void*)kern, lds, &configured)) return rc;
    const int items = (a.N / 32 + 3) / 4 * a.n_split;
    const int blocks = a.m_split == 2 ? 16 * ((items + 7) / 8) : items;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, s, a);
    TR_HIP(hipGetLastError());
    return TR_OK;
}

int tr_launch_linear(const void* x, int32_t n_out, const void* const* w, void* const* y, const int32_t* n_features, void* partial,
                     int32_t M, int32_t K, hipStream_t s)
{
    TrLinearArgs a;
    memset(&a, 0, sizeof a);
    a.x = (const __bf16*)x;
    a.n_out = n_out;
    int32_t N = 0;
    for (int j = 0; j < n_out; ++j) {
        a.w[j] = (const __bf16*)w[j];
        a.y[j] = (__bf16*)y[j];
        a.tile0[j] = N / 32;
        N += n_features[j];
    }
    for (int j = n_out; j <= TR_LINEAR_MAX_OUT; ++j) a.tile0[j] = N / 32;
    a.partial = (float*)partial;
    a.M = M;
    a.N = N;
    a.K = K;
    const int n_split = tr_linear_splits(M, N, K);
    if (const DirectTile* t = direct_plan(M, N, K, n_split)) {
        a.n_split = a.m_split = 1;
        a.row_tiles = (M + 16 * t->xb - 1) / (16 * t->xb);
        a.row_magic = 65536 / a.row_tiles + 1;
        return t->launch(a, s);
    }
    a.n_split = n_split;
    a.m_split = lin_m_split(M, N, K);
    int rc;
    const bool deep = !lin_large(N, K);
    switch (a.m_split == 2 ? 2 : (M + 31) / 32) {
    case 1: rc = deep ? launch_linear_mt<1, true>(a, s) : launch_linear_mt<1, false>(a, s); break;
    case 2: rc = deep ? launch_linear_mt<2, true>(a, s) : launch_linear_mt<2, false>(a, s); break;
    case 3: rc = deep ? launch_linear_mt<3, true>(a, s) : launch_linear_mt<3, false>(a, s); break;
    default: rc = deep ? launch_linear_mt<4, true>(a, s) : launch_linear_mt<4, false>(a, s); break;
    }
    if (rc) return rc;
    if (a.n_split > 1) {
        const int64_t total4 = (int64_t)M * N / 4;
        hipLaunchKernelGGL(linear_combine_kernel, dim3((unsigned)((total4 + 255) / 256)), dim3(256), 0, s, a);
        TR_HIP(hipGetLastError());
    }
    return TR_OK;
}
