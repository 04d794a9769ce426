// fp32 attention path: plain FMA arithmetic, one workgroup per (query token, query head).
// Used for fp32 storage.  Most such requests are small (the tiny fp32 configuration: 64 rows over 144 keys), so a launch
// is latency and the layout is chosen for a short dependent chain:
//   * D/4 lanes share a key, a lane holds four channels: K and V rows are read as whole 16-byte pieces, and the lane that
//     multiplied its channels of K accumulates the same channels of V.
//   * Each such group of lanes walks its own keys, KEYS of them at a time with all their loads in flight (the first batch
//     is requested before the query is rotated), and keeps its own running maximum, denominator and weighted sum.  The
//     groups of the workgroup are merged once, through LDS.
// One wave per row with a key per lane, then a channel per lane, read K with a stride of a row and walked V in a chain as
// long as the keys: 16 query tokens x 4 heads over 144 keys of 64 channels took 16.4 us in the trace, now 6.1 (the whole
// request 19.1 -> 9.3 us), 2048 rows of 2048 keys 276 -> 99.
#include "tr_internal.h"

#include <algorithm>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4))); // the caller's rows may start at any element

struct F32Row {
    const float* q;   // raw query vector
    float* out;
    int key_lo, key_hi, kvh;
    int pos;
};

// Keys in flight per group of lanes.  Four take 85 vector registers, so five waves share a SIMD; with eight (134, three waves)
// 16384 rows of 1024 keys took 410 us against 353 (head size 128: 897, 732), packed chunks of 24 tokens, 153600 rows, 179
// against 123, and 64 rows of 128 keys 6.3 against 6.0.
constexpr int KEYS = 4;

// Sum over the D/4 lanes of a key (a power of two, neighbouring lanes).
template <int LANES> __device__ __forceinline__ float group_sum(float x)
{
#pragma unroll
    for (int o = LANES / 2; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

template <int D, int NW>
__device__ __forceinline__ void attn_f32_row(const F32Row& r, const float* __restrict__ k, const float* __restrict__ v,
                                             int n_kv_heads, const double* theta, float scale, int rope_half)
{
    constexpr int LANES = D / 4, GROUPS = 64 * NW / LANES;
    __shared__ f32x4 qs[D / 4];
    __shared__ f32x4 os[GROUPS][D / 4];
    __shared__ float ml[GROUPS][2];
    const int tid = threadIdx.x, grp = tid / LANES, c4 = tid % LANES;
    const int64_t row = (int64_t)n_kv_heads * (D / 4); // 16-byte pieces per cache row
    const f32x4_any* kp = (const f32x4_any*)k + (int64_t)r.kvh * (D / 4) + c4;
    const f32x4_any* vp = (const f32x4_any*)v + (int64_t)r.kvh * (D / 4) + c4;
    f32x4 kx[KEYS], vx[KEYS];
    auto load = [&](int j0) { // keys past the last visible one read that one and get no weight
#pragma unroll
        for (int i = 0; i < KEYS; ++i) {
            const int64_t at = (int64_t)min(j0 + GROUPS * i, r.key_hi) * row;
            kx[i] = kp[at];
            vx[i] = vp[at];
        }
    };
    int j = r.key_lo + grp;
    load(j);
    if (tid < D / 2) { // rotation in fp64, one pair per thread
        double sn, cn;
        tr_sincos((double)r.pos * theta[tid], &sn, &cn);
        const int ia = rope_half ? tid : 2 * tid, ib = rope_half ? tid + D / 2 : 2 * tid + 1; // the pair's two channels
        const double xa = (double)r.q[ia], xb = (double)r.q[ib];
        ((float*)qs)[ia] = (float)(xa * cn - xb * sn);
        ((float*)qs)[ib] = (float)(xb * cn + xa * sn);
    }
    __syncthreads();
    const f32x4 q = qs[c4];
    f32x4 o = {0.0f, 0.0f, 0.0f, 0.0f};
    float m = -INFINITY, l = 0.0f;
    while (j <= r.key_hi) {
        float s[KEYS], top = m;
#pragma unroll
        for (int i = 0; i < KEYS; ++i) {
            float x = q[0] * kx[i][0];
#pragma unroll
            for (int e = 1; e < 4; ++e) x = fmaf(q[e], kx[i][e], x);
            s[i] = j + GROUPS * i <= r.key_hi ? group_sum<LANES>(x) * scale : -INFINITY;
            top = fmaxf(top, s[i]);
        }
        // a batch whose scores are all -inf (a product that overflowed) gives the group no weight, it must not make NaN of
        // the other groups' keys
        const float alpha = top == -INFINITY ? 1.0f : expf(m - top);
        // a batch is summed before it is added, so the running sums are rounded once per batch (relative error against 64 bits,
        // mean over 48 launches of 9 .. 4200 keys, 2.2e-7 -> 1.8e-7; a step per key in one chain of all keys gave 6.3e-7)
        f32x4 ob = {0.0f, 0.0f, 0.0f, 0.0f};
        float lb = 0.0f;
#pragma unroll
        for (int i = 0; i < KEYS; ++i) {
            const bool visible = j + GROUPS * i <= r.key_hi && s[i] != -INFINITY;
            const float p = visible ? expf(s[i] - top) : 0.0f;
            lb += p;
#pragma unroll
            for (int e = 0; e < 4; ++e) ob[e] = visible ? fmaf(p, vx[i][e], ob[e]) : ob[e];
        }
        l = fmaf(l, alpha, lb);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = fmaf(o[e], alpha, ob[e]);
        m = top;
        j += GROUPS * KEYS;
        if (j <= r.key_hi) load(j);
    }
    os[grp][c4] = o;
    if (c4 == 0) {
        ml[grp][0] = m;
        ml[grp][1] = l;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < (D + 64 * NW - 1) / (64 * NW); ++i) { // a channel at a time; groups without a visible key have weight 0
        const int t = tid + 64 * NW * i;
        if (t >= D) break;
        float M = -INFINITY, L = 0.0f, x = 0.0f;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) M = fmaxf(M, ml[g][0]);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const float w = expf(ml[g][0] - M);
            L = fmaf(w, ml[g][1], L);
            x = fmaf(w, ((const float*)os[g])[t], x);
        }
        r.out[t] = x / L;
    }
}

template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void prefix_attn_f32_kernel(const TrPrefixArgs a, uint32_t row0)
{
    // row = (packed token of the call, query head); this launch covers rows from row0 on
    const uint32_t row = row0 + blockIdx.x;
    const int tq = a.seq[0].q_row0 + (int)(row / (uint32_t)a.n_q_heads);
    const int hq = (int)(row % (uint32_t)a.n_q_heads);
    int lo = 0, hi = a.n_seq - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (a.seq[mid].q_row0 <= tq) lo = mid; else hi = mid - 1;
    }
    const TrSeqDesc sd = a.seq[lo];
    const int i = tq - sd.q_row0;
    F32Row r;
    r.q = (const float*)a.q + ((int64_t)tq * a.n_q_heads + hq) * D;
    r.out = (float*)a.out + ((int64_t)tq * a.n_q_heads + hq) * D;
    r.key_lo = sd.kv_row0;
    r.key_hi = sd.kv_row0 + (sd.kv_len - sd.n_q) + i;
    r.kvh = hq / a.group;
    r.pos = a.q_pos[tq];
    attn_f32_row<D, NW>(r, (const float*)a.k, (const float*)a.v, a.n_kv_heads, a.theta, a.scale, a.rope_half);
}

template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void blockdiag_attn_f32_kernel(const TrBlockDiagArgs a, uint32_t row0)
{
    const uint32_t row = row0 + blockIdx.x;
    const int t = (int)(row / (uint32_t)a.n_q_heads);
    const int hq = (int)(row % (uint32_t)a.n_q_heads);
    F32Row r;
    r.q = (const float*)a.q + ((int64_t)t * a.n_q_heads + hq) * D;
    r.out = (float*)a.out + ((int64_t)t * a.n_q_heads + hq) * D;
    r.key_lo = min(max(a.tok_start[t], 0), t);
    r.key_hi = t;
    r.kvh = hq / a.group;
    r.pos = a.pos ? a.pos[t] : t - r.key_lo;
    attn_f32_row<D, NW>(r, (const float*)a.k, (const float*)a.v, a.n_kv_heads, a.theta, a.scale, a.rope_half);
}

// Waves per row.  A row is a chain of latencies, one for each batch of keys (16 at head size 64, 8 at 128), which more waves
// shorten; but a compute unit runs about sixteen of these waves at a time, so with many rows the workgroups take turns.  The
// launch is priced in units of a batch's latency, which grows by 8 % with every resident wave, a turn costing one more, and
// the cheapest division is taken.  Where the rows see very different numbers of keys (a causal triangle) the last turn fills
// up as short rows end, and the longest row's batches come on top.  mean, longest: keys a row sees.  Over 352 launches (64 to
// 262144 rows of 8 to 2048 keys, squares, triangles, packed chunks, both head sizes) the choice is within 0.6 % of the best of
// the four on average and 11 % at worst.  us for 1 / 2 / 4 / 8 waves:
//                head size 64                                         head size 128
//   64 rows      24 keys    5.0  4.3  4.6  5.2                        16 keys    6.2  5.0  4.4  4.6
//                128 keys   11.4 7.8  6.4  6.0                        64 keys    12.6 8.1  6.3  5.5
//   768 rows     32 keys    5.9  5.4  5.3  9.1                        24 keys    7.7  6.1  5.4  8.1
//                512 keys   36.3 21.9 15.6 18.8                       256 keys   39.9 23.2 16.0 16.9
//   2048 rows    48 keys    7.7  6.9  8.6  16.9                       96 keys    20.0 14.9 15.9 22.1
//                2048 keys  140  99.4 102  113                        2048 keys  307  199  202  219
//   16384 rows   128 keys   54.9 59.1 75.5 127                        128 keys   108  108  123  165
//                1024 keys  353  362  374  430                        1024 keys  732  922  798  891
int waves_per_row(int64_t rows, int64_t mean, int64_t longest, int head_dim)
{
    const int64_t per_cu = (rows + TrChip::CUS - 1) / TrChip::CUS;
    const bool uneven = 5 * mean < 4 * longest;
    int best = 1;
    double least = 0.0;
    for (int w = 1; w <= 8; w *= 2) {
        const int64_t resident = 16 / w, full = per_cu / resident, rest = per_cu % resident;
        auto batches = [&](int64_t keys) { return std::max(1.0, (double)keys / (w * (KEYS * 256 / head_dim)) + 0.25); };
        auto turn = [&](int64_t n) { return 1.0 + batches(mean) * (1.0 + 0.08 * (double)(n * w)); };
        double cost = (double)full * turn(resident) + 0.7 * (batches(longest) - batches(mean));
        if (rest) cost += uneven && full ? turn(resident) * (double)rest / (double)resident : turn(rest);
        if (w == 1 || cost < least) {
            least = cost;
            best = w;
        }
    }
    return best;
}

// kern over `rows` rows with `threads` threads each, in launches of at most 2^31 threads (one has fewer than 2^32)
template <class Args> int launch_rows(void (*kern)(Args, uint32_t), const Args& a, int64_t rows, int threads, hipStream_t s)
{
    const int64_t most = ((int64_t)1 << 31) / threads;
    for (int64_t row0 = 0; row0 < rows; row0 += most) {
        const int64_t n = rows - row0 < most ? rows - row0 : most;
        hipLaunchKernelGGL(kern, dim3((unsigned)n), dim3(threads), 0, s, a, (uint32_t)row0);
        TR_HIP(hipGetLastError());
    }
    return TR_OK;
}

} // namespace

int tr_launch_prefix_attn_f32(const TrPrefixArgs& a, int head_dim, int total_rows, hipStream_t s)
{
    int64_t toks = 0, keys = 0, longest = 0;
    for (int i = 0; i < a.n_seq; ++i) {
        const int64_t n = a.seq[i].n_q;
        toks += n;
        keys += n * (a.seq[i].kv_len - n) + n * (n + 1) / 2;
        if (n > 0) longest = std::max<int64_t>(longest, a.seq[i].kv_len);
    }
    const int waves = waves_per_row(total_rows, toks > 0 ? keys / toks : 0, longest, head_dim);
#define KERN(D) (waves == 8 ? prefix_attn_f32_kernel<D, 8> : waves == 4 ? prefix_attn_f32_kernel<D, 4> : waves == 2 ? prefix_attn_f32_kernel<D, 2> : prefix_attn_f32_kernel<D, 1>)
    return launch_rows(head_dim == 128 ? KERN(128) : KERN(64), a, total_rows, 64 * waves, s);
#undef KERN
}

int tr_launch_blockdiag_attn_f32(const TrBlockDiagArgs& a, int64_t longest, int head_dim, hipStream_t s)
{
    const int64_t rows = (int64_t)a.total_tokens * a.n_q_heads;
    const int waves = waves_per_row(rows, longest / 2, longest, head_dim);
#define KERN(D) (waves == 8 ? blockdiag_attn_f32_kernel<D, 8> : waves == 4 ? blockdiag_attn_f32_kernel<D, 4> : waves == 2 ? blockdiag_attn_f32_kernel<D, 2> : blockdiag_attn_f32_kernel<D, 1>)
    return launch_rows(head_dim == 128 ? KERN(128) : KERN(64), a, rows, 64 * waves, s);
#undef KERN
}
