// fp32 attention path: plain FMA arithmetic, one workgroup per (query token, query head).
// Used for fp32 storage.  Such requests are small (the tiny fp32 configuration: 64 rows over 144 keys), so a launch is
// pure latency and the layout is chosen for a short dependent chain:
//   * D/4 lanes share a key, a lane holds four channels: K and V rows are read as whole 16-byte pieces, and the lane that
//     multiplied its channels of K accumulates the same channels of V.
//   * Each such group of lanes walks its own keys, KEYS of them at a time with all their loads in flight (the first batch
//     is requested before the query is rotated), and keeps its own running maximum, denominator and weighted sum.  The
//     groups of the workgroup are merged once, through LDS.
// One wave per row with a key per lane, then a channel per lane, read K with a stride of a row and walked V in a chain as
// long as the keys: 16 query tokens x 4 heads over 144 keys of 64 channels took 16.4 us in the trace, now 6.4 (the whole
// request 19.1 -> 9.6 us).
#include "tr_internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4))); // the caller's rows may start at any element

struct F32Row {
    const float* q;   // raw query vector
    float* out;
    int key_lo, key_hi, kvh;
    int pos;
};

constexpr int KEYS = 8; // keys in flight per group of lanes

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
        sincos((double)r.pos * theta[tid], &sn, &cn);
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
        l *= alpha;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] *= alpha;
#pragma unroll
        for (int i = 0; i < KEYS; ++i) {
            const bool visible = j + GROUPS * i <= r.key_hi && s[i] != -INFINITY;
            const float p = visible ? expf(s[i] - top) : 0.0f;
            l += p;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = visible ? fmaf(p, vx[i][e], o[e]) : o[e];
        }
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

// Waves per row.  A row is a chain of latencies, which more waves shorten; but every wave requests a whole batch of keys
// (`batch` of them) whether the row sees that many or not, and once the rows alone fill the chip a wave without keys of its
// own only delays another row.  So the more rows there are, the more keys a wave has to have.  keys: what a row sees on
// average.  us for 1 / 2 / 4 / 8 waves, head size 64 (in brackets: one wave per row with a key per lane, the form before):
//   64 rows     24 keys   4.8  4.8  4.9  6.0 (5.4)    136 keys  12.2  8.0  7.0  6.4 (10.4)   2040 keys  123  65   35   22  (98)
//   512 rows    24 keys   5.1  5.0  5.5  8.1 (5.6)    136 keys  12.4  8.7  7.9  9.2 (11.0)   2040 keys  129  71   40   42  (121)
//   2048 rows   16 keys   6.2  8.8  15   27  (6.9)    112 keys  13.6  15   17   26  (15.6)   2016 keys  145  144  120  155 (203)
//   16384 rows  32 keys   30   41   82   188 (31)     256 keys  132   139  176  282 (170)    1024 keys  477  466  496  684 (614)
int waves_per_row(int64_t rows, int64_t keys, int head_dim)
{
    const int batch = KEYS * 256 / head_dim;
    const int least = rows <= 512 ? batch / 4 : rows <= 2048 ? batch : 2 * batch;
    int waves = rows <= 256 ? 8 : rows <= 2048 ? 4 : 2;
    while (waves > 1 && (int64_t)waves * least > keys) waves /= 2;
    return waves;
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
    int64_t toks = 0, keys = 0;
    for (int i = 0; i < a.n_seq; ++i) {
        const int64_t n = a.seq[i].n_q;
        toks += n;
        keys += n * (a.seq[i].kv_len - n) + n * (n + 1) / 2;
    }
    const int waves = waves_per_row(total_rows, toks > 0 ? keys / toks : 0, head_dim);
#define KERN(D) (waves == 8 ? prefix_attn_f32_kernel<D, 8> : waves == 4 ? prefix_attn_f32_kernel<D, 4> : waves == 2 ? prefix_attn_f32_kernel<D, 2> : prefix_attn_f32_kernel<D, 1>)
    return launch_rows(head_dim == 128 ? KERN(128) : KERN(64), a, total_rows, 64 * waves, s);
#undef KERN
}

int tr_launch_blockdiag_attn_f32(const TrBlockDiagArgs& a, int64_t mean_keys, int head_dim, hipStream_t s)
{
    const int64_t rows = (int64_t)a.total_tokens * a.n_q_heads;
    const int waves = waves_per_row(rows, mean_keys, head_dim);
#define KERN(D) (waves == 8 ? blockdiag_attn_f32_kernel<D, 8> : waves == 4 ? blockdiag_attn_f32_kernel<D, 4> : waves == 2 ? blockdiag_attn_f32_kernel<D, 2> : blockdiag_attn_f32_kernel<D, 1>)
    return launch_rows(head_dim == 128 ? KERN(128) : KERN(64), a, rows, 64 * waves, s);
#undef KERN
}
