// Host side of the C-ABI under AddressSanitizer and UndefinedBehaviorSanitizer, on the CPU.
//
// Built by tests/test_sanitizers.py from csrc/tr_api.hip (host pass compiled with -fsanitize=address,undefined) and
// this file, which stands in for the kernel launchers of the other translation units: no kernel runs, with or
// without a GPU in the machine.  Every entry point is driven with seeded random shapes and request mixes; "device" buffers are ordinary
// host allocations that nothing dereferences.  The launcher stand-ins receive the argument blocks the real kernels
// would get and check, on the host, what a kernel relies on without checking it itself: descriptor counts inside
// their arrays, copy runs inside the source and the destination, work-item counts that match the descriptors, and
// partial-result rows that fit the workspace the matching *_workspace_size() call announced.
// Exit status 0 and "host abi sanitizer run ok" on stdout mean no check and no sanitizer fired.
#include <hip/hip_runtime.h>

#include <cinttypes>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/turborag.h"
#include "../../paper_2410_07590_amd/csrc/tr_internal.h"

namespace {

struct Expect {
    int64_t src_rows = 0;       // rows of the store (assemble) or of the new-token arrays (append)
    int64_t dst_rows = 0;       // capacity of the destination cache
    const char* ws = nullptr;   // workspace handed to the call
    size_t ws_bytes = 0;
    int head_dim = 0;
    long launches = 0;
    int64_t next_src = -1, next_dst = 0; // >= 0: appended rows follow one another from here, over all launches
    int64_t next_pos = -1;               // >= 0: so do the position ids of the descriptors
} g_ex;

long g_checks = 0;
const char* g_call = "";   // the library call in progress, for the messages

#define REQUIRE(cond, ...)                                                      \
    do {                                                                        \
        ++g_checks;                                                             \
        if (!(cond)) {                                                          \
            std::fprintf(stderr, "host_abi_san: %s:%d: %s: ", __FILE__, __LINE__, #cond); \
            std::fprintf(stderr, __VA_ARGS__);                                  \
            std::fprintf(stderr, "\n  during %s\n", g_call);                   \
            std::exit(1);                                                       \
        }                                                                       \
    } while (0)

void partial_rows_fit(const _Float16* ws_o, const float* ws_ml, int64_t rows, const char* who, bool f32 = false)
{
    if (rows == 0) return;
    const char *end = g_ex.ws + g_ex.ws_bytes, *a0 = (const char*)ws_o, *a1 = a0 + rows * g_ex.head_dim * (f32 ? 4 : 2);
    REQUIRE(a0 >= g_ex.ws && a1 <= end, "%s: %" PRId64 " partial rows leave the workspace of %zu bytes", who, rows, g_ex.ws_bytes);
    REQUIRE((const char*)ws_ml >= g_ex.ws && (const char*)(ws_ml + rows * 2) <= end, "%s: statistics of %" PRId64 " partial rows leave the workspace", who, rows);
    const char *b0 = (const char*)ws_ml, *b1 = (const char*)(ws_ml + rows * 2);
    REQUIRE(a1 <= b0 || b1 <= a0, "%s: partial outputs and their statistics overlap", who);
}

struct Rng {
    uint64_t s;
    explicit Rng(uint64_t seed) : s(seed * 0x9E3779B97F4A7C15ull + 1) {}
    uint32_t next() { s = s * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(s >> 33); }
    int in(int lo, int hi) { return lo + (int)(next() % (uint32_t)(hi - lo + 1)); }
};

}  // namespace

// ---- launcher stand-ins ------------------------------------------------------------------------------------------

int tr_launch_assemble(const TrAssembleArgs& a, int, int n_blocks, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(a.n_desc >= 0 && a.n_desc <= TR_MAX_COPY_DESC, "assemble: %d descriptors", a.n_desc);
    REQUIRE(a.span_units > 0 && a.span_units % 256 == 0, "assemble: span of %d units", a.span_units);
    int blk = 0;
    for (int i = 0; i < a.n_desc; ++i) {
        const TrCopyDesc& d = a.desc[i];
        REQUIRE(d.n_rows > 0, "assemble: run %d is empty", i);
        REQUIRE(d.src_row >= 0 && (int64_t)d.src_row + d.n_rows <= g_ex.src_rows, "assemble: run %d reads rows %d..+%d of %" PRId64, i, d.src_row, d.n_rows, g_ex.src_rows);
        REQUIRE(d.dst_row >= 0 && (int64_t)d.dst_row + d.n_rows <= g_ex.dst_rows, "assemble: run %d writes rows %d..+%d of %" PRId64, i, d.dst_row, d.n_rows, g_ex.dst_rows);
        REQUIRE(d.blk_start == blk, "assemble: run %d starts at block %d, expected %d", i, d.blk_start, blk);
        blk += (int)(((int64_t)d.n_rows * a.row_units + a.span_units - 1) / a.span_units);
    }
    if (a.app.n_q > 0) {
        REQUIRE(a.app.first_block == blk, "assemble: appended tokens start at block %d, expected %d", a.app.first_block, blk);
        REQUIRE(a.app.dst_row0 >= 0 && (int64_t)a.app.dst_row0 + a.app.n_q <= g_ex.dst_rows, "assemble: appended tokens leave the cache");
        REQUIRE(n_blocks > blk, "assemble: no block for the appended tokens");
        REQUIRE(n_blocks - blk == tr_append_blocks(a.app.n_q, a.row_units, a.half_dim), "assemble: %d blocks for %d appended tokens", n_blocks - blk, a.app.n_q);
        REQUIRE((int64_t)n_blocks * 256 < (int64_t)1 << 32, "assemble: %d blocks in one launch", n_blocks);
        g_ex.next_dst += g_ex.next_src >= 0 ? a.app.n_q : 0;
    } else {
        REQUIRE(n_blocks == blk, "assemble: %d blocks launched, descriptors cover %d", n_blocks, blk);
    }
    return 0;
}

int tr_launch_append(const TrAppendArgs& a, int dtype, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(a.n_desc >= 0 && a.n_desc <= TR_MAX_APPEND_DESC, "append: %d descriptors", a.n_desc);
    int64_t tokens = 0;
    for (int i = 0; i < a.n_desc; ++i) {
        const TrAppendDesc& d = a.desc[i];
        REQUIRE(d.n_q >= 0 && d.q_row0 >= 0 && (int64_t)d.q_row0 + d.n_q <= g_ex.src_rows, "append: request %d reads tokens %d..+%d of %" PRId64, i, d.q_row0, d.n_q, g_ex.src_rows);
        REQUIRE(d.dst_row0 >= 0 && (int64_t)d.dst_row0 + d.n_q <= g_ex.dst_rows, "append: request %d writes rows %d..+%d of %" PRId64, i, d.dst_row0, d.n_q, g_ex.dst_rows);
        REQUIRE(a.tok0[i] == tokens, "append: request %d starts at token %d of the launch, expected %" PRId64, i, a.tok0[i], tokens);
        if (g_ex.next_src >= 0) {
            REQUIRE(d.q_row0 == g_ex.next_src && d.dst_row0 == g_ex.next_dst, "append: rows %d -> %d, expected %" PRId64 " -> %" PRId64, d.q_row0, d.dst_row0, g_ex.next_src, g_ex.next_dst);
            REQUIRE(g_ex.next_pos < 0 || d.pos0 == g_ex.next_pos, "append: position %d, expected %" PRId64, d.pos0, g_ex.next_pos);
            g_ex.next_src += d.n_q;
            g_ex.next_dst += d.n_q;
            g_ex.next_pos += g_ex.next_pos >= 0 ? d.n_q : 0;
        }
        tokens += d.n_q;
    }
    const int units = a.head_dim * (dtype == TR_BF16 ? 2 : 4) / 16;
    REQUIRE(tokens <= TR_MAX_APPEND_TOKENS && tr_append_blocks(tokens, a.n_kv_heads * units, a.head_dim / 2) * 64 * TR_APPEND_WAVES_PER_BLOCK < (int64_t)1 << 32,
            "append: %" PRId64 " tokens in one launch", tokens);
    REQUIRE(tokens == a.total_tokens, "append: %" PRId64 " tokens in the descriptors, %d announced", tokens, a.total_tokens);
    return 0;
}

static void check_prefix(const TrPrefixArgs& a, int wg_rows, const char* who)
{
    REQUIRE(a.n_seq >= 1 && a.n_seq <= TR_MAX_SEQ, "%s: %d requests in one launch", who, a.n_seq);
    REQUIRE(a.group == a.n_q_heads / a.n_kv_heads, "%s: group %d", who, a.group);
    int item = 0;
    int64_t rows = 0;
    for (int i = 0; i < a.n_seq; ++i) {
        const TrSeqDesc& d = a.seq[i];
        REQUIRE(d.item0 == item, "%s: request %d starts at item %d, expected %d", who, i, d.item0, item);
        REQUIRE(d.n_split >= 1 && d.n_tiles >= 1, "%s: request %d has %d tiles, %d splits", who, i, d.n_tiles, d.n_split);
        if (wg_rows > 32)
            REQUIRE((int64_t)d.n_tiles * a.tok_per_tile >= d.n_q, "%s: request %d: %d tiles of %d tokens for %d tokens", who, i, d.n_tiles, a.tok_per_tile, d.n_q);
        REQUIRE(d.n_split == 1 || (d.split_len > 0 && d.split_len % 64 == 0), "%s: request %d: split length %d", who, i, d.split_len);
        REQUIRE((int64_t)d.n_split * d.split_len >= d.kv_len || d.n_split == 1, "%s: request %d: %d splits of %d keys for %d keys", who, i, d.n_split, d.split_len, d.kv_len);
        item += d.n_tiles * d.n_split * a.n_kv_heads;
        if (d.n_split > 1) {
            const int64_t last = (int64_t)d.ws_row0 + (int64_t)d.n_split * a.n_kv_heads * d.n_q * a.group;
            rows = last > rows ? last : rows;
        }
    }
    REQUIRE(item == a.n_items, "%s: %d items in the descriptors, %d announced", who, item, a.n_items);
    partial_rows_fit(a.ws_o, a.ws_ml, rows, who, a.partial_f32);
}

int tr_launch_prefix_attn(const TrPrefixArgs& a, int, int wg_rows, bool, int, hipStream_t)
{
    ++g_ex.launches;
    check_prefix(a, wg_rows, "prefix attention");
    return 0;
}

int tr_launch_prefix_attn_f32(const TrPrefixArgs& a, int, int, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(a.n_seq >= 1 && a.n_seq <= TR_MAX_SEQ, "fp32 prefix attention: %d requests in one launch", a.n_seq);
    return 0;
}

int tr_launch_rope_table(double*, int n_pos, int half_dim, const double*, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(n_pos >= 0 && half_dim > 0 && half_dim <= 64, "rope table: %d positions, %d pairs", n_pos, half_dim);
    return 0;
}

int tr_launch_rope_rows(const void*, void*, const int32_t*, int n_chunks, int max_chunk_len, int32_t*, const double*, int table_rows,
                        int64_t total_tokens, const tr_shape*, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(n_chunks >= 0 && total_tokens >= 0 && table_rows >= max_chunk_len, "rope rows: table of %d rows for chunks of up to %d", table_rows, max_chunk_len);
    return 0;
}

int tr_launch_blockdiag_attn(const TrBlockDiagArgs& a, const TrPrefixArgs* combine, int, int, int, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(a.n_seg >= 1 && a.n_seg <= TR_MAX_BD_SEG, "block-diagonal attention: %d segments", a.n_seg);
    int item = 0, tiles = 0;
    int64_t rows = 0;
    for (int i = 0; i < a.n_seg; ++i) {
        const TrBdSeg& s = a.seg[i];
        REQUIRE(s.item0 == item, "block-diagonal attention: segment %d starts at item %d, expected %d", i, s.item0, item);
        REQUIRE(s.n_tiles >= 1 && s.n_split >= 1 && s.tile_hi - s.n_tiles + 1 >= 0 && s.tile_hi < a.n_tiles, "block-diagonal attention: segment %d covers tiles %d..%d of %d",
                i, s.tile_hi - s.n_tiles + 1, s.tile_hi, a.n_tiles);
        REQUIRE(s.tok0 >= 0 && (int64_t)s.tok0 + s.n_tok <= a.total_tokens, "block-diagonal attention: segment %d covers tokens %d..+%d of %d", i, s.tok0, s.n_tok, a.total_tokens);
        item += s.n_tiles * s.n_split;
        tiles += s.n_tiles;
        if (s.n_split > 1) {
            REQUIRE(s.split_len > 0 && s.split_len % 64 == 0, "block-diagonal attention: segment %d: split length %d", i, s.split_len);
            const int64_t last = (int64_t)s.ws_row0 + (int64_t)s.n_split * a.n_kv_heads * s.n_tok * a.group;
            rows = last > rows ? last : rows;
        }
    }
    REQUIRE(item == a.items_per_head, "block-diagonal attention: %d items per head in the segments, %d announced", item, a.items_per_head);
    REQUIRE(tiles == a.n_tiles, "block-diagonal attention: segments cover %d of %d row tiles", tiles, a.n_tiles);
    partial_rows_fit(a.ws_o, a.ws_ml, rows, "block-diagonal attention");
    if (combine) REQUIRE(combine->n_seq >= 1 && combine->n_seq <= TR_MAX_SEQ, "block-diagonal merge: %d descriptors", combine->n_seq);
    return 0;
}

int tr_launch_gather_attn(const TrGatherArgs& a, const TrPrefixArgs&, int, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(a.n_seg >= 1 && a.n_seg <= TR_MAX_GATHER_SEG, "gather attention: %d segments", a.n_seg);
    int tile = 0;
    for (int i = 0; i < a.n_seg; ++i) {
        const TrGatherSeg& s = a.seg[i];
        REQUIRE(s.tile0 == tile, "gather attention: segment %d starts at tile %d, expected %d", i, s.tile0, tile);
        REQUIRE(s.n_rows > 0 && s.src_row >= 0, "gather attention: segment %d has %d rows from %d", i, s.n_rows, s.src_row);
        if (i + 1 < a.n_seg) REQUIRE((int64_t)s.src_row + s.n_rows <= g_ex.src_rows, "gather attention: segment %d leaves the store", i);
        tile += (s.n_rows + 63) / 64;
    }
    REQUIRE(tile == a.n_tiles_total, "gather attention: %d tiles in the segments, %d announced", tile, a.n_tiles_total);
    REQUIRE(a.n_split >= 1 && (int64_t)a.n_split * a.tiles_per_split >= a.n_tiles_total, "gather attention: %d splits of %d tiles for %d", a.n_split, a.tiles_per_split, a.n_tiles_total);
    REQUIRE(a.n_items == a.row_tiles * a.n_split * a.n_kv_heads, "gather attention: %d items", a.n_items);
    if (a.n_split > 1) partial_rows_fit(a.ws_o, a.ws_ml, (int64_t)a.n_split * a.n_kv_heads * a.n_q * a.group, "gather attention");
    return 0;
}

int tr_launch_blockdiag_attn_f32(const TrBlockDiagArgs& a, int64_t, int, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(a.total_tokens >= 0, "fp32 block-diagonal attention: %d tokens", a.total_tokens);
    return 0;
}

// the real split policy lives beside the kernel; any deterministic count exercises the workspace arithmetic
int tr_linear_splits(int32_t M, int32_t N, int32_t K) { return 1 + (int)(((int64_t)M + N + K / 64) % 4); }

int tr_launch_linear(const void*, int32_t n_out, const void* const* w, void* const* y, const int32_t* n_features, void* partial, int32_t M, int32_t K, hipStream_t)
{
    ++g_ex.launches;
    REQUIRE(n_out >= 1 && n_out <= TR_LINEAR_MAX_OUT, "linear: %d weights", n_out);
    int64_t N = 0;
    for (int j = 0; j < n_out; ++j) {
        REQUIRE(w[j] && y[j] && n_features[j] > 0, "linear: weight %d", j);
        N += n_features[j];
    }
    const int splits = tr_linear_splits(M, (int32_t)N, K);
    if (splits > 1) {
        const char* end = g_ex.ws + g_ex.ws_bytes;
        REQUIRE((const char*)partial >= g_ex.ws && (const char*)partial + (size_t)splits * M * N * 4 <= end, "linear: %d partial sums of %d x %" PRId64 " leave the workspace of %zu bytes",
                splits, M, N, g_ex.ws_bytes);
    }
    return 0;
}

int tr_launch_mfma_loop_probe(int iters, int, float*, hipStream_t, double* flops)
{
    ++g_ex.launches;
    *flops = (double)iters;
    return 0;
}

// ---- the driver --------------------------------------------------------------------------------------------------

namespace {

#define OK(call)                                                                              \
    do {                                                                                      \
        g_call = #call;                                                                       \
        const int rc_ = (call);                                                               \
        REQUIRE(rc_ == TR_OK, "%s returned %d: %s", #call, rc_, tr_last_error());             \
    } while (0)
#define FAILS(call, code)                                                                     \
    do {                                                                                      \
        g_call = #call;                                                                       \
        const int rc_ = (call);                                                               \
        REQUIRE(rc_ == (code), "%s returned %d, expected %d (%s)", #call, rc_, (int)(code), tr_last_error()); \
        REQUIRE(std::strlen(tr_last_error()) > 0, "%s left no message", #call);               \
    } while (0)

tr_shape make_shape(Rng& r)
{
    static const int heads[][2] = {{4, 4}, {28, 4}, {32, 8}, {8, 1}, {16, 8}, {64, 1}, {2, 2}};
    const int i = r.in(0, 6);
    tr_shape s;
    std::memset(&s, 0, sizeof s);
    s.n_q_heads = heads[i][0];
    s.n_kv_heads = heads[i][1];
    s.head_dim = r.in(0, 1) ? 128 : 64;
    s.dtype = r.in(0, 3) ? TR_BF16 : TR_F32;
    s.rope_base = r.in(0, 1) ? 1e6 : 1e4;
    s.rope_layout = r.in(0, 1);
    return s;
}

struct Buffers {   // stand-ins for device memory, 256-byte aligned like real allocations; nothing dereferences them
    std::vector<void*> keep;
    void* get(size_t bytes)
    {
        void* p = std::aligned_alloc(256, ((bytes ? bytes : 1) + 255) / 256 * 256);
        if (!p) std::exit(2);
        keep.push_back(p);
        return p;
    }
    ~Buffers()
    {
        for (void* p : keep) std::free(p);
    }
};

void one_request_mix(uint64_t seed)
{
    Rng r(seed);
    Buffers dev;
    const tr_shape sh = make_shape(r);
    const int esz = sh.dtype == TR_BF16 ? 2 : 4;
    const size_t row_bytes = (size_t)sh.n_kv_heads * sh.head_dim * esz;
    const size_t qrow_bytes = (size_t)sh.n_q_heads * sh.head_dim * esz;
    g_ex.head_dim = sh.head_dim;

    // a store of ragged chunks
    const int n_store = r.in(1, 40);
    std::vector<int64_t> row_start(n_store + 1, 0);
    for (int i = 0; i < n_store; ++i) row_start[i + 1] = row_start[i] + r.in(r.in(0, 9) ? 1 : 0, 300);
    const int64_t store_rows = row_start[n_store];
    tr_store* store = nullptr;
    OK(tr_store_create(&sh, dev.get(store_rows * row_bytes), dev.get(store_rows * row_bytes), row_start.data(), n_store, &store));

    // requests
    const int n_req = r.in(1, 12);
    std::vector<int32_t> ids, cu_chunks(1, 0), modes, cu_q(1, 0);
    std::vector<int64_t> crs(1, 0);
    std::vector<std::vector<int64_t>> offsets(n_req);
    for (int q = 0; q < n_req; ++q) {
        const int k = r.in(0, 12);
        std::vector<int32_t> mine(k);
        for (auto& c : mine) c = r.in(0, n_store - 1);
        const int mode = r.in(0, 1);
        offsets[q].assign(k + 1, -1);
        std::vector<int32_t> pos;
        OK(tr_plan(store, mine.data(), k, mode, offsets[q].data(), nullptr, 0));
        const int64_t n_doc = offsets[q][k];
        pos.assign(n_doc ? n_doc : 1, -1);
        OK(tr_plan(store, mine.data(), k, mode, offsets[q].data(), pos.data(), n_doc));
        if (n_doc > 0) FAILS(tr_plan(store, mine.data(), k, mode, offsets[q].data(), pos.data(), n_doc - 1), TR_ERR_BAD_PLAN);
        const int n_q = r.in(1, r.in(0, 3) ? 40 : 300);
        ids.insert(ids.end(), mine.begin(), mine.end());
        cu_chunks.push_back((int32_t)ids.size());
        modes.push_back(mode);
        cu_q.push_back(cu_q.back() + n_q);
        crs.push_back(crs.back() + n_doc + n_q + r.in(0, 3));
    }
    if (n_store > 0) {
        int32_t bad = n_store;
        int64_t off2[2];
        FAILS(tr_plan(store, &bad, 1, 0, off2, nullptr, 0), TR_ERR_BAD_CHUNK_ID);
    }
    const int64_t cache_rows = crs.back();
    const int total_q = cu_q.back();
    void* ck = dev.get(cache_rows * row_bytes);
    void* cv = dev.get(cache_rows * row_bytes);
    void* qd = dev.get(total_q * qrow_bytes);
    void* od = dev.get(total_q * qrow_bytes);
    void* knew = dev.get(total_q * row_bytes);
    void* vnew = dev.get(total_q * row_bytes);
    const int32_t* q_pos = (const int32_t*)dev.get((size_t)total_q * 4);

    // batched assemble + append
    g_ex.src_rows = store_rows;
    g_ex.dst_rows = cache_rows;
    OK(tr_kv_assemble_batched(store, ids.data(), cu_chunks.data(), modes.data(), crs.data(), n_req, ck, cv, cache_rows, nullptr));
    g_ex.src_rows = total_q;
    OK(tr_kv_append_batched(&sh, knew, vnew, q_pos, cu_q.data(), crs.data(), n_req, ck, cv, cache_rows, nullptr));

    // batched attention; a workspace one byte short is refused before any launch
    {
        const size_t wb = tr_prefill_attn_batched_workspace_size(&sh, cu_q.data(), crs.data(), n_req);
        g_ex.ws = (const char*)dev.get(wb);
        g_ex.ws_bytes = wb;
        OK(tr_prefill_attn_batched(&sh, qd, ck, cv, q_pos, cu_q.data(), crs.data(), n_req, od, (void*)g_ex.ws, wb, nullptr));
        if (wb > 0) {
            const long before = g_ex.launches;
            FAILS(tr_prefill_attn_batched(&sh, qd, ck, cv, q_pos, cu_q.data(), crs.data(), n_req, od, (void*)g_ex.ws, wb - 1, nullptr), TR_ERR_WORKSPACE);
            REQUIRE(g_ex.launches == before, "a refused call launched something");
        }
    }

    // per request: assemble (three forms), append, attention (workspace, static scratch, gather), decode
    for (int q = 0; q < n_req; ++q) {
        const int k = cu_chunks[q + 1] - cu_chunks[q];
        const int32_t* mine = ids.data() + cu_chunks[q];
        const int n_q = cu_q[q + 1] - cu_q[q];
        const int64_t n_doc = offsets[q][k], kv_len = n_doc + n_q;
        g_ex.src_rows = store_rows;
        g_ex.dst_rows = kv_len;
        OK(tr_kv_assemble(store, mine, offsets[q].data(), k, modes[q], ck, cv, kv_len, nullptr));
        OK(tr_kv_assemble_raw(store, mine, offsets[q].data(), k, modes[q], ck, cv, kv_len, nullptr));
        OK(tr_kv_assemble_append(store, mine, offsets[q].data(), k, modes[q], knew, vnew, q_pos, n_q, ck, cv, kv_len, nullptr));
        if (n_doc > 0) FAILS(tr_kv_assemble(store, mine, offsets[q].data(), k, modes[q], ck, cv, n_doc - 1, nullptr), TR_ERR_BAD_PLAN);
        g_ex.src_rows = n_q;
        OK(tr_kv_append(&sh, knew, vnew, q_pos, n_q, ck, cv, n_doc, kv_len, nullptr));

        size_t wb = tr_prefill_attn_workspace_size(&sh, n_q, kv_len);
        g_ex.ws = (const char*)dev.get(wb);
        g_ex.ws_bytes = wb;
        OK(tr_prefill_attn(&sh, qd, ck, cv, q_pos, n_q, kv_len, od, (void*)g_ex.ws, wb, nullptr));

        if (sh.dtype == TR_BF16) {
            g_ex.src_rows = store_rows;
            wb = tr_prefill_attn_gather_workspace_size(store, mine, offsets[q].data(), k, modes[q], n_q);
            g_ex.ws = (const char*)dev.get(wb);
            g_ex.ws_bytes = wb;
            const int rc = tr_prefill_attn_gather(store, mine, offsets[q].data(), k, modes[q], qd, ck, cv, q_pos, n_q, kv_len, od, (void*)g_ex.ws, wb, nullptr);
            REQUIRE(rc == TR_OK || rc == TR_ERR_UNSUPPORTED, "tr_prefill_attn_gather returned %d: %s", rc, tr_last_error());
        }
    }
    {
        std::vector<int64_t> drs(n_req + 1, 0);
        for (int q = 0; q < n_req; ++q) drs[q + 1] = drs[q] + r.in(1, 5000);
        void* dk = dev.get(drs[n_req] * row_bytes);
        void* dv = dev.get(drs[n_req] * row_bytes);
        const size_t wb = tr_decode_attn_workspace_size(&sh, drs.data(), n_req);
        g_ex.ws = (const char*)dev.get(wb);
        g_ex.ws_bytes = wb;
        const int rc = tr_decode_attn(&sh, qd, dk, dv, q_pos, drs.data(), n_req, od, (void*)g_ex.ws, wb, nullptr);
        REQUIRE(rc == TR_OK || rc == TR_ERR_UNSUPPORTED, "tr_decode_attn returned %d: %s", rc, tr_last_error());
    }

    // offline chunk prefill and the one-pass sequence form
    {
        const int n_chunks = r.in(1, 20);
        std::vector<int32_t> lens(n_chunks);
        int64_t total = 0;
        int max_len = 0;
        for (auto& l : lens) {
            l = r.in(r.in(0, 5) ? 1 : 0, r.in(0, 4) ? 200 : 1500);
            total += l;
            max_len = l > max_len ? l : max_len;
        }
        void* q2 = dev.get(total * qrow_bytes);
        void* o2 = dev.get(total * qrow_bytes);
        void* k2 = dev.get(total * row_bytes);
        void* v2 = dev.get(total * row_bytes);
        void* kr = dev.get(total * row_bytes);
        const int32_t* cu_dev = (const int32_t*)dev.get((size_t)(n_chunks + 1) * 4);
        size_t wb = tr_chunk_prefill_attn_workspace_size(&sh, total, max_len);
        g_ex.ws = (const char*)dev.get(wb);
        g_ex.ws_bytes = wb;
        OK(tr_chunk_prefill_attn(&sh, q2, k2, v2, cu_dev, n_chunks, total, max_len, o2, kr, (void*)g_ex.ws, wb, nullptr));

        const int n_tail = r.in(0, 200), mode = r.in(0, 1);
        const int64_t T = total + n_tail;
        std::vector<int32_t> seg(T ? T : 1), pos(T ? T : 1);
        OK(tr_sequence_plan(lens.data(), n_chunks, n_tail, mode, -1, seg.data(), pos.data(), T));
        if (T > 0) FAILS(tr_sequence_plan(lens.data(), n_chunks, n_tail, mode, -1, seg.data(), pos.data(), T - 1), TR_ERR_BAD_PLAN);
        void* q3 = dev.get(T * qrow_bytes);
        void* o3 = dev.get(T * qrow_bytes);
        void* k3 = dev.get(T * row_bytes);
        void* v3 = dev.get(T * row_bytes);
        void* kr3 = dev.get(T * row_bytes);
        g_ex.src_rows = g_ex.dst_rows = T;   // the key rotation of this entry point goes through the append launcher
        for (int with_host = 0; with_host < 2; ++with_host) {
            const int32_t* host_seg = with_host ? seg.data() : nullptr;
            wb = tr_sequence_prefill_attn_workspace_size(&sh, host_seg, T);
            g_ex.ws = (const char*)dev.get(wb);
            g_ex.ws_bytes = wb;
            OK(tr_sequence_prefill_attn(&sh, q3, k3, v3, (const int32_t*)dev.get((size_t)(T ? T : 1) * 4), (const int32_t*)dev.get((size_t)(T ? T : 1) * 4), host_seg, T, o3,
                                        kr3, (void*)g_ex.ws, wb, nullptr));
        }
    }

    // linear layers of up to four weights
    {
        const int M = r.in(1, 128), K = 64 * r.in(1, 60), n_out = r.in(1, 4);
        int32_t nf[4];
        const void* w[4];
        void* y[4];
        for (int j = 0; j < n_out; ++j) {
            nf[j] = 64 * r.in(1, 60);
            w[j] = dev.get((size_t)nf[j] * K * 2);
            y[j] = dev.get((size_t)M * nf[j] * 2);
        }
        const size_t wb = tr_linear_workspace_size(M, n_out, nf, K);
        void* ws = dev.get(wb);
        g_ex.ws = (const char*)ws;
        g_ex.ws_bytes = wb;
        const int rc = tr_linear(dev.get((size_t)M * K * 2), M, K, n_out, w, y, nf, ws, wb, nullptr);
        REQUIRE(rc == TR_OK || rc == TR_ERR_SHAPE || rc == TR_ERR_UNSUPPORTED, "tr_linear returned %d: %s", rc, tr_last_error());
    }
    OK(tr_store_destroy(store));
}

void argument_errors()
{
    tr_shape sh;
    std::memset(&sh, 0, sizeof sh);
    sh.n_q_heads = 28; sh.n_kv_heads = 4; sh.head_dim = 128; sh.dtype = TR_BF16; sh.rope_base = 1e6;
    char buf[64];
    tr_store* st = nullptr;
    int64_t rs[3] = {0, 4, 2};
    FAILS(tr_store_create(&sh, buf, buf, rs, 2, &st), TR_ERR_INVALID_ARG);
    FAILS(tr_store_create(nullptr, buf, buf, rs, 2, &st), TR_ERR_INVALID_ARG);
    tr_shape bad = sh;
    bad.head_dim = 96;
    FAILS(tr_prefill_attn(&bad, buf, buf, buf, (const int32_t*)buf, 1, 1, buf, nullptr, 0, nullptr), TR_ERR_SHAPE);
    FAILS(tr_prefill_attn(&sh, nullptr, buf, buf, (const int32_t*)buf, 1, 1, buf, nullptr, 0, nullptr), TR_ERR_INVALID_ARG);
    FAILS(tr_set_tuning("no_such_knob", 1), TR_ERR_INVALID_ARG);
    FAILS(tr_set_tuning(nullptr, 1), TR_ERR_INVALID_ARG);
    double flops = 0;
    FAILS(tr_probe_mfma_loop(0, 0, (float*)buf, sizeof buf, &flops, nullptr), TR_ERR_INVALID_ARG);
    FAILS(tr_probe_mfma_loop(10, 0, (float*)buf, sizeof buf, &flops, nullptr), TR_ERR_INVALID_ARG);
    REQUIRE(tr_prefill_attn_static_scratch_bytes() > 0, "static scratch size");
}

// Decode batches that the plan cuts further than it takes to fill the chip run with less workspace than that cut asks for.
void decode_workspaces()
{
    tr_shape sh;
    std::memset(&sh, 0, sizeof sh);
    sh.n_q_heads = 32; sh.n_kv_heads = 8; sh.head_dim = g_ex.head_dim = 128; sh.dtype = TR_BF16; sh.rope_base = 5e5;
    Buffers dev;
    char buf[64];
    auto decode = [&](const std::vector<int64_t>& start, const void* ws, size_t bytes) {
        g_ex.ws = (const char*)ws;
        g_ex.ws_bytes = bytes;
        return tr_decode_attn(&sh, buf, buf, buf, (const int32_t*)buf, start.data(), (int32_t)start.size() - 1, buf, (void*)ws, bytes, nullptr);
    };
    std::vector<int64_t> full(1, 0), part(1, 0), two_launches(1, 0); // 320 pairs; 200; 320 and 200
    for (int i = 0; i < 40; ++i) full.push_back(full.back() + 140 * i + 5);
    int64_t cut_in_two = 0; // requests of `part` that are, where the cut only fills the chip
    for (int i = 0; i < 25; ++i) {
        const int64_t len = i ? 143 + 7 * i : 6500;
        part.push_back(part.back() + len);
        cut_in_two += len > 256;
    }
    for (int i = 0; i < 64; ++i) two_launches.push_back(two_launches.back() + (i < 40 ? 140 * i + 5 : 90));
    for (size_t i = 1; i < part.size(); ++i) two_launches.push_back(two_launches.back() + part[i] - part[i - 1]);
    const size_t rows = 2 * 32 * cut_in_two, least = (rows * 128 * 2 + 255) / 256 * 256 + (rows * 8 + 255) / 256 * 256;
    for (const auto* start : {&full, &part, &two_launches}) {
        const size_t need = tr_decode_attn_workspace_size(&sh, start->data(), (int32_t)start->size() - 1), lowest = start == &full ? 0 : least;
        char* ws = (char*)dev.get(need + 256);
        REQUIRE(need > lowest, "the even cut needs %zu bytes, this one %zu", lowest, need);
        for (size_t bytes : {need + 256, need, need - 1, lowest + 256, lowest}) OK(decode(*start, ws, bytes));
        const long before = g_ex.launches;
        if (lowest == 0) {
            OK(decode(*start, nullptr, 0));
            OK(decode(*start, nullptr, need));
            OK(decode(*start, ws + 16, need)); // not aligned: as none
            REQUIRE(g_ex.launches == before + 3, "%ld launches", g_ex.launches - before);
        } else {
            FAILS(decode(*start, ws, lowest - 1), TR_ERR_WORKSPACE);
            FAILS(decode(*start, ws, 0), TR_ERR_WORKSPACE);
            FAILS(decode(*start, nullptr, need), TR_ERR_WORKSPACE);
            FAILS(decode(*start, ws + 16, need), TR_ERR_WORKSPACE);
            REQUIRE(g_ex.launches == before, "a refused call launched something");
        }
    }
}

// Rows of keys too wide for the kernels' offsets are refused before anything is launched.
void wide_rows()
{
    tr_shape sh;
    std::memset(&sh, 0, sizeof sh);
    sh.head_dim = g_ex.head_dim = 128; sh.dtype = TR_BF16; sh.rope_base = 1e4;
    alignas(256) static char buf[1 << 16];
    const int32_t* i32 = (const int32_t*)buf;
    const int64_t start[] = {0, 40};
    for (int over = 0; over < 2; ++over) {
        const int rc = over ? TR_ERR_UNSUPPORTED : TR_OK;
        auto gives = [&](int got, const char* what) { REQUIRE(got == rc, "%s with %d heads returned %d", what, sh.n_kv_heads, got); };
        const long before = g_ex.launches;
        sh.n_q_heads = sh.n_kv_heads = (1 << 27) / 256 + over; // 32 rows of them are 4 GiB
        gives(tr_decode_attn(&sh, buf, buf, buf, i32, start, 1, buf, nullptr, 0, nullptr), "decode");
        gives(tr_prefill_attn(&sh, buf, buf, buf, i32, 32, 40, buf, nullptr, 0, nullptr), "short prefill");
        sh.n_q_heads = sh.n_kv_heads = (1 << 26) / 256 + over; // 64 rows
        gives(tr_prefill_attn(&sh, buf, buf, buf, i32, 33, 40, buf, nullptr, 0, nullptr), "prefill");
        g_ex.src_rows = g_ex.dst_rows = 40;
        g_ex.ws = buf;
        g_ex.ws_bytes = sizeof buf;
        gives(tr_sequence_prefill_attn(&sh, buf, buf, buf, i32, i32, nullptr, 40, buf, buf, nullptr, 0, nullptr), "sequence");
        REQUIRE(tr_chunk_prefill_attn_workspace_size(&sh, 40, 40) <= sizeof buf, "scratch of 40 tokens");
        gives(tr_chunk_prefill_attn(&sh, buf, buf, buf, i32, 1, 40, 40, buf, buf, buf, sizeof buf, nullptr), "chunks");
        const int64_t rows[] = {0, 32}, off[] = {0, 32};
        const int32_t id[] = {0};
        tr_store* st = nullptr;
        OK(tr_store_create(&sh, buf, buf, rows, 1, &st));
        gives(tr_prefill_attn_gather(st, id, off, 1, TR_POS_COMPOSITE, buf, buf, buf, i32, 8, 40, buf, nullptr, 0, nullptr), "gather");
        OK(tr_store_destroy(st));
        REQUIRE(over == 0 || g_ex.launches == before, "a refused call launched something");
    }
}

// More tokens than one launch holds: every row is covered once, in order, by launches of a legal size.
void appends_of_many_tokens()
{
    char buf[256];
    const int32_t* pos = (const int32_t*)buf;
    const int64_t MAX = TR_MAX_APPEND_TOKENS;
    for (int heads : {1, 40}) // one group of lanes per token, and twenty
    for (int64_t n : {MAX - 1, MAX, MAX + 1, 2 * MAX, 5 * MAX + 7, ((int64_t)1 << 31) - 1 - 1000}) {
        tr_shape sh;
        std::memset(&sh, 0, sizeof sh);
        sh.n_q_heads = sh.n_kv_heads = heads; sh.head_dim = heads == 1 ? 64 : 128; sh.dtype = heads == 1 ? TR_BF16 : TR_F32; sh.rope_base = 1e4;
        auto expect = [&](int64_t src, int64_t dst, int64_t pos0) {
            g_ex.next_src = src; g_ex.next_dst = dst; g_ex.next_pos = pos0;
        };
        g_ex.src_rows = n; g_ex.dst_rows = n + 1000;
        expect(0, 1000, -1);
        OK(tr_kv_append(&sh, buf, buf, pos, (int32_t)n, buf, buf, 1000, n + 1000, nullptr));
        REQUIRE(g_ex.next_dst == n + 1000, "%" PRId64 " of %" PRId64 " tokens appended", g_ex.next_dst - 1000, n);
        // two requests: the second one begins in the middle of a launch
        const int32_t cu[] = {0, 100, (int32_t)n};
        const int64_t start[] = {0, 100, n};
        expect(0, 0, -1);
        OK(tr_kv_append_batched(&sh, buf, buf, pos, cu, start, 2, buf, buf, n, nullptr));
        REQUIRE(g_ex.next_dst == n, "%" PRId64 " of %" PRId64 " tokens appended", g_ex.next_dst, n);
        // a store of un-rotated keys, both position schemes
        const int64_t rows[] = {0, 100, n};
        tr_store* st = nullptr;
        OK(tr_store_create(&sh, buf, buf, rows, 2, &st));
        const int32_t ids[] = {0, 1}, last[] = {1};
        const int64_t off1[] = {0, n - 100};
        expect(0, 0, 0);
        OK(tr_kv_assemble_raw(st, ids, rows, 2, TR_POS_REORDERED, buf, buf, n, nullptr));
        REQUIRE(g_ex.next_dst == n && g_ex.next_pos == n, "%" PRId64 " of %" PRId64 " rows assembled", g_ex.next_dst, n);
        expect(100, 0, 0);
        OK(tr_kv_assemble_raw(st, last, off1, 1, TR_POS_COMPOSITE, buf, buf, n, nullptr));
        REQUIRE(g_ex.next_dst == n - 100, "%" PRId64 " of %" PRId64 " rows assembled", g_ex.next_dst, n - 100);
        // documents, and the tokens behind them in the same launch or in their own
        const int64_t off2[] = {0, 100};
        expect(0, 100, -1);
        OK(tr_kv_assemble_append(st, ids, off2, 1, TR_POS_REORDERED, buf, buf, pos, (int32_t)n, buf, buf, n + 1000, nullptr));
        REQUIRE(g_ex.next_dst == n + 100, "%" PRId64 " of %" PRId64 " tokens appended", g_ex.next_dst - 100, n);
        OK(tr_store_destroy(st));
    }
    g_ex.next_src = g_ex.next_pos = -1;
}

}  // namespace

int main(int argc, char** argv)
{
    const int rounds = argc > 1 ? std::atoi(argv[1]) : 300;
    argument_errors();
    appends_of_many_tokens();
    decode_workspaces();
    wide_rows();
    const char* knobs[] = {"wg_rows", "target_items", "min_split_keys", "bd_piece_tiles"};
    const int values[][3] = {{0, 128, 32}, {0, 64, 2048}, {0, 64, 1024}, {0, 1, 8}};
    for (int i = 0; i < rounds; ++i) {
        if (i % 25 == 0)   // the launch policy under a few overrides as well
            for (int kn = 0; kn < 4; ++kn) OK(tr_set_tuning(knobs[kn], values[kn][(i / 25 + kn) % 3]));
        one_request_mix(1000 + i);
    }
    std::printf("host abi sanitizer run ok: %d request mixes, %ld launches stood in for, %ld checks\n", rounds, g_ex.launches, g_checks);
    return 0;
}
