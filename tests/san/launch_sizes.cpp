// The launches of calls with very many rows, on the CPU: this program defines the runtime's launch entry points itself, so the
// built library's launches end here and only their sizes are looked at.  A launch has fewer than 2^32 threads.
// Argument: path of libturborag_hip.so.  Exit status 0 and "launch sizes ok" on stdout mean every launch was legal and the
// workgroups of each call add up, also where a rule chooses between two divisions of the work.
#include <dlfcn.h>
#include <initializer_list>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../../include/turborag.h"

struct Dim3 {
    uint32_t x, y, z;
};
static uint64_t blocks, largest;
static uint32_t block_threads, n_blocks; // of the last launch

static Dim3 next_grid, next_block;
extern "C" unsigned __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t, void*)
{
    next_grid = grid;
    next_block = block;
    return 0;
}
extern "C" int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream)
{
    *grid = next_grid;
    *block = next_block;
    *lds = 0;
    *stream = nullptr;
    return 0;
}
extern "C" int hipLaunchKernel(const void*, Dim3 grid, Dim3 block, void**, size_t, void*)
{
    const uint64_t n = (uint64_t)grid.x * grid.y * grid.z, threads = n * block.x * block.y * block.z;
    blocks += n;
    block_threads = block.x;
    n_blocks = grid.x;
    if (threads > largest) largest = threads;
    return 0;
}
extern "C" int hipGetLastError(void) { return 0; }
extern "C" int hipGetDevice(int* d)
{
    *d = 0;
    return 0;
}
extern "C" int hipFuncSetAttribute(const void*, int, int) { return 0; }

static void* lib;
static void* entry(const char* name)
{
    void* p = dlsym(lib, name);
    if (!p) {
        fprintf(stderr, "%s\n", dlerror());
        exit(1);
    }
    return p;
}
#define CALL(name) ((decltype(&name))entry(#name))

static void check(const char* what, int64_t n, int rc, uint64_t want_blocks)
{
    if (rc != TR_OK || blocks != want_blocks || largest >= (uint64_t)1 << 32) {
        fprintf(stderr, "%s of %lld: status %d, %llu workgroups (expected %llu), largest launch %llu threads\n", what, (long long)n, rc,
                (unsigned long long)blocks, (unsigned long long)want_blocks, (unsigned long long)largest);
        exit(1);
    }
    blocks = largest = 0;
}

// A group of head_dim / 2 lanes owns up to twice as many units of a token's row, a workgroup has 256 lanes; many tokens whose
// rows leave half of a group idle share lanes instead.
static void appends()
{
    static char buf[4096] __attribute__((aligned(256)));
    const struct {
        int dtype, heads, head_dim, tokens, lanes; // lanes per token
    } cases[] = {
        {TR_BF16, 1, 64, 64, 32},      {TR_BF16, 1, 64, 8191, 32},    {TR_BF16, 1, 64, 8192, 8},      {TR_BF16, 2, 64, 16383, 32},
        {TR_BF16, 2, 64, 16384, 8},    {TR_BF16, 3, 64, 1 << 20, 32}, {TR_BF16, 8, 64, 100, 32},      {TR_BF16, 9, 64, 1001, 64},
        {TR_BF16, 17, 64, 1001, 96},   {TR_BF16, 1, 128, 4095, 64},   {TR_BF16, 1, 128, 4097, 16},    {TR_BF16, 2, 128, 8191, 64},
        {TR_BF16, 2, 128, 8192, 16},   {TR_BF16, 3, 128, 1 << 20, 64}, {TR_BF16, 8, 128, 1 << 20, 64}, {TR_BF16, 9, 128, 77, 128},
        {TR_F32, 1, 64, 8191, 32},     {TR_F32, 1, 64, 8193, 16},     {TR_F32, 2, 64, 1 << 20, 32},   {TR_F32, 5, 64, 3, 64},
        {TR_F32, 1, 128, 1 << 20, 64}, {TR_F32, 40, 128, 1000, 640},
    };
    for (const auto& c : cases) {
        tr_shape s;
        memset(&s, 0, sizeof s);
        s.n_q_heads = s.n_kv_heads = c.heads;
        s.head_dim = c.head_dim;
        s.rope_base = 1e4;
        s.dtype = c.dtype;
        for (int half : {0, 1}) {
            s.rope_layout = half ? TR_ROPE_HALF : TR_ROPE_INTERLEAVED;
            check("append", c.tokens, CALL(tr_kv_append)(&s, buf, buf, (const int32_t*)buf, c.tokens, buf, buf, 0, c.tokens, nullptr),
                  ((uint64_t)c.tokens * c.lanes + 255) / 256);
        }
    }
}

// fp32 attention: waves per row by the number of rows, the keys a row sees and how many turns the rows take on the chip.
static void fp32_waves()
{
    static char buf[4096] __attribute__((aligned(256)));
    const int32_t* idx = (const int32_t*)buf;
    const struct {
        int heads, head_dim, n_q, kv_len, waves;
    } prefill[] = {
        {4, 64, 1, 12, 1},     {4, 64, 1, 20, 2},      {4, 64, 1, 40, 4},      {4, 64, 1, 130, 8},     {4, 64, 16, 144, 8},   {4, 128, 1, 6, 1},
        {4, 128, 1, 10, 2},    {4, 128, 1, 20, 4},     {4, 128, 1, 70, 8},     {8, 128, 16, 17, 4},    {8, 128, 200, 201, 4}, {32, 64, 16, 24, 2},
        {32, 64, 16, 36, 4},   {32, 64, 16, 100, 8},   {32, 64, 28, 100, 4},   {32, 64, 32, 2000, 4},  {32, 64, 56, 100, 2},  {32, 64, 64, 800, 2},
        {32, 128, 64, 400, 2}, {32, 64, 96, 600, 4},   {32, 64, 112, 600, 1},  {32, 64, 250, 500, 1},  {32, 128, 128, 300, 2}, {32, 64, 1024, 1100, 1},
    };
    for (const auto& c : prefill) {
        tr_shape s;
        memset(&s, 0, sizeof s);
        s.n_q_heads = s.n_kv_heads = c.heads;
        s.head_dim = c.head_dim;
        s.rope_base = 1e4;
        s.dtype = TR_F32;
        check("fp32 rows", c.n_q, CALL(tr_prefill_attn)(&s, buf, buf, buf, idx, c.n_q, c.kv_len, buf, nullptr, 0, nullptr), (uint64_t)c.n_q * c.heads);
        if (block_threads != 64u * c.waves) {
            fprintf(stderr, "fp32 prefill of %d x %d rows of %d over %d keys: %u threads a row, expected %d waves\n", c.n_q, c.heads, c.head_dim, c.kv_len, block_threads, c.waves);
            exit(1);
        }
    }
    const struct {
        int head_dim, chunk, n_chunks, waves;
    } offline[] = {{64, 32, 16, 2}, {64, 512, 1, 4}, {64, 64, 64, 1}, {64, 512, 8, 1}, {64, 24, 200, 1}, {128, 32, 8, 4}, {128, 100, 1, 8}};
    for (const auto& c : offline) {
        tr_shape s;
        memset(&s, 0, sizeof s);
        s.n_q_heads = 4;
        s.n_kv_heads = 2;
        s.head_dim = c.head_dim;
        s.rope_base = 1e4;
        s.dtype = TR_F32;
        const int64_t total = (int64_t)c.chunk * c.n_chunks;
        const int rc = CALL(tr_chunk_prefill_attn)(&s, buf, buf, buf, idx, c.n_chunks, total, c.chunk, buf, buf, buf, (size_t)1 << 30, nullptr);
        if (rc != TR_OK || block_threads != 64u * c.waves) {
            fprintf(stderr, "fp32 chunks, %d x %d of %d: status %d, %u threads a row, expected %d waves\n", c.n_chunks, c.chunk, c.head_dim, rc, block_threads, c.waves);
            exit(1);
        }
        blocks = largest = 0;
    }
}

// Merge of split keys: a wave per row for more than eight splits of few rows, D/8 lanes per row otherwise (two waves to a
// workgroup).
static void merges()
{
    static char buf[4096] __attribute__((aligned(256)));
    const int32_t* idx = (const int32_t*)buf;
    const struct {
        int heads, head_dim, n_q, kv_len, splits, rows_per_block;
    } cases[] = {
        {2, 128, 16, 256 * 64, 64, 2},    {2, 128, 16, 256 * 9, 9, 2},      {2, 128, 16, 256 * 8, 8, 8},      {2, 64, 16, 256 * 64, 64, 2},
        {2, 64, 16, 256 * 9, 9, 2},       {2, 64, 16, 256 * 8, 8, 16},      {2, 128, 512, 256 * 16, 16, 2},   {2, 128, 513, 256 * 16, 16, 8},
        {2, 64, 513, 256 * 16, 16, 16},   {2, 128, 513, 256 * 17, 17, 2},   {2, 128, 1024, 256 * 20, 20, 2},  {2, 128, 1025, 256 * 20, 20, 8},
        {2, 64, 1025, 256 * 20, 20, 16},
    };
    for (const auto& c : cases) {
        tr_shape s;
        memset(&s, 0, sizeof s);
        s.n_q_heads = c.heads;
        s.n_kv_heads = 1;
        s.head_dim = c.head_dim;
        s.rope_base = 1e4;
        s.dtype = TR_BF16;
        const size_t ws = CALL(tr_prefill_attn_workspace_size)(&s, c.n_q, c.kv_len), row = 2 * (size_t)c.head_dim + 8;
        const uint32_t rows = (uint32_t)(c.n_q * c.heads), want = (rows + c.rows_per_block - 1) / c.rows_per_block;
        const int rc = CALL(tr_prefill_attn)(&s, buf, buf, buf, idx, c.n_q, c.kv_len, buf, buf, ws, nullptr);
        if (rc != TR_OK || ws / row / rows != (size_t)c.splits || n_blocks != want) {
            fprintf(stderr, "merge of %zu splits (expected %d) of %u rows of %d: status %d, %u workgroups, expected %u\n", ws / row / rows, c.splits, rows, c.head_dim, rc, n_blocks, want);
            exit(1);
        }
    }
    blocks = largest = 0;
}

int main(int, char** argv)
{
    lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) {
        fprintf(stderr, "%s\n", dlerror());
        return 1;
    }
    static char buf[4096] __attribute__((aligned(256)));
    const int32_t* idx = (const int32_t*)buf;
    tr_shape s;
    memset(&s, 0, sizeof s);
    s.n_q_heads = s.n_kv_heads = 1;
    s.rope_base = 1e4;
    s.dtype = TR_F32;
    for (int d : {64, 128})
        for (int64_t n : {((int64_t)1 << 25) - 1, (int64_t)1 << 25, ((int64_t)1 << 26) - 1, ((int64_t)1 << 28) + 3}) {
            s.head_dim = d;
            check("fp32 prefill", n, CALL(tr_prefill_attn)(&s, buf, buf, buf, idx, (int32_t)n, n, buf, nullptr, 0, nullptr), (uint64_t)n);
            // one pass over packed segments: the keys are turned, at a head size of 64 by 16 lanes per token and at one of 128
            // by 64, then the attention
            const int64_t tokens = d == 64 ? 16 : 4;
            check("fp32 sequence", n, CALL(tr_sequence_prefill_attn)(&s, buf, buf, buf, idx, idx, nullptr, n, buf, buf, nullptr, 0, nullptr),
                  (uint64_t)n + (uint64_t)((n + tokens - 1) / tokens));
        }
    appends();
    fp32_waves();
    merges();
    puts("launch sizes ok");
    return 0;
}
