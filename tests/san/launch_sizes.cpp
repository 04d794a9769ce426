// The launches of calls with very many rows, on the CPU: this program defines the runtime's launch entry points itself, so the
// built library's launches end here and only their sizes are looked at.  A launch has fewer than 2^32 threads.
// Argument: path of libturborag_hip.so.  Exit status 0 and "launch sizes ok" on stdout mean every launch was legal and the
// workgroups of each call add up.
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
template <class F> F* entry(F*, const char* name)
{
    void* p = dlsym(lib, name);
    if (!p) {
        fprintf(stderr, "%s\n", dlerror());
        exit(1);
    }
    return (F*)p;
}
#define CALL(name) entry(&name, #name)

static void check(const char* what, int64_t n, int rc, uint64_t want_blocks)
{
    if (rc != TR_OK || blocks != want_blocks || largest >= (uint64_t)1 << 32) {
        fprintf(stderr, "%s of %lld: status %d, %llu workgroups (expected %llu), largest launch %llu threads\n", what, (long long)n, rc,
                (unsigned long long)blocks, (unsigned long long)want_blocks, (unsigned long long)largest);
        exit(1);
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
            // one pass over packed segments: a wave per token turns the keys (four to a workgroup), then the attention
            check("fp32 sequence", n, CALL(tr_sequence_prefill_attn)(&s, buf, buf, buf, idx, idx, nullptr, n, buf, buf, nullptr, 0, nullptr),
                  (uint64_t)n + (uint64_t)(n + 3) / 4);
        }
    puts("launch sizes ok");
    return 0;
}
