// Launches of the walks on a device of a chosen size, without a GPU: the HIP
// calls that the library makes on its way to a launch are answered here (the
// executable's definitions come before the runtime's), and the launches are
// printed instead of made.
//
// usage: ref <compute units> <V> <R> <D> <rrs|traversal>
// prints one line: workgroups a request, tokens of a slice, whether a slice is
// held in LDS, dynamic LDS bytes, LDS bytes of a held slice.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include <hip/hip_runtime.h>

#include "../paper_2609_33652_amd/csrc/tsb_internal.hpp"

static int g_cus = 256;
static dim3 g_grid, g_block;
static size_t g_shared;

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = g_cus, hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
// 160 KB of LDS a compute unit, 2048 threads
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t lds) {
    const int by_lds = lds ? (int)((160u << 10) / lds) : 64;
    return *n = by_lds < 2048 / threads ? by_lds : 2048 / threads, hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t) {
    g_grid = grid;
    g_block = block;
    g_shared = shared;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* st) {
    *grid = g_grid;
    *block = g_block;
    *shared = g_shared;
    *st = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t shared, hipStream_t) {
    g_grid = grid;  // the last launch of a call is its walk
    g_block = block;
    g_shared = shared;
    return hipSuccess;
}
}

int main(int argc, char** argv) {
    if (argc != 6) return 2;
    g_cus = atoi(argv[1]);
    tsb_config c{};
    c.V = atoi(argv[2]);
    c.R = atoi(argv[3]);
    c.D = atoi(argv[4]);
    c.B = 4;
    c.K = 2;
    c.temperature = 1.0f;
    c.dtype = TSB_BF16;
    void* const p = (void*)0x100000;  // never dereferenced
    tsb_tree t;
    tsb_verdict o;
    memset(&t, 1, sizeof t);
    memset(&o, 1, sizeof o);
    const bool trav = !strcmp(argv[5], "traversal");
    auto* fn = trav ? tsb_verify_traversal : tsb_verify;
    const tsb_status s = fn(&c, p, (const double*)p, p, &t, (const int32_t*)p, 0u, &o, p, tsb_workspace_bytes(&c), nullptr);
    if (s != TSB_OK) {
        printf("error %d %s\n", (int)s, tsb_last_error());
        return 1;
    }
    if (g_block.x != (unsigned)tsb::kWalkThreadsPerGroup || g_grid.x % c.R) return 3;
    const int G = (int)g_grid.x / c.R, span = tsb::walk_span(c.V, G);
    const bool held = span <= tsb::kWalkHeldTokens;
    printf("%d %d %d %zu %zu\n", G, span, held ? 1 : 0, g_shared, held ? (size_t)span * 2 * sizeof(double) : 0);
    return 0;
}
