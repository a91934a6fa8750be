// Driver for tests/test_host_dispatch.py: the kernels' host side (which variant a call takes, its grid) compiled for the CPU alone and
// linked with the stand-ins below in place of the HIP runtime.  A launch is checked, not made.  For calls over all storage types, sizes
// and head counts it holds what the dispatcher relies on: a call that a rule says a channel-planar (or one-launch) kernel takes is taken.
#include <hip/hip_runtime.h>

#include <cstdio>

#include "../paper_2205_14756_amd/csrc/msla_kernels.h"

static long g_launches = 0, g_failures = 0;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
static dim3 g_grid, g_block;
static size_t g_lds;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    g_grid = grid, g_block = block, g_lds = lds, g_stream = stream;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = g_grid, *block = g_block, *lds = g_lds, *stream = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
    ++g_launches;
    const unsigned long threads = (unsigned long)grid.x * block.x;
    if (grid.x == 0 || block.x == 0 || block.x > 1024 || threads > 0xffffffffUL || lds > 160 * 1024) {
        std::fprintf(stderr, "a launch of %u x %u threads, %zu bytes of LDS\n", grid.x, block.x, lds);
        ++g_failures;
    }
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace msla {
int compute_units() { return 256; }
}

int main() {
    char x[64];
    long planar_x = 0, planar_out = 0, tokens_first = 0, one_launch = 0;
    const int sides[][2] = {{1, 1}, {1, 3}, {7, 7}, {17, 19}, {53, 67}, {64, 128}, {131, 133}, {256, 256}};
    for (int dt = 0; dt < 3; ++dt)
        for (int C = 16; C <= 528; C += 16)
            for (const auto& hw : sides)
                for (int B : {1, 3, 16, 400}) {
                    const int N = hw[0] * hw[1];
                    const long T = (long)B * N;
                    if (T > (1L << 21)) continue;
                    for (int heads : {1, C / 16, 21, 32, 40}) {
                        const bool in = msla::qkv_project_takes_planar(dt, T, C, heads, N);
                        if (in && msla::launch_qkv_project(dt, x, x, x, heads * 16, x, heads * 32, 32, T * heads * 32, T, C, heads, nullptr, N) != hipSuccess) {
                            std::fprintf(stderr, "type %d, %d x %d tokens, %d channels, %d heads: a planar x is refused\n", dt, B, N, C, heads);
                            ++g_failures;
                        }
                        planar_x += in;
                        for (int S = 1; S <= 3; ++S) {
                            const bool out = msla::apply_project_writes_planar(dt, T, N, S * heads, C);
                            if (msla::launch_apply_project(dt, x, x, (const float*)x, x, x, nullptr, T, N, S * heads, C, 1e-15f, nullptr, out) != hipSuccess) {
                                std::fprintf(stderr, "type %d, %d x %d tokens, %d channels, %d head-branches: planar %d is refused\n", dt, B, N, C, S * heads, out);
                                ++g_failures;
                            }
                            planar_out += out;
                            tokens_first += !out;
                        }
                    }
                    for (int E : {16, 80, C, 4 * C}) {
                        const int rows = msla::ffn_block_rows(dt, B, C, hw[0], hw[1], E);
                        const hipError_t e = msla::launch_ffn_fused(dt, x, x, x, x, x, B, C, hw[0], hw[1], E, 1, nullptr);
                        if (e != (rows ? hipSuccess : hipErrorNotSupported)) {
                            std::fprintf(stderr, "type %d, %d x %d x %d tokens, %d -> %d channels: one launch in %d rows: %d\n", dt, B, hw[0], hw[1], C, E, rows, (int)e);
                            ++g_failures;
                        }
                        one_launch += rows != 0;
                    }
                }
    if (!planar_x || !planar_out || !tokens_first || !one_launch) {
        std::fprintf(stderr, "a kind of call was not reached: %ld %ld %ld %ld\n", planar_x, planar_out, tokens_first, one_launch);
        ++g_failures;
    }
    if (g_failures) return 1;
    std::printf("host dispatch ok: %ld launches, %ld planar x, %ld planar out, %ld FFNs in one launch\n", g_launches, planar_x, planar_out, one_launch);
    return 0;
}
