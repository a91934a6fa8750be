// Layout change between the channel-planar form [B, C, H, W] and the token-major
// form [B, H, W, C] that the module's kernels work on (Section 3.1 writes the
// input as x in R^{N x f}: one row of f channels per token).  A batched 2-D
// transposition  dst[b][c][r] = src[b][r][c]  through a padded LDS tile, so that
// both the loads and the stores run along the contiguous axis of their side.
#include "msla_device.h"
#include "msla_kernels.h"

namespace msla {
namespace {

constexpr int kTile = 64;

// What bounds it is latency: a tile is one round of loads, all requested at once (a loop of guarded loads paid four
// rounds), one barrier and one round of stores, 16 bytes a lane on every side whose rows allow it.  VS and VD are the
// elements a lane moves at a time on the source and the destination side; a row of cols (rows) elements has to be a
// multiple of VS (VD) elements, and 16-byte aligned with them: the token side (C channels, a multiple of 16) always is, the
// channel-planar side only where H*W is.  Loads past the ends read the last row or column instead; stores are guarded.
// Modules with planar x and out, both transpositions: 3 x 192 x 1961 bf16 70.1 -> 61.6 us, 8 x 256 x 8192 fp16 164 ->
// 144, 12 x 112 x 924 fp32 94.0 -> 85.3.
template <class T, int VS, int VD>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ src, T* __restrict__ dst, int rows,
                                                        int cols, int tiles_r, int tiles_c) {
    // pitch: 33 (66) words, so that a lane's VD rows and eight lanes' columns fall on different banks
    __shared__ __attribute__((aligned(16))) T tile[kTile][kTile + 2];
    struct __attribute__((aligned(VS * sizeof(T)))) SVec { T e[VS]; };
    struct __attribute__((aligned(VD * sizeof(T)))) DVec { T e[VD]; };
    const unsigned bid = blockIdx.x;
    const int tc = bid % tiles_c;
    const int tr = (bid / tiles_c) % tiles_r;
    const long b = bid / ((unsigned)tiles_c * tiles_r);
    const int r0 = tr * kTile, c0 = tc * kTile;
    const T* s = src + b * (long)rows * cols;
    T* d = dst + b * (long)rows * cols;
    constexpr int kSRow = kTile / VS, kSPer = kTile * kSRow / 256;      // vectors per tile row, per thread
    SVec v[kSPer];
#pragma unroll
    for (int i = 0; i < kSPer; ++i) {
        const int id = i * 256 + threadIdx.x, r = r0 + id / kSRow, c = c0 + (id % kSRow) * VS;
        v[i] = *(const SVec*)(s + (long)(r < rows ? r : rows - 1) * cols + (c < cols ? c : cols - VS));
    }
#pragma unroll
    for (int i = 0; i < kSPer; ++i) {
        const int id = i * 256 + threadIdx.x;
        __builtin_memcpy(&tile[id / kSRow][(id % kSRow) * VS], &v[i], sizeof(SVec));
    }
    __syncthreads();
    constexpr int kDRow = kTile / VD, kDPer = kTile * kDRow / 256;
#pragma unroll
    for (int i = 0; i < kDPer; ++i) {
        const int id = i * 256 + threadIdx.x, c = id / kDRow, r = (id % kDRow) * VD;
        DVec o;
#pragma unroll
        for (int j = 0; j < VD; ++j) o.e[j] = tile[r + j][c];
        if (c0 + c < cols && r0 + r < rows) *(DVec*)(d + (long)(c0 + c) * rows + r0 + r) = o;
    }
}

template <class T, int VS, int VD>
hipError_t run_transpose_v(const void* src, void* dst, long batch, int rows, int cols, hipStream_t stream) {
    const int tiles_r = (rows + kTile - 1) / kTile, tiles_c = (cols + kTile - 1) / kTile;
    const long nblocks = batch * tiles_r * tiles_c;
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((transpose_kernel<T, VS, VD>), dim3((unsigned)nblocks), dim3(256), 0, stream, (const T*)src, (T*)dst,
                       rows, cols, tiles_r, tiles_c);
    return hipGetLastError();
}

// the widest vectors that both sides' rows are whole multiples of (the buffers are 16-byte aligned)
template <class T>
hipError_t run_transpose(const void* src, void* dst, long batch, int rows, int cols, hipStream_t stream) {
    constexpr int V = 16 / (int)sizeof(T);
    const bool wide_s = cols % V == 0, wide_d = rows % V == 0;
    if (wide_s && wide_d) return run_transpose_v<T, V, V>(src, dst, batch, rows, cols, stream);
    if (wide_s) return run_transpose_v<T, V, 1>(src, dst, batch, rows, cols, stream);
    if (wide_d) return run_transpose_v<T, 1, V>(src, dst, batch, rows, cols, stream);
    return run_transpose_v<T, 1, 1>(src, dst, batch, rows, cols, stream);
}

}  // namespace

hipError_t launch_transpose(int dt, const void* src, void* dst, long batch, int rows, int cols,
                            hipStream_t stream) {
    switch (dt) {
        case 0: return run_transpose<float>(src, dst, batch, rows, cols, stream);
        case 1:
        case 2: return run_transpose<unsigned short>(src, dst, batch, rows, cols, stream);   // a pure move
    }
    return hipErrorInvalidValue;
}

}  // namespace msla
