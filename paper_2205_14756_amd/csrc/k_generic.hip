// The module for head sizes other than 16 (Section 3.1 fixes only "d channels per group"; 8 and 32 are
// the other sizes the architecture family uses).
//
// Head size 32.  fp32 storage: multi-scale aggregation and the Eq. (3) state as plain vector-ALU kernels
// templated on the head size D, following the definitions step by step with fp32 sums throughout (16-bit
// storage takes the tiled matrix-core kernel of k_aggregate32.hip instead); all types: the fixed-order sum of
// the partial states and the normalise-and-apply pass below.  The same storage points as the head-size-16
// path: projected Q/K/V and the Q tokens of every branch are stored in the storage type; aggregated K and V
// only feed the state.
//
//   generic_branch_state_kernel   one branch (raw, or depthwise k x k + grouped 1x1) of one (image, head,
//                                 chunk of 64-token groups): writes that branch's Q tokens, accumulates
//                                 KV = sum_n relu(K_n)^T [V_n, 1] into a per-workgroup partial state
//   generic_state_finalize_kernel fixed-order sum of the partial states
//   generic_apply_kernel          att_n = relu(Q_n) KV[:, :D] / (relu(Q_n) KV[:, D] + eps), on the matrix cores in fp32
//
// Head size 8 needs no kernels of its own: two heads side by side are one head of 16 whose grouped 1x1 is
// block-diagonal and whose state is used block by block (pair_head8_weights_kernel arranges the weights
// that way; the finalize step of the head-size-16 path masks the state operands).
#include <algorithm>
#include <type_traits>

#include "msla_device.h"
#include "msla_kernels.h"

namespace msla {
namespace {

constexpr int kGenThreads = 256;
constexpr int kGenTokens = 64;       // tokens per step of a workgroup

template <class T, int D>
__global__ __launch_bounds__(kGenThreads) void generic_branch_state_kernel(
    const T* __restrict__ qkv, const T* __restrict__ w_dw, const T* __restrict__ w_gpw, T* __restrict__ q_ms,
    float* __restrict__ partials, int H, int W, int heads, int S, int branch, int ks, int nchunks, int groups_per_chunk) {
    constexpr int kState = D * (D + 1);
    constexpr int kAcc = (kState + kGenThreads - 1) / kGenThreads;
    __shared__ float dw[kGenTokens][3 * D];       // depthwise sums (or, raw branch, the tokens themselves)
    __shared__ float rk[kGenTokens][D];           // rectified K of the branch
    __shared__ float vv[kGenTokens][D];           // V of the branch
    const int h = blockIdx.x % heads;
    const int chunk = (blockIdx.x / heads) % nchunks;
    const int b = blockIdx.x / (heads * nchunks);
    const int N = H * W;
    const int Ct = heads * D;
    const long ts = 3L * Ct;                                   // elements from token to token of qkv
    const T* img = qkv + (long)b * N * ts + (long)h * 3 * D;   // this head's 3*D channels of token 0
    const int P = (ks - 1) / 2;
    const T* wd = w_dw + (long)h * 3 * D * ks * ks;            // [3*D][ks][ks] of this head
    const T* wg = w_gpw + (long)h * 3 * D * D;                 // [3*D][D] of this head

    float acc[kAcc];
#pragma unroll
    for (int i = 0; i < kAcc; ++i) acc[i] = 0.f;

    const int n_groups = (N + kGenTokens - 1) / kGenTokens;
    const int g_begin = chunk * groups_per_chunk;
    const int g_end = g_begin + groups_per_chunk < n_groups ? g_begin + groups_per_chunk : n_groups;
    for (int g = g_begin; g < g_end; ++g) {
        const int n0 = g * kGenTokens;
        // ---- A: depthwise k x k sums of the group's tokens (zero padding), or the raw tokens
        for (int it = threadIdx.x; it < kGenTokens * 3 * D; it += kGenThreads) {
            const int tk = it / (3 * D), c = it - tk * (3 * D);
            const int n = n0 + tk;
            float s = 0.f;
            if (n < N) {
                if (ks == 0) {
                    s = Traits<T>::to_f32(img[(long)n * ts + c]);
                } else {
                    const int y = n / W, x = n - y * W;
                    for (int u = 0; u < ks; ++u) {
                        const int yy = y + u - P;
                        if (yy < 0 || yy >= H) continue;
                        for (int v = 0; v < ks; ++v) {
                            const int xx = x + v - P;
                            if (xx < 0 || xx >= W) continue;
                            s = fmaf(Traits<T>::to_f32(wd[(c * ks + u) * ks + v]),
                                     Traits<T>::to_f32(img[((long)yy * W + xx) * ts + c]), s);
                        }
                    }
                }
            }
            dw[tk][c] = s;
        }
        __syncthreads();
        // ---- B: grouped 1x1 (D -> D inside each of Q, K, V); Q is stored, relu(K) and V go on to the state
        for (int it = threadIdx.x; it < kGenTokens * 3 * D; it += kGenThreads) {
            const int tk = it / (3 * D), c = it - tk * (3 * D);
            const int t = c / D, o = c - t * D;
            const int n = n0 + tk;
            float s;
            if (ks == 0) {
                s = dw[tk][c];
            } else {
                s = 0.f;
#pragma unroll 8
                for (int e = 0; e < D; ++e) s = fmaf(Traits<T>::to_f32(wg[(long)c * D + e]), dw[tk][t * D + e], s);
            }
            if (t == 0) {
                if (n < N) q_ms[((long)b * N + n) * ((long)S * Ct) + (long)(branch * heads + h) * D + o] = Traits<T>::from_f32(s);
            } else if (t == 1) {
                rk[tk][o] = n < N ? fmaxf(s, 0.f) : 0.f;       // Eq. (2); tokens past the image contribute nothing
            } else {
                vv[tk][o] = s;
            }
        }
        __syncthreads();
        // ---- C: KV[e][f] += sum_n relu(K_n[e]) * (f < D ? V_n[f] : 1)
#pragma unroll
        for (int i = 0; i < kAcc; ++i) {
            const int idx = threadIdx.x + i * kGenThreads;
            if (idx < kState) {
                const int e = idx / (D + 1), f = idx - e * (D + 1);
                float s = acc[i];
                if (f < D) {
                    for (int tk = 0; tk < kGenTokens; ++tk) s = fmaf(rk[tk][e], vv[tk][f], s);
                } else {
                    for (int tk = 0; tk < kGenTokens; ++tk) s += rk[tk][e];
                }
                acc[i] = s;
            }
        }
        __syncthreads();
    }
    float* out = partials + ((((long)b * S + branch) * heads + h) * nchunks + chunk) * kState;
#pragma unroll
    for (int i = 0; i < kAcc; ++i) {
        const int idx = threadIdx.x + i * kGenThreads;
        if (idx < kState) out[idx] = acc[i];
    }
}

// Fixed-order sum of the partial states: 64 entries of one state a workgroup, its four waves a quarter of the chunks each,
// 16 loads in flight a wave.  Few heads mean many chunks, and one workgroup a state then waited for one load latency per
// eight chunks and 256 entries (a module of 3 heads, 135 x 111 tokens, two scales: 171 chunks for each of 9 states, 123.7 ->
// 71.4 us).
constexpr int kFinEntries = 64;
template <int D>
__global__ __launch_bounds__(kGenThreads) void generic_state_finalize_kernel(const float* __restrict__ partials,
                                                                             float* __restrict__ kv32, int nchunks) {
    static_assert(kGenThreads == 4 * kFinEntries, "a wave is the 64 entries, the waves are the quarters");
    constexpr int kState = D * (D + 1), kParts = (kState + kFinEntries - 1) / kFinEntries;
    __shared__ float quarter[4][kFinEntries];
    const long sid = blockIdx.x / kParts;
    const int e = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = (int)(blockIdx.x % kParts) * kFinEntries + e;
    const float* p = partials + sid * nchunks * kState + (j < kState ? j : kState - 1);
    const int c_begin = (int)((long)nchunks * w / 4), c_end = (int)((long)nchunks * (w + 1) / 4);
    float v = 0.f;
    for (int c0 = c_begin; c0 < c_end; c0 += 16) {
        float part[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) part[i] = p[(long)(c0 + i < c_end ? c0 + i : c_end - 1) * kState];
#pragma unroll
        for (int i = 0; i < 16; ++i) v += c0 + i < c_end ? part[i] : 0.f;
    }
    quarter[w][e] = v;
    __syncthreads();
    if (w == 0 && j < kState) kv32[sid * kState + j] = (quarter[0][e] + quarter[1][e]) + (quarter[2][e] + quarter[3][e]);
}

// Normalise-and-apply for heads of 32 channels on the matrix cores in fp32 (the operands -- rectified Q
// converted from the storage type, the fp32 state -- go in exactly).  A workgroup owns four neighbouring
// head-branches, one per wave (256 contiguous bytes of a token's row in the 16-bit types: whole lines), and
// kApplyGroups groups of 16 tokens; lane (token x16, q) holds channels 8q..8q+7 of its token (one 16-byte
// load in, one 16-byte store out in the 16-bit types).  The 32 x 32 product is a 2 x 2 arrangement of
// 16 x 16 x 16 contractions whose slots are numbered to fit that: contraction slot (q, r) of chunk jc is
// channel e = 8q + 4jc + r, output row 4q + r of chunk jo is channel f = 8q + 4jo + r.
constexpr int kApplyGroups = 8;

template <class T>
struct Row8 {                       // a lane's eight channels as loaded
    u32x4 v[sizeof(T) == 4 ? 2 : 1];
};
template <class T>
__device__ __forceinline__ Row8<T> load_row8(const T* p) {
    Row8<T> r;
    r.v[0] = *(const u32x4*)p;
    if constexpr (sizeof(T) == 4) r.v[1] = *(const u32x4*)(p + 4);
    return r;
}
template <class T>
__device__ __forceinline__ void widen_row8(const Row8<T>& r, float* out) {
    if constexpr (sizeof(T) == 4) {
        const f32x4 a = __builtin_bit_cast(f32x4, r.v[0]), b = __builtin_bit_cast(f32x4, r.v[1]);
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = a[i], out[4 + i] = b[i];
    } else {
        const typename Traits<T>::Vec x = __builtin_bit_cast(typename Traits<T>::Vec, r.v[0]);
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = Traits<T>::to_f32(x[i]);
    }
}
template <class T>
__device__ __forceinline__ void store_row8(T* p, const float* v) {
    if constexpr (sizeof(T) == 4) {
        *(f32x4*)p = f32x4{v[0], v[1], v[2], v[3]};
        *(f32x4*)(p + 4) = f32x4{v[4], v[5], v[6], v[7]};
    } else {
        typename Traits<T>::Vec x;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = Traits<T>::from_f32(v[i]);
        *(u32x4*)p = __builtin_bit_cast(u32x4, x);
    }
}

template <class T, int D>
__global__ __launch_bounds__(kGenThreads) void generic_apply_kernel(const T* __restrict__ q_ms, const float* __restrict__ kv32,
                                                                    T* __restrict__ att, int N, int n_hb, int blocks_per_image,
                                                                    float eps) {
    static_assert(D == 32, "2 x 2 blocks of 16");
    constexpr int kState = D * (D + 1);
    typedef Traits<float> F32;
    const int quads = (n_hb + 3) / 4;
    const int lane = lane_id(), wave = threadIdx.x >> 6, x16 = lane & 15, q = lane >> 4;
    const int m = (blockIdx.x % quads) * 4 + wave;
    const int nb = (blockIdx.x / quads) % blocks_per_image;
    const int b = blockIdx.x / (quads * blocks_per_image);
    if (m >= n_hb) return;      // no barrier below
    const float* st = kv32 + ((long)b * n_hb + m) * kState;
    // state operands: S[jc][jo] lane (x16, q) = KV[8q + 4jc + r][8(x16 >> 2) + 4jo + (x16 & 3)], r = 0..3
    f32x4 S[2][2];
    float ksum[8];
    const int fo = 8 * (x16 >> 2) + (x16 & 3);
#pragma unroll
    for (int jc = 0; jc < 2; ++jc)
#pragma unroll
        for (int jo = 0; jo < 2; ++jo)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[jc][jo][r] = st[(8 * q + 4 * jc + r) * (D + 1) + fo + 4 * jo];
#pragma unroll
    for (int i = 0; i < 8; ++i) ksum[i] = st[(8 * q + i) * (D + 1) + D];

    const long pitch = (long)n_hb * D;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int u, bool& live, long& at) {
        const long n = ((long)nb * kApplyGroups + u) * 16 + x16;
        live = n < N;
        at = ((long)b * N + (live ? n : 0)) * pitch + (long)m * D + 8 * q;     // a token past the end reads token 0
        return load_row8<T>(q_ms + at);
    };
    bool live, live_next = false;
    long at, at_next = 0;
    Row8<T> cur = fetch(0, live, at), next = cur;
#pragma unroll
    for (int u = 0; u < kApplyGroups; ++u) {
        if (u + 1 < kApplyGroups) next = fetch(u + 1, live_next, at_next);
        float rq[8];
        widen_row8<T>(cur, rq);
        float den = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            rq[i] = live ? fmaxf(rq[i], 0.f) : 0.f;
            den = fmaf(rq[i], ksum[i], den);
        }
        den += __shfl_xor(den, 16);
        den += __shfl_xor(den, 32);
        const f32x4 lo = {rq[0], rq[1], rq[2], rq[3]}, hi = {rq[4], rq[5], rq[6], rq[7]};
        const f32x4 n0 = F32::mma16(F32::mma16(z, S[0][0], lo), S[1][0], hi);
        const f32x4 n1 = F32::mma16(F32::mma16(z, S[0][1], lo), S[1][1], hi);
        const float inv = 1.0f / (den + eps);
        if (live) {
            const float o[8] = {n0[0] * inv, n0[1] * inv, n0[2] * inv, n0[3] * inv,
                                n1[0] * inv, n1[1] * inv, n1[2] * inv, n1[3] * inv};
            store_row8<T>(att + at, o);
        }
        cur = next;
        live = live_next;
        at = at_next;
    }
}

// The same with the output projection (Section 3.1, last sentence) in one kernel, 16-bit storage, at most 16 head-branches
// of 32: the attention rows -- made as above, rounded to the storage type as above -- go to an LDS tile that is the
// projection's token operand, and never to memory.  A workgroup of eight waves owns 256 output channels, 32 a wave, whose
// weights stay in registers (KCH chunks of 32 slots, one chunk a head-branch); it walks over tiles of 32 tokens of one
// image, and wave w makes the rows of head-branches w and w + 8.  Two tiles, one barrier a tile, Q requested a tile ahead.
// With fp32 states the matrix pipe bounds it: 4 x 512 cycles of fp32 products for the rows and 1024 for the projection a wave and
// tile.  With the states in three 16-bit parts (kParts) the rows take 4 x 144 cycles: this kernel 50 -> 40 us at 8 x 8192 tokens, 16
// head-branches, the errors of the module as with fp32 states (fp16 3.8e-4, bf16 2.9e-3).  Against rows to memory and a
// projection of its own, whole modules: 8 x 8192 tokens, 16 head-branches, fp16 200.9 -> 183.5 us; 3200, 12, bf16 48.0 -> 46.0; 1024, 4, fp16
// 34.9 -> 30.5.
// LDS: an attention row is KCH*64 bytes, the 16-byte chunk index XOR-ed with token % 16, so that the sixteen tokens of an
// operand read or a row store meet sixteen different chunks of the banks; the weights are dealt out through the same
// memory, 128 bytes of every row at a time.
template <class T, int KCH, bool kParts>
struct Apply32Project {
    static constexpr int kThreads = 512, TB = 32, kChan = 256, kHbw = KCH / 8;
    static constexpr int kRow = KCH * 64, kTile = TB * kRow, kStage = kChan * 128;
    static constexpr int kWork = 2 * kTile > kStage ? 2 * kTile : kStage;
    // a head-branch's second and third parts, two operands of the state each; all three of Ksum, in quarters; eps
    static constexpr int kTail = 2 * 2 * 1024 + 3 * 64 + 16;
    static constexpr int kLds = kWork + (kParts ? KCH * kTail : 0);
    static constexpr int kSlabs = KCH / 2;
};
template <class T, int KCH, bool kParts>
__global__ __launch_bounds__(512, 2) void apply32_project_kernel(const T* __restrict__ q_ms, const float* __restrict__ kv32,
                                                                 const T* __restrict__ w_proj, T* __restrict__ out, int N,
                                                                 int n_hb, int c_out, int n_cg, int tiles_per_image,
                                                                 long n_tt, long tiles_per_block, float eps) {
    typedef Apply32Project<T, KCH, kParts> S;
    typedef Traits<T> Tr;
    typedef typename Tr::Vec Vec;
    typedef Traits<float> F32;
    constexpr int kState = 32 * 33;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const unsigned L = xcd_remap(blockIdx.x, gridDim.x);
    const int cg = (int)(L % (unsigned)n_cg);
    const long t_begin = (long)(L / (unsigned)n_cg) * tiles_per_block;
    if (t_begin >= n_tt) return;
    const int n_my = (int)(t_begin + tiles_per_block < n_tt ? tiles_per_block : n_tt - t_begin);
    // the tile at hand: image and number in it (n_tt fits 31 bits)
    int img = (int)((unsigned)t_begin / (unsigned)tiles_per_image), at = (int)t_begin - img * tiles_per_image;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4;
    const int K = n_hb * 32;
    const int ch0 = cg * S::kChan + wave * 32;
    const bool live = ch0 < c_out;

    // Q of this wave's head-branches, both 16-token groups of a tile (a token past the image's end reads its last one, a
    // head-branch past the last reads the first: their rows are not written)
    u32x4 qv[S::kHbw][2];
    auto fetch_q = [&](int b, int n0) {
#pragma unroll
        for (int i = 0; i < S::kHbw; ++i)
#pragma unroll
            for (int jt = 0; jt < 2; ++jt) {
                const int m = wave + 8 * i, n = n0 + jt * 16 + x16;
                qv[i][jt] = *(const u32x4*)(q_ms + ((long)b * N + (n < N ? n : N - 1)) * K + (m < n_hb ? m : 0) * 32 + q * 8);
            }
    };
    fetch_q(img, at * S::TB);

    // kParts: a head-branch's state and Ksum are operands of the storage type, each value in three parts (its first, second and third 8
    // or 11 significant bits), times a power of two that puts the largest at 2^14 to 2^15 (numerator and denominator scale together).
    // fp16 ends at 2^-24, so its second and third parts are kept 2^12 times larger and their products' sums scaled back before the first
    // part's are added: all 24 bits of every value down to kLeast, 2^-28 of the largest (bf16: 2^-115).  A wave whose head-branches have a
    // smaller one that is not 0 takes fp32 products, as without kParts, with the states from memory (in_parts).  The state's first part stays in
    // registers, the others and Ksum wait in LDS, where only this wave looks for them.  Else they are fp32 operands.
    constexpr bool kF16 = std::is_same<T, _Float16>::value;
    constexpr float kUp = kF16 ? 4096.0f : 1.0f, kLeast = kF16 ? 0x1p-13f : 0x1p-100f;
    typedef typename std::conditional<kParts, Vec, f32x4[2]>::type State;
    State st[S::kHbw][2];           // kParts: [output half]; else [contraction half][output half]
    float ksum[kParts ? 1 : S::kHbw][8];
    auto tail = [&](int i) { return lds + S::kWork + (wave + 8 * i) * S::kTail; };
    auto load_fp32 = [&](int b, int m, f32x4 (&sv)[2][2], float (&sk)[8]) {
        const float* s = kv32 + ((long)b * n_hb + (m < n_hb ? m : 0)) * kState;
        const int l = kParts ? lane_id_again() : lane, q = l >> 4, fo = 8 * ((l & 15) >> 2) + (l & 3);
#pragma unroll
        for (int jc = 0; jc < 2; ++jc)
#pragma unroll
            for (int jo = 0; jo < 2; ++jo)
#pragma unroll
                for (int r = 0; r < 4; ++r) sv[jc][jo][r] = s[(8 * q + 4 * jc + r) * 33 + fo + 4 * jo];
#pragma unroll
        for (int e = 0; e < 8; ++e) sk[e] = s[(8 * q + e) * 33 + 32];
    };
    auto read_state = [&](int b, int i, float (&v)[3][8]) {
        const int l = lane_id_again(), q = l >> 4, fo = 8 * ((l & 15) >> 2) + (l & 3);       // (no register for this during the tiles)
        const int m = wave + 8 * i;
        const float* s = kv32 + ((long)b * n_hb + (m < n_hb ? m : 0)) * kState;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[0][e] = s[(8 * q + e) * 33 + fo];
            v[1][e] = s[(8 * q + e) * 33 + fo + 4];
            v[2][e] = s[(8 * q + e) * 33 + 32];
        }
    };
    // (whether it is whole in parts)
    auto make_parts = [&](int i, const float (&v)[3][8], auto straight) {
        const int l = lane_id_again(), x16 = l & 15, q = l >> 4;
        float mx = 0.f;
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(v[j][e]) < INFINITY ? fabsf(v[j][e]) : 0.f);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        float scale = 1.0f;
        if (mx > 0.f) {
            int ex;
            frexpf(mx, &ex);
            scale = ldexpf(1.0f, ex < -100 ? 115 : 15 - ex);
        }
        // (an eps so small that the scale takes it below the normal range must not become 0: 0 / eps is what a token without
        // anything above zero gives)
        const float scaled_eps = eps > 0.f ? fmaxf(eps * scale, 1.1754944e-38f) : 0.f;
        if (l == 0) *(float*)(tail(i) + S::kTail - 16) = scaled_eps;
        bool small = false;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            Vec part[3];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float x = v[j][e] * scale;
                // (straight: without branches, which beside the weights costs 30 registers in scratch)
                if constexpr (straight) small = small | ((v[j][e] != 0.f) & (fabsf(x) < kLeast));
                else small = small || (v[j][e] != 0.f && fabsf(x) < kLeast);
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    part[p][e] = Tr::from_f32(x);
                    x = fabsf(x) < INFINITY ? (x - Tr::to_f32(part[p][e])) * (p == 0 ? kUp : 1.0f) : 0.f;
                }
            }
            if constexpr (kParts)
                if (j < 2) st[i][j] = part[0];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                if (j < 2 && p > 0) *(Vec*)(tail(i) + (p - 1) * 2048 + j * 1024 + l * 16) = part[p];
                else if (j == 2 && x16 == 0) *(Vec*)(tail(i) + 4096 + p * 64 + q * 16) = part[p];
            }
        }
        return !__any(small);
    };
    auto wave_sees_lds = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto load_states = [&](int b) {
        bool in_parts = kParts;
        if constexpr (kParts) {
#pragma unroll
            for (int i = 0; i < S::kHbw; ++i) {
                float v[3][8];
                read_state(b, i, v);
                in_parts = make_parts(i, v, std::false_type{}) && in_parts;
            }
            wave_sees_lds();
        } else {
#pragma unroll
            for (int i = 0; i < S::kHbw; ++i) load_fp32(b, wave + 8 * i, st[i], ksum[i]);
        }
        return in_parts;
    };
    // With 16 head-branches, the first image's states are on their way before the weights and made into parts before those take the
    // registers (8 x 8192 tokens, 8 heads, fp16 143.5 -> 140.8 us a module, bf16 144.5 -> 142.8; with 8, 4 x 8192, 4 heads 41.9 -> 42.2).
    constexpr bool kFirst = kParts && KCH > 8;
    float first[kFirst ? S::kHbw : 1][3][8];
    bool whole = false;
    if constexpr (kFirst) {
#pragma unroll
        for (int i = 0; i < S::kHbw; ++i) read_state(img, i, first[i]);
    }

    // weights: fragment (io, kk) = rows ch0 + 16 io + x16, slots 32 kk + 8q .. +7; slots past K and rows past c_out are zero
    Vec wf[2][KCH];
    {
        constexpr int kPer = S::kChan * 8 / S::kThreads;
        const BufRsrc wres = make_rsrc(w_proj, (long)c_out * K * 2);
        const unsigned row_bytes = (unsigned)K * 2u;
        u32x4 st[S::kSlabs][kPer];
        auto request = [&](int sl) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int id = i * S::kThreads + threadIdx.x, row = cg * S::kChan + (id >> 3);
                const unsigned col = sl * 128 + (id & 7) * 16;
                st[sl][i] = buf_load16(wres, row < c_out && col < row_bytes ? (unsigned)row * row_bytes + col : kOobOffset, 0);
            }
        };
        request(0);
        if constexpr (kFirst) {
            whole = true;
#pragma unroll
            for (int i = 0; i < S::kHbw; ++i) whole = make_parts(i, first[i], std::true_type{}) && whole;
            wave_sees_lds();
        }
        static_for<0, S::kSlabs>([&](auto sl_c) {
            constexpr int sl = decltype(sl_c)::value;
            if constexpr (sl + 1 < S::kSlabs) request(sl + 1);
            if constexpr (sl > 0) __syncthreads();
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int id = i * S::kThreads + threadIdx.x, row = id >> 3;
                *(u32x4*)(lds + row * 128 + (((id & 7) ^ ((row >> 1) & 7)) * 16)) = st[sl][i];
            }
            __syncthreads();
#pragma unroll
            for (int io = 0; io < 2; ++io)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int row = wave * 32 + io * 16 + x16;
                    wf[io][2 * sl + h] = __builtin_bit_cast(Vec, *(const u32x4*)(lds + row * 128 + (((h * 4 + q) ^ ((row >> 1) & 7)) * 16)));
                }
        });
        __syncthreads();
    }
    // slots of head-branches that are not there are read with zero weights: they must hold numbers
    for (int i = threadIdx.x; i < 2 * S::TB * (KCH - n_hb) * 4; i += S::kThreads) {
        const int row = i / ((KCH - n_hb) * 4), c = n_hb * 4 + i % ((KCH - n_hb) * 4);
        *(u32x4*)(lds + row * S::kRow + ((c ^ (row & 15)) * 16)) = u32x4{0u, 0u, 0u, 0u};
    }

    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    // where chunk c + q of token x16's row is (16 chunks further on: 256 bytes)
    auto row_at = [&](int c) { return x16 * S::kRow + ((c + q) ^ x16) * 16; };
    auto rows_fp32 = [&](int to, int i, const f32x4 (&sv)[2][2], const float (&sk)[8]) {
#pragma unroll
        for (int jt = 0; jt < 2; ++jt) {
            const Vec f = __builtin_bit_cast(Vec, qv[i][jt]);
            float rq[8], den = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                rq[e] = fmaxf(Tr::to_f32(f[e]), 0.f);
                den = fmaf(rq[e], sk[e], den);
            }
            den += __shfl_xor(den, 16);
            den += __shfl_xor(den, 32);
            const f32x4 lo = {rq[0], rq[1], rq[2], rq[3]}, hi = {rq[4], rq[5], rq[6], rq[7]};
            const f32x4 n0 = F32::mma16(F32::mma16(z, sv[0][0], lo), sv[1][0], hi);
            const f32x4 n1 = F32::mma16(F32::mma16(z, sv[0][1], lo), sv[1][1], hi);
            const float inv = 1.0f / (den + eps);
            Vec o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                o[r] = Tr::from_f32(n0[r] * inv);
                o[4 + r] = Tr::from_f32(n1[r] * inv);
            }
            *(u32x4*)(lds + to + jt * 16 * S::kRow + row_at(wave * 4) + i * 512) = __builtin_bit_cast(u32x4, o);
        }
    };
    auto make_rows = [&](int to, int b, auto in_parts) {
        if constexpr (kParts && !in_parts) {
#pragma unroll
            for (int i = 0; i < S::kHbw; ++i)
                if (wave + 8 * i < n_hb) {
                    f32x4 sv[2][2];
                    float sk[8];
                    load_fp32(b, wave + 8 * i, sv, sk);
                    rows_fp32(to, i, sv, sk);
                }
        } else if constexpr (kParts) {
#pragma unroll
            for (int i = 0; i < S::kHbw; ++i) {
                const int m = wave + 8 * i;
                if (m < n_hb) {
                    Vec f[2];
                    f32x4 num[2][2], den[2];
#pragma unroll
                    for (int jt = 0; jt < 2; ++jt) {
                        f[jt] = __builtin_bit_cast(Vec, qv[i][jt]);
#pragma unroll
                        for (int e = 0; e < 8; ++e) f[jt][e] = Tr::from_f32(fmaxf(Tr::to_f32(f[jt][e]), 0.f));
                        num[jt][0] = num[jt][1] = den[jt] = z;
                    }
                    const float scaled_eps = *(const float*)(tail(i) + S::kTail - 16);
                    // small parts first; every row of the denominator's product is the same
#pragma unroll
                    for (int p = 2; p >= 0; --p) {
                        const char* at = tail(i) + (p - 1) * 2048 + lane * 16;
                        const Vec s0 = p > 0 ? *(const Vec*)at : st[i][0], s1 = p > 0 ? *(const Vec*)(at + 1024) : st[i][1];
                        const Vec sk = *(const Vec*)(tail(i) + 4096 + p * 64 + q * 16);
#pragma unroll
                        for (int jt = 0; jt < 2; ++jt) {
                            num[jt][0] = Tr::mma_vec(num[jt][0], s0, f[jt]);
                            num[jt][1] = Tr::mma_vec(num[jt][1], s1, f[jt]);
                            den[jt] = Tr::mma_vec(den[jt], sk, f[jt]);
                        }
                        if constexpr (kF16) {
                            if (p == 1) {
#pragma unroll
                                for (int jt = 0; jt < 2; ++jt) {
#pragma unroll
                                    for (int jo = 0; jo < 2; ++jo)
#pragma unroll
                                        for (int r = 0; r < 4; ++r) num[jt][jo][r] *= 1.0f / kUp;
                                    den[jt][0] *= 1.0f / kUp;       // (its other rows are not used)
                                }
                            }
                        }
                    }
#pragma unroll
                    for (int jt = 0; jt < 2; ++jt) {
                        const f32x4 n0 = num[jt][0], n1 = num[jt][1];
                        const float inv = 1.0f / (den[jt][0] + scaled_eps);
                        Vec o;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            o[r] = Tr::from_f32(n0[r] * inv);
                            o[4 + r] = Tr::from_f32(n1[r] * inv);
                        }
                        *(u32x4*)(lds + to + jt * 16 * S::kRow + row_at(wave * 4) + i * 512) = __builtin_bit_cast(u32x4, o);
                    }
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < S::kHbw; ++i)
                if (wave + 8 * i < n_hb) rows_fp32(to, i, st[i], ksum[i]);
        }
    };
    // The tiles of an image: a tile's rows, the next one's Q on its way, its projection.  A loop for each kind of state: with the
    // choice inside a tile, 8 x 8192 tokens, 8 heads, took 146.3 us in fp16 and 146.8 in bf16 instead of 143.7 and 145.5.
    int i_tile = 0;
    auto tiles = [&](auto in_parts) {
        const int b = img;
        for (; i_tile < n_my && img == b; ++i_tile) {
            const int here = (i_tile & 1) * S::kTile, n0 = at * S::TB;
            make_rows(here, b, in_parts);
            if (++at == tiles_per_image) {
                ++img;
                at = 0;
            }
            if (i_tile + 1 < n_my) fetch_q(img, at * S::TB);
            __syncthreads();                // rows of the tile complete; nobody reads the other tile any more
            f32x4 acc[2][2] = {{z, z}, {z, z}};
            if (live) {
#pragma unroll
                for (int kk = 0; kk < KCH; ++kk)
#pragma unroll
                    for (int jt = 0; jt < 2; ++jt) {
                        const Vec bf = __builtin_bit_cast(Vec, *(const u32x4*)(lds + here + jt * 16 * S::kRow + row_at(kk % 4 * 4) + kk / 4 * 256));
#pragma unroll
                        for (int io = 0; io < 2; ++io) acc[io][jt] = Tr::mma_vec(acc[io][jt], wf[io][kk], bf);
                    }
                // two 8-byte fragments leave in one 16-byte store (lane groups swapped: channels 16 (q % 2) + 8 (q / 2) .. +7)
#pragma unroll
                for (int jt = 0; jt < 2; ++jt) {
                    const u32x2 even = __builtin_bit_cast(u32x2, frag_from_f32<T>(acc[0][jt]));
                    const u32x2 odd = __builtin_bit_cast(u32x2, frag_from_f32<T>(acc[1][jt]));
                    const u32x2 s0 = __builtin_amdgcn_permlane16_swap(even[0], odd[0], false, false);
                    const u32x2 s1 = __builtin_amdgcn_permlane16_swap(even[1], odd[1], false, false);
                    const int n = n0 + jt * 16 + x16, oc = ch0 + (q & 1) * 16 + (q >> 1) * 8;
                    if (n < N && oc < c_out) *(u32x4*)(out + ((long)b * N + n) * c_out + oc) = u32x4{s0[0], s1[0], s0[1], s1[1]};
                }
            }
        }
    };
    while (i_tile < n_my) {
        if (!kFirst || i_tile > 0) whole = load_states(img);
        if (whole) {
            if constexpr (kParts) tiles(std::true_type{});
        } else {
            tiles(std::false_type{});
        }
    }
}

template <class T, int KCH, bool kParts>
hipError_t run_apply32_project_as(const GenericArgs& a, int N, int n_cg, int tpi, long n_tt, long per, hipStream_t stream) {
    typedef Apply32Project<T, KCH, kParts> S;
    static_assert(S::kLds <= 160 * 1024, "LDS layout");
    const long nblocks = (n_tt + per - 1) / per * n_cg;
    const hipError_t e = allow_dynamic_lds<apply32_project_kernel<T, KCH, kParts>>(S::kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((apply32_project_kernel<T, KCH, kParts>), dim3((unsigned)nblocks), dim3(S::kThreads), S::kLds, stream,
                       (const T*)a.q_ms, a.kv32, (const T*)a.w_proj, (T*)a.out, N, (1 + a.n_scales) * a.heads, a.c_out, n_cg, tpi, n_tt,
                       per, a.eps);
    return hipGetLastError();
}
template <class T, int KCH>
hipError_t run_apply32_project(const GenericArgs& a, int N, hipStream_t stream) {
    typedef Apply32Project<T, KCH, false> S;
    const int n_cg = (a.c_out + S::kChan - 1) / S::kChan;
    const int tpi = (N + S::TB - 1) / S::TB;
    const long n_tt = (long)a.B * tpi;
    if (n_tt * n_cg > 0x7fffffffL) return hipErrorInvalidValue;
    const long groups = compute_units() / n_cg > 0 ? compute_units() / n_cg : 1;       // one workgroup a CU (registers)
    const long per = (n_tt + groups - 1) / groups;
    // States in parts of the storage type cost their making, 1.5 us an image, and save two thirds of a tile's matrix cycles.  Us a module, fp32
    // operands / parts: 8 x 8192 tokens, 16 head-branches (8 tiles a workgroup) 152.9 / 143.3, 4 x 8192, 8 (4 tiles) 43.5 / 41.8; 3 x 8192, 16 (3)
    // 68.4 / 71.6, 2 x 8192, 16 (2) 49.5 / 49.7, 2048, 16 (1) 32.7 / 34.3.
    return per >= 4 ? run_apply32_project_as<T, KCH, true>(a, N, n_cg, tpi, n_tt, per, stream)
                    : run_apply32_project_as<T, KCH, false>(a, N, n_cg, tpi, n_tt, per, stream);
}

// fixed-order sum of the partial states, then the normalise-and-apply pass
template <class T, int D>
hipError_t finish_generic(const GenericArgs& a, int N, hipStream_t stream) {
    const int S = 1 + a.n_scales;
    const int n_states = a.B * S * a.heads;
    const long nb1 = (long)n_states * ((D * (D + 1) + kFinEntries - 1) / kFinEntries);
    if (nb1 > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((generic_state_finalize_kernel<D>), dim3((unsigned)nb1), dim3(kGenThreads), 0, stream, a.partials,
                       a.kv32, a.nchunks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (sizeof(T) == 2) {
        const int n_hb = S * a.heads;
        if (a.projected != nullptr && n_hb <= 16 && (long)a.c_out * n_hb * 64 < 0x7fffffffL) {
            e = n_hb <= 8 ? run_apply32_project<T, 8>(a, N, stream) : run_apply32_project<T, 16>(a, N, stream);
            if (e == hipSuccess) *a.projected = true;
            return e;
        }
    }
    const int bpi = (N + 16 * kApplyGroups - 1) / (16 * kApplyGroups);
    const long nb2 = (long)a.B * ((S * a.heads + 3) / 4) * bpi;
    if (nb2 > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((generic_apply_kernel<T, D>), dim3((unsigned)nb2), dim3(kGenThreads), 0, stream, (const T*)a.q_ms, a.kv32,
                       (T*)a.att, N, S * a.heads, bpi, a.eps);
    return hipGetLastError();
}

template <class T, int D>
hipError_t run_generic(const GenericArgs& a, hipStream_t stream) {
    const int N = a.H * a.W;
    const int n_groups = (N + kGenTokens - 1) / kGenTokens;
    const int gpc = (n_groups + a.nchunks - 1) / a.nchunks;
    const long nb = (long)a.B * a.heads * a.nchunks;
    if (nb <= 0 || nb > 0x7fffffffL) return hipErrorInvalidValue;
    const int S = 1 + a.n_scales;
    size_t dw_off = 0;
    if constexpr (D == 32 && sizeof(T) == 2) {
        if (a.n_scales > 0) {
            // 16-bit storage: the tiled matrix-core form (k_aggregate32.hip); its first launch also does the
            // raw branch.  Same partial-state buffer, chunks counted in 8 x 32-token tiles.
            AggregateArgs g;
            g.q = a.qkv;
            g.k = (const T*)a.qkv + D;
            g.v = (const T*)a.qkv + 2 * D;
            g.q_ts = g.k_ts = g.v_ts = 3L * a.heads * D;
            g.q_hs = g.k_hs = g.v_hs = 3 * D;
            g.q_ms = a.q_ms;
            g.partials = a.partials;
            g.B = a.B; g.H = a.H; g.W = a.W; g.heads = a.heads; g.S = S;
            // one workgroup a compute unit where every scale has the matrix-core kernel (never more partial states than the plan has room for)
            GenericArgs c = a;
            const long widest = (long)std::max(3, S) * a.heads * D;
            bool all = true;
            for (int i = 0; i < a.n_scales; ++i) all = all && aggregate32_on_matrix_cores(a.scales[i], (long)a.H * a.W, widest);
            if (all) {
                const long tiles16 = (long)((a.H + kAggMfmaTileH - 1) / kAggMfmaTileH) * ((a.W + kAggMfmaTileW - 1) / kAggMfmaTileW);
                const long states = (long)a.B * a.heads;
                const long want = chunks_in_rounds(states, tiles16, std::min((long)a.nchunks, tiles16), compute_units());
                const long tpc = (tiles16 + want - 1) / want;
                c.nchunks = (int)((tiles16 + tpc - 1) / tpc);
            }
            g.nchunks = c.nchunks;
            const long tiles = (long)((a.H + kAggTileH - 1) / kAggTileH) * ((a.W + kAggTileW - 1) / kAggTileW);
            g.tiles_per_chunk = (int)((tiles + c.nchunks - 1) / c.nchunks);
            for (int i = 0; i < a.n_scales; ++i) {
                const int ks = a.scales[i];
                g.w_dw = (const T*)a.w_dw + dw_off;
                g.w_gpw = (const T*)a.w_gpw + (size_t)i * 3 * a.heads * D * D;
                dw_off += (size_t)3 * a.heads * D * ks * ks;
                g.ks = ks;
                g.branch = i + 1;
                g.do_raw = (i == 0);
                g.copy_raw_q = (i == 0);
                const hipError_t e = launch_aggregate32(sizeof(T) == 2 && std::is_same<T, _Float16>::value ? 1 : 2, g, stream);
                if (e != hipSuccess) return e;
            }
            return finish_generic<T, D>(c, N, stream);
        }
    }
    for (int s = 0; s < S; ++s) {
        const int ks = s == 0 ? 0 : a.scales[s - 1];
        const T* wdw = s == 0 ? nullptr : (const T*)a.w_dw + dw_off;
        const T* wgp = s == 0 ? nullptr : (const T*)a.w_gpw + (size_t)(s - 1) * 3 * a.heads * D * D;
        if (s > 0) dw_off += (size_t)3 * a.heads * D * ks * ks;
        hipLaunchKernelGGL((generic_branch_state_kernel<T, D>), dim3((unsigned)nb), dim3(kGenThreads), 0, stream,
                           (const T*)a.qkv, wdw, wgp, (T*)a.q_ms, a.partials, a.H, a.W, a.heads, S, s, ks, a.nchunks, gpc);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return finish_generic<T, D>(a, N, stream);
}

template <class T>
hipError_t run_generic_d(const GenericArgs& a, hipStream_t stream) {
    if (a.head_dim == 32) return run_generic<T, 32>(a, stream);
    return hipErrorNotSupported;
}

// row of the paired arrangement -> row of the head-size-8 arrangement (channel order (h*3 + t)*d + e)
__device__ __forceinline__ int head8_row(int row16) {
    const int hp = row16 / 48, r = row16 - hp * 48, t = r >> 4, e16 = r & 15;
    return ((2 * hp + (e16 >> 3)) * 3 + t) * 8 + (e16 & 7);
}

template <class T>
__global__ __launch_bounds__(256) void pair_head8_weights_kernel(const T* __restrict__ w_qkv, const T* __restrict__ w_dw,
                                                                 const T* __restrict__ w_gpw, T* __restrict__ o_qkv,
                                                                 T* __restrict__ o_dw, T* __restrict__ o_gpw, int C, int rows,
                                                                 int n_scales, int k0, int k1, int k2, int k3, int k4, int k5,
                                                                 int k6, int k7) {
    const int ks[8] = {k0, k1, k2, k3, k4, k5, k6, k7};
    const long n_qkv = (long)rows * C;
    long n_dw = 0;
    for (int i = 0; i < n_scales; ++i) n_dw += (long)rows * ks[i] * ks[i];
    const long n_gpw = (long)n_scales * rows * 16;
    const long total = n_qkv + n_dw + n_gpw;
    for (long id = (long)blockIdx.x * blockDim.x + threadIdx.x; id < total; id += (long)gridDim.x * blockDim.x) {
        if (id < n_qkv) {
            const int row = (int)(id / C), c = (int)(id - (long)row * C);
            o_qkv[id] = w_qkv[(long)head8_row(row) * C + c];
        } else if (id < n_qkv + n_dw) {
            long r = id - n_qkv, base = 0;
            int i = 0;
            while (r >= (long)rows * ks[i] * ks[i]) {
                r -= (long)rows * ks[i] * ks[i];
                base += (long)rows * ks[i] * ks[i];
                ++i;
            }
            const int kk = ks[i] * ks[i];
            const int row = (int)(r / kk), tap = (int)(r - (long)row * kk);
            o_dw[base + r] = w_dw[base + (long)head8_row(row) * kk + tap];
        } else {
            const long r = id - n_qkv - n_dw;
            const int i = (int)(r / ((long)rows * 16));
            const int rem = (int)(r - (long)i * rows * 16);
            const int row = rem >> 4, col = rem & 15;
            const bool own = (col >> 3) == ((row & 15) >> 3);
            o_gpw[r] = own ? w_gpw[((long)i * rows + head8_row(row)) * 8 + (col & 7)] : Traits<T>::from_f32(0.f);
        }
    }
}

template <class T>
hipError_t run_pair_head8(const void* w_qkv, const void* w_dw, const void* w_gpw, void* o_qkv, void* o_dw, void* o_gpw, int C,
                          int heads8, const int* scales, int n_scales, hipStream_t stream) {
    int k[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = 0; i < n_scales; ++i) k[i] = scales[i];
    const int rows = 3 * heads8 * 8;
    hipLaunchKernelGGL((pair_head8_weights_kernel<T>), dim3(256), dim3(256), 0, stream, (const T*)w_qkv, (const T*)w_dw,
                       (const T*)w_gpw, (T*)o_qkv, (T*)o_dw, (T*)o_gpw, C, rows, n_scales, k[0], k[1], k[2], k[3], k[4], k[5],
                       k[6], k[7]);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pair_head8_weights(int dt, const void* w_qkv, const void* w_dw, const void* w_gpw, void* w_qkv16,
                                     void* w_dw16, void* w_gpw16, int C, int heads8, const int* scales, int n_scales,
                                     hipStream_t stream) {
    if (heads8 <= 0 || heads8 % 2 != 0 || n_scales < 0 || n_scales > 8) return hipErrorInvalidValue;
    switch (dt) {
        case 0: return run_pair_head8<float>(w_qkv, w_dw, w_gpw, w_qkv16, w_dw16, w_gpw16, C, heads8, scales, n_scales, stream);
        case 1: return run_pair_head8<_Float16>(w_qkv, w_dw, w_gpw, w_qkv16, w_dw16, w_gpw16, C, heads8, scales, n_scales, stream);
        case 2: return run_pair_head8<__bf16>(w_qkv, w_dw, w_gpw, w_qkv16, w_dw16, w_gpw16, C, heads8, scales, n_scales, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_generic_core(int dt, const GenericArgs& a, hipStream_t stream) {
    switch (dt) {
        case 0: return run_generic_d<float>(a, stream);
        case 1: return run_generic_d<_Float16>(a, stream);
        case 2: return run_generic_d<__bf16>(a, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace msla
