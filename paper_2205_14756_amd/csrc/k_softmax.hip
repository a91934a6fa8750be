// Softmax attention, the comparison point of ReLU linear attention (Section 3.1: Eq. (1) with
// Sim(Q, K) = exp(Q K^T / sqrt(d)); Fig. 3 compares the latency of the two forms):
//     O_i = sum_j exp(Q_i . K_j / sqrt(d)) V_j / sum_j exp(Q_i . K_j / sqrt(d))
// per image and head on a projected map qkv [B, N, 3*heads*16] (channel (h*3 + t)*16 + e).
//
// It is quadratic in N by definition; it is written the way such a kernel is written when it has to
// be fast (one pass over the keys with a running maximum and running sums, nothing of size N x N
// ever stored), so that the ratio to the linear form is a fair one.  Two kernels: the 16-bit types take
// softmax_attention32_kernel (below), fp32 the following one.  A workgroup of 4 waves takes
// 64 queries of one (image, head), a wave 16 of them, and walks over the keys 64 at a time:
//     S^T[key][query] = K . Q^T      four 16x16x4 MFMAs per 16 keys; lane (query x16, q) gets keys 4q..4q+3
//     running max per query (in-lane over 16 values, two shuffles over the four q groups), P = 2^(S - max)
//     O^T[f][query]  += V^T . P^T    the same; P's fragment is S's
// K (row-major) and V (transposed, so a lane's four keys are contiguous) go through LDS once per
// workgroup and key block, the next block's loads in flight during the arithmetic.
#include "msla_device.h"
#include "msla_kernels.h"

namespace msla {
namespace {

constexpr int kSmQ = 64;        // queries per workgroup
constexpr int kSmK = 64;        // keys per iteration

__global__ __launch_bounds__(256) void softmax_attention_kernel(const float* __restrict__ qkv, float* __restrict__ att, int N,
                                                                int heads, int q_blocks) {
    typedef Traits<float> Tr;
    constexpr int kKRow = 16 * 4 + 16;                               // K tile [key][16 d], padded
    constexpr int kVRow = kSmK * 4 + 16;                             // V^T tile [f][64 keys], padded
    __shared__ __attribute__((aligned(16))) char ldsK[2][kSmK * kKRow];
    __shared__ __attribute__((aligned(16))) char ldsV[2][16 * kVRow];

    const int qb = blockIdx.x % q_blocks;
    const int h = (blockIdx.x / q_blocks) % heads;
    const int b = blockIdx.x / (q_blocks * heads);
    const int wave = threadIdx.x >> 6, lane = lane_id(), x16 = lane & 15, q = lane >> 4;
    const long ts = 3L * heads * 16;                                  // elements from token to token
    const float* base = qkv + (long)b * N * ts + (long)h * 48;

    // this lane's query (column x16 of the wave's 16): its channels 4q..4q+3, scaled by log2(e)/sqrt(d)
    const int my_query = qb * kSmQ + wave * 16 + x16;
    f32x4 qf = {0.f, 0.f, 0.f, 0.f};
    if (my_query < N) qf = load_frag<float>(base + (long)my_query * ts + q * 4);
    constexpr float kScale = 0.25f * 1.4426950408889634f;             // 1/sqrt(16) * log2(e)

    // cooperative loads of a key block: thread t < 128 brings 4 d-channels of K, t >= 128 of V, of two keys
    constexpr int kRowsPerPass = 32;                                  // keys covered by 128 threads, four a key
    constexpr int kPasses = kSmK / kRowsPerPass;
    const int half = threadIdx.x >> 7, t7 = threadIdx.x & 127;
    u32x4 stage[kPasses];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int key = k0 + p * kRowsPerPass + t7 / 4;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (key < N) v = *(const u32x4*)(base + (long)key * ts + 16 + half * 16 + (t7 % 4) * 4);
            stage[p] = v;
        }
    };
    auto park = [&](int buf) {
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int key = p * kRowsPerPass + t7 / 4;
            const int c0 = (t7 % 4) * 4;
            if (half == 0) {
                // K: row-major (fragments go to and from these rows as two 8-byte words: 16-byte ones take 0.6 % longer)
                store_frag<float>(ldsK[buf] + key * kKRow + c0 * 4, __builtin_bit_cast(f32x4, stage[p]));
            } else {
                const f32x4 e = __builtin_bit_cast(f32x4, stage[p]);          // V: transposed, element by element
#pragma unroll
                for (int j = 0; j < 4; ++j) *(float*)(ldsV[buf] + (c0 + j) * kVRow + key * 4) = e[j];
            }
        }
    };

    float m_run = -INFINITY;            // running maximum of this lane's query (same in its four q lanes)
    float l_run = 0.f;                  // running sum over this lane's own keys
    f32x4 o = {0.f, 0.f, 0.f, 0.f};     // O^T[f = 4q + r][query x16]
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};

    fetch(0);
    park(0);
    __syncthreads();
    const int n_blocks = (N + kSmK - 1) / kSmK;
    for (int blk = 0; blk < n_blocks; ++blk) {
        const int buf = blk & 1;
        if (blk + 1 < n_blocks) fetch((blk + 1) * kSmK);
        // scores of 64 keys x 16 queries: s[g][r] = key 16g + 4q + r
        f32x4 s[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 kf = load_frag<float>(ldsK[buf] + (g * 16 + x16) * kKRow + q * 16);
            s[g] = Tr::mma16(z, kf, qf);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = blk * kSmK + g * 16 + q * 4 + r;
                s[g][r] = key < N ? s[g][r] * kScale : -INFINITY;
                mx = fmaxf(mx, s[g][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);             // finite from the first block on: it holds key 0
        const float keep = exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= keep;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] *= keep;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            f32x4 p;
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = exp2f(s[g][r] - m_new);
            l_run += (p[0] + p[1]) + (p[2] + p[3]);
            const f32x4 vf = load_frag<float>(ldsV[buf] + x16 * kVRow + (g * 16 + q * 4) * 4);
            o = Tr::mma16(o, vf, p);
        }
        if (blk + 1 < n_blocks) park(buf ^ 1);
        __syncthreads();
    }
    // the denominators: sum over the four q lanes of a query
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    const float inv = 1.0f / l_run;
    // lane (query x16, q) holds channels f = 4q..4q+3 of its query: 16 contiguous bytes
    if (my_query < N)
        *(f32x4*)(att + ((long)b * N + my_query) * (heads * 16) + h * 16 + q * 4) =
            f32x4{o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
}

// ---------------------------------------------------------------- 16-bit storage types
// What bounds this form is the vector ALU: each score takes half a maximum, a multiply-add, an exponential and half
// a conversion (22 cycles of a SIMD measured for 64 scores, against 6 of the matrix pipe).  So everything else is
// kept off it.  The products are 32x32x16 matrix instructions (the contraction of K . Q^T is the head size, 16: the
// 16x16 form spends the same cycles on a quarter of the scores).  A lane then holds 16 of the 32 keys of ONE query,
// so a maximum needs one exchange between the wave's halves per 64 keys.  The sums of the weights are a row of ones
// under V^T.  The accumulators are rescaled whenever one of the wave's queries finds a larger score, so that the weights
// are at most 1 and the heaviest of a block lie just below it, where the 16-bit grid is relatively finest.  (Letting the
// maximum lag behind by up to 2^8 saves most of the rescaling, 85 instead of 89 us, but spreads the weights over the whole
// grid: relative error 2.92e-4 instead of 2.79e-4 in fp16, 2.33e-3 instead of 2.23e-3 in bf16.)  Weights below 2^-126
// of the largest are flushed to zero by the exponential instruction.  The key test exists in a ragged last tile only.
// 8 x 16 heads, 2048 tokens, fp16 (537 M scores): 89 us; with 16x16 products and a rescaling in every block, 232 us.
constexpr int kSm2Keys = 128;           // keys per LDS tile
constexpr int kSm2VRow = kSm2Keys * 2 + 16;                 // V^T row in LDS, padded by one 16-byte slot
constexpr int kSm2KBytes = kSm2Keys * 32;                   // K tile: two planes [half of d][key][16 bytes]
constexpr int kSm2VBytes = 18 * kSm2VRow;                   // 16 channels, a row of ones, a row of zeros
constexpr int kSm2Lds = 2 * (kSm2KBytes + kSm2VBytes);

typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x16 mma32(f32x16 c, f16x8 a, f16x8 b) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mma32(f32x16 c, bf16x8 a, bf16x8 b) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// kSplit: false -- a wave has 32 queries of its own and walks all keys; true -- the four waves share 32 queries,
// wave w takes keys 32w..32w+31 of every tile, and the four partial results are merged in LDS at the end.
template <class T, bool kSplit>
__global__ __launch_bounds__(256, 4) void softmax_attention32_kernel(const T* __restrict__ qkv, T* __restrict__ att, int N,
                                                                     int heads, int q_blocks) {
    typedef Traits<T> Tr;
    typedef typename Tr::Vec Vec;
    __shared__ __attribute__((aligned(16))) char lds[kSm2Lds];
    char* const ldsK = lds;                                     // two buffers
    char* const ldsV = lds + 2 * kSm2KBytes;

    const unsigned bid = xcd_remap(blockIdx.x, gridDim.x);      // the query blocks of a head share an L2
    const int qb = bid % q_blocks;
    const int h = (bid / q_blocks) % heads;
    const int b = bid / (q_blocks * heads);
    const int wave = threadIdx.x >> 6, lane = lane_id(), col = lane & 31, half = lane >> 5;
    const long ts = 3L * heads * 16;                            // elements from token to token
    const T* base = qkv + (long)b * N * ts + (long)h * 48;
    constexpr float kScale = 0.25f * 1.4426950408889634f;       // 1/sqrt(16) * log2(e)

    const int my_query = kSplit ? qb * 32 + col : qb * 128 + wave * 32 + col;
    const Vec qf = __builtin_bit_cast(Vec, *(const u32x4*)(base + (long)(my_query < N ? my_query : N - 1) * ts + half * 8));

    // the constant rows of both V^T buffers
    for (int i = threadIdx.x; i < 2 * 2 * kSm2VRow / 2; i += 256) {
        const int buf = i / kSm2VRow, j = i % kSm2VRow;         // kSm2VRow / 2 elements of ones, then of zeros
        *(T*)(ldsV + buf * kSm2VBytes + 16 * kSm2VRow + j * 2) = Tr::from_f32(j < kSm2VRow / 2 ? 1.0f : 0.0f);
    }

    // a tile's loads: thread t brings channels 8c..8c+7 of K and of V of key t / 2, c = t % 2.  A key past the end
    // reads the last one: its scores are masked, its V is zeroed.
    const int t_key = threadIdx.x >> 1, t_c = threadIdx.x & 1;
    u32x4 stage_k, stage_v;
    auto fetch = [&](int k0) {
        const int key = k0 + t_key < N ? k0 + t_key : N - 1;
        const T* p = base + (long)key * ts + 16 + t_c * 8;
        stage_k = *(const u32x4*)p;
        stage_v = *(const u32x4*)(p + 16);
        if (k0 + t_key >= N) stage_v = u32x4{0u, 0u, 0u, 0u};
    };
    // V^T rows keep the keys of a 32-key group in the order in which the lanes hold their weights: matrix
    // instruction p, half, then the eight contraction slots
    const int t_pos = (t_key & ~31) + ((t_key >> 4) & 1) * 16 + ((t_key >> 2) & 1) * 8 + ((t_key >> 3) & 1) * 4 + (t_key & 3);
    auto park = [&](int buf) {
        *(u32x4*)(ldsK + buf * kSm2KBytes + t_c * (kSm2Keys * 16) + t_key * 16) = stage_k;
        T e[8];
        __builtin_memcpy(e, &stage_v, 16);
#pragma unroll
        for (int j = 0; j < 8; ++j) *(T*)(ldsV + buf * kSm2VBytes + (t_c * 8 + j) * kSm2VRow + t_pos * 2) = e[j];
    };

    float m_run = -INFINITY;            // what this lane's query's exponents are taken relative to
    f32x16 o;                           // O^T[row][query col]: rows 0..15 channels, row 16 the sum of the weights
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = z[i] = 0.f;
    const char* const k_lane = ldsK + half * (kSm2Keys * 16) + col * 16;
    const char* const v_lane = ldsV + (col < 17 ? col : 17) * kSm2VRow + half * 16;

    // kSub groups of 32 keys of the tile in `buf`, from group `first` on
    auto sweep = [&](auto nsub, auto ragged, int buf, int first, int k0) {
        constexpr int kSub = decltype(nsub)::value;
        f32x16 s[kSub];
#pragma unroll
        for (int u = 0; u < kSub; ++u) {
            const Vec kf = __builtin_bit_cast(Vec, *(const u32x4*)(k_lane + buf * kSm2KBytes + (first + u) * 512));
            s[u] = mma32(z, kf, qf);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < kSub; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if constexpr (decltype(ragged)::value) {
                    const int key = k0 + (first + u) * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
                    if (key >= N) s[u][i] = -INFINITY;
                }
                mx = fmaxf(mx, s[u][i]);
            }
        const unsigned mx_bits = __builtin_bit_cast(unsigned, mx);
        const auto both = __builtin_amdgcn_permlane32_swap(mx_bits, mx_bits, false, false);
        const unsigned mx_lo = both[0], mx_hi = both[1];           // the lower and the upper half's maximum
        mx = fmaxf(__builtin_bit_cast(float, mx_lo), __builtin_bit_cast(float, mx_hi)) * kScale;
        if (__any(mx > m_run)) {
            const float m_new = fmaxf(m_run, mx);
            // (nothing seen yet, or nothing but masked keys: no weight is in o)
            const float keep = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
#pragma unroll
            for (int i = 0; i < 9; ++i) o[i] *= keep;
        }
        const float m_sub = m_run == -INFINITY ? 0.0f : m_run;      // a split wave whose keys so far are all masked
#pragma unroll
        for (int u = 0; u < kSub; ++u)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                Vec pf;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    pf[j] = Tr::from_f32(__builtin_amdgcn_exp2f(__builtin_fmaf(s[u][p * 8 + j], kScale, -m_sub)));
                const Vec vf = __builtin_bit_cast(Vec, *(const u32x4*)(v_lane + buf * kSm2VBytes + (first + u) * 64 + p * 32));
                o = mma32(o, vf, pf);
            }
    };
    constexpr std::integral_constant<int, kSplit ? 1 : 2> nsub;

    fetch(0);
    park(0);
    __syncthreads();
    const int n_full = N / kSm2Keys, n_tiles = (N + kSm2Keys - 1) / kSm2Keys;
    const int first = kSplit ? wave : 0, last = kSplit ? wave + 1 : 4;
    // a wave whose queries are all past the end has nothing to do, nor has anyone with the last tile's groups that are
    // (2048 sequences of 64 tokens 12.1 -> 7.8 us, 4096 of 16 20.5 -> 8.6; with 64 queries a workgroup and 16x16 products 9.5
    // and 11.8)
    const bool live = kSplit || qb * 128 + wave * 32 < N;
    for (int tile = 0; tile < n_full; ++tile) {
        const int buf = tile & 1, k0 = tile * kSm2Keys;
        if (tile + 1 < n_tiles) fetch(k0 + kSm2Keys);
        if (live) {
#pragma unroll 2
            for (int g = first; g < last; g += nsub) sweep(nsub, std::false_type{}, buf, g, k0);
        }
        if (tile + 1 < n_tiles) park(buf ^ 1);
        __syncthreads();
    }
    if (n_full < n_tiles) {             // the ragged last tile
#pragma unroll 1
        for (int g = first; g < last && live && n_full * kSm2Keys + g * 32 < N; g += nsub)
            sweep(nsub, std::true_type{}, n_full & 1, g, n_full * kSm2Keys);
        __syncthreads();
    }

    if constexpr (kSplit) {
        // merge the four waves: [wave][17 rows][32 queries] and [wave][32 maxima], over the dead tiles
        float* const part = (float*)lds;
        float* const pm = part + 4 * 17 * 32;
        static_assert(4 * 18 * 32 * 4 <= kSm2Lds, "merge area");
#pragma unroll
        for (int i = 0; i < 8; ++i) part[(wave * 17 + 8 * (i >> 2) + 4 * half + (i & 3)) * 32 + col] = o[i];
        if (half == 0) {
            part[(wave * 17 + 16) * 32 + col] = o[8];
            pm[wave * 32 + col] = m_run;
        }
        __syncthreads();
        const int query = threadIdx.x >> 3, f0 = (threadIdx.x & 7) * 2;
        float m = pm[query];
#pragma unroll
        for (int w = 1; w < 4; ++w) m = fmaxf(m, pm[w * 32 + query]);
        float l = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = pm[w * 32 + query];
            const float sc = mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mw - m);
            l = __builtin_fmaf(sc, part[(w * 17 + 16) * 32 + query], l);
            a0 = __builtin_fmaf(sc, part[(w * 17 + f0) * 32 + query], a0);
            a1 = __builtin_fmaf(sc, part[(w * 17 + f0 + 1) * 32 + query], a1);
        }
        const float inv = 1.0f / l;
        if (qb * 32 + query < N) {
            T r[2] = {Tr::from_f32(a0 * inv), Tr::from_f32(a1 * inv)};
            uint32_t w;
            __builtin_memcpy(&w, r, 4);
            *(uint32_t*)(att + ((long)b * N + qb * 32 + query) * (heads * 16) + h * 16 + f0) = w;
        }
    } else {
        const float inv = 1.0f / __shfl(o[8], col);             // row 16 sits in the lower half's lanes
        if (my_query < N) {
            T* out = att + ((long)b * N + my_query) * (heads * 16) + h * 16 + half * 4;
            store_frag<T>(out, frag_from_f32<T>(f32x4{o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv}));
            store_frag<T>(out + 8, frag_from_f32<T>(f32x4{o[4] * inv, o[5] * inv, o[6] * inv, o[7] * inv}));
        }
    }
}

template <class T>
hipError_t run_softmax(const void* qkv, void* att, int B, int N, int heads, hipStream_t stream) {
    if constexpr (sizeof(T) == 2) {
        // four waves with 128 queries between them wherever that gives every compute unit a workgroup or more;
        // below that the keys are split over the waves and a workgroup has 32 queries
        // (8 heads of 2048 tokens, 128 wide workgroups: 19.8 us wide, 14.2 split; 256 of them: 20.1 wide, 21.3 split)
        const long wide = (long)B * heads * ((N + 127) / 128);
        const bool split = wide < compute_units();
        const int qb = split ? (N + 31) / 32 : (N + 127) / 128;
        const long n = (long)B * heads * qb;
        if (n <= 0 || n > 0x7fffffffL) return hipErrorInvalidValue;
        if (split)
            hipLaunchKernelGGL((softmax_attention32_kernel<T, true>), dim3((unsigned)n), dim3(256), 0, stream, (const T*)qkv,
                               (T*)att, N, heads, qb);
        else
            hipLaunchKernelGGL((softmax_attention32_kernel<T, false>), dim3((unsigned)n), dim3(256), 0, stream, (const T*)qkv,
                               (T*)att, N, heads, qb);
        return hipGetLastError();
    } else {
        const int q_blocks = (N + kSmQ - 1) / kSmQ;
        const long nblocks = (long)B * heads * q_blocks;
        if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
        hipLaunchKernelGGL(softmax_attention_kernel, dim3((unsigned)nblocks), dim3(256), 0, stream, (const float*)qkv, (float*)att,
                           N, heads, q_blocks);
        return hipGetLastError();
    }
}

}  // namespace

hipError_t launch_softmax_attention(int dt, const void* qkv, void* att, int B, int N, int heads, hipStream_t stream) {
    switch (dt) {
        case 0: return run_softmax<float>(qkv, att, B, N, heads, stream);
        case 1: return run_softmax<_Float16>(qkv, att, B, N, heads, stream);
        case 2: return run_softmax<__bf16>(qkv, att, B, N, heads, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace msla
