// Multi-scale token aggregation fused with the state of Eq. (3), 16-bit storage types, for maps that give every compute unit a
// tile or two: one workgroup takes one (image, head) and one tile of 8 x 32 tokens, and optionally computes that tile's Q, K
// and V from x itself (Section 3.1: the projection below Eq. (1), then the aggregation of the last paragraph).
//
// What bounds such a call is not work but the chain of waits: 1.7 us pass from the end of one kernel to the first
// instruction of the next, and 2 us more to its first data.  So there is one kernel less (the projection's
// products for a tile, halo included, take 1.5 us), all eight waves stage the tile with every load in flight
// at once, and then all eight sweep it (aggregate_sweep.h), instead of four waves staging for eight others as in the kernel that
// walks many tiles (k_aggregate_mfma.hip).  8192 tokens of 128 channels, 8 heads, fp16: some 9 us from first to last instruction (first
// data at 2.5, staged at 6, swept in 1.8) where projection, launch and aggregation took 5.5 + 1.7 + 8.8; the module
// 23.5 -> 19.8 us, the block 44.4 -> 38.5.
//
// Projection: 16 tokens x 48 channels a step, D[token][channel] = x W^T with x fragments straight from memory and the head's 48
// rows of weights in LDS; a lane ends up with four tokens of one channel, which is the channel-planar form that the sweep wants.
// Values are rounded to the storage type there, exactly as when Q, K and V are stored between two kernels.  Q of the tile's own
// tokens, for the multi-scale map, is multiplied again with the operands swapped: through an identity matrix, an infinite value (an
// fp16 overflow) would turn the same channel of its 15 neighbours into NaN.
#include <algorithm>
#include <type_traits>

#include "aggregate_sweep.h"
#include "msla_kernels.h"

namespace msla {
namespace {

constexpr int kTH = kAggSmallTileH, kTW = kAggSmallTileW;
constexpr int kSmallWaves = 8;
constexpr int kSmallThreads = kSmallWaves * 64;
constexpr int kRows = kTH / (kSmallWaves / 2);      // a wave sweeps one of two 16-column strips, 2 rows
static_assert(kTW == 32 && kRows == 2, "eight waves: two strips x four row pairs");

// KSA, KSB: filter sizes of the scales (KSB 0: one scale); KC: 32-channel steps of the projection (0: Q, K and V are read)
template <int KSA, int KSB, int KC>
struct SLds {
    static constexpr int KS = KSA > KSB ? KSA : KSB;
    static constexpr int P = (KS - 1) / 2;
    static constexpr int LH = kTH + 2 * P, LW = kTW + 2 * P;
    static constexpr int kChanBytes = planar_chan_bytes(LH);
    static constexpr int kPlanarBytes = (48 * kChanBytes + 15) / 16 * 16;
    static constexpr int kWPitch = KC * 64 + 32;                // (32 mod 128 bytes: sixteen rows' operand reads without bank conflicts)
    static constexpr int kWBytes = KC > 0 ? 48 * kWPitch : 0;
    static constexpr int kTransAll = kSmallWaves * 2 * kTransBytes;
    // the weights are dead when the sweep begins
    static constexpr int kWork = kWBytes > kTransAll ? kWBytes : kTransAll;
    static constexpr int kTapsA = 48 * KSA * KSA * 2, kTapsB = 48 * KSB * KSB * 2;     // the head's filter taps, 16-byte pieces
    static constexpr int kBytes = kPlanarBytes + kWork + kTapsA + kTapsB;
    // 16-token groups of the halo tile: two per row, and the 2P columns behind them, four rows a group
    static constexpr int kGroups = 2 * LH + (LH + 3) / 4;
    static constexpr int kPer = (kGroups + kSmallWaves - 1) / kSmallWaves;
    static_assert(LW <= 36 && kBytes <= 160 * 1024, "LDS layout");
};

// KSB: a second scale of the same module (0: none), with its filters w_dw_b, w_gpw_b and branch_b; it sweeps the same staged tile.
// One scale leaves room for two workgroups a compute unit, 128 registers a wave, if x goes through them in two halves, one after
// the other, and the filter's operands are made when the tile is staged.  That costs a lone workgroup nothing measurable.  Two scales
// would spill.
template <class T, int KSA, int KSB, int KC>
__global__ __launch_bounds__(kSmallThreads, KSB == 0 ? 4 : 2) void aggregate_small_kernel(AggregateArgs a, const T* w_dw_b, const T* w_gpw_b,
                                                                           int branch_b) {
    constexpr int KS = KSA > KSB ? KSA : KSB;
    typedef Traits<T> Tr;
    typedef typename Tr::Frag Frag;
    typedef typename Tr::Vec Vec;
    typedef SLds<KSA, KSB, KC> L;
    constexpr int P = L::P, SZ = (int)sizeof(T);
    constexpr bool kProject = KC > 0, kTwo = KSB == 0;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* const planar = lds;
    char* const w_lds = lds + L::kPlanarBytes;
    char* const taps_lds = w_lds + L::kWork;

    const unsigned Lid = xcd_remap(blockIdx.x, gridDim.x);      // the heads of a tile share an L2
    if (Lid >= (unsigned)a.B * a.heads * a.nchunks) return;
    const int h = Lid % a.heads;
    const int tile = (Lid / a.heads) % a.nchunks;
    const int b = Lid / (a.heads * a.nchunks);
    const int Ct = a.heads * 16;
    const long N = (long)a.H * a.W;
    const long img_tok0 = (long)b * N;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x16 = lane & 15, q = lane >> 4;
    const int tiles_x = (a.W + kTW - 1) / kTW;
    const int ty0 = tile / tiles_x * kTH, tx0 = tile % tiles_x * kTW;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};

    constexpr int kScales = KSB > 0 ? 2 : 1, kB = KSB > 0 ? KSB : KSA;
    T* q_ms = (T*)a.q_ms;
    const unsigned q_ms_tb = (unsigned)(a.S * Ct * SZ);

    // ---------------- staging.  Group g of the halo tile: 16 tokens in a row (two groups a row), or the last columns
    // (32 .. 35) of four rows.  Token slot i of it:
    auto at_row = [&](int g, int i) { return g < 2 * L::LH ? g >> 1 : 4 * (g - 2 * L::LH) + (i >> 2); };
    auto at_col = [&](int g, int i) { return g < 2 * L::LH ? (g & 1) * 16 + i : 32 + (i & 3); };
    // the token in the image, or -1 outside the tile or the image
    auto token = [&](int g, int i) {
        const int ly = at_row(g, i), lx = at_col(g, i), gy = ty0 - P + ly, gx = tx0 - P + lx;
        return ly < L::LH && lx < L::LW && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W ? gy * a.W + gx : -1;
    };
    // ... if it is one of the tile's own (halo tokens belong to other tiles)
    auto own_token = [&](int g, int i) {
        const int ly = at_row(g, i), lx = at_col(g, i);
        return ly >= P && ly < P + kTH && lx >= P && lx < P + kTW ? token(g, i) : -1;
    };
    constexpr int kX = kProject ? KC : 1;
    constexpr int kHalf = kProject && kTwo ? (L::kPer + 1) / 2 : L::kPer;       // groups in flight at once
    u32x4 xf[kHalf][kX];                    // x fragments, or K | V
    u32x2 qf[L::kPer];                      // Q (when it is read)
    auto fetch_x = [&](int first) {
        const BufRsrc rx = make_rsrc((const T*)a.q + img_tok0 * a.C, N * a.C * SZ);
#pragma unroll
        for (int j = 0; j < kHalf; ++j) {
            const int t = token(wave + kSmallWaves * (first + j), x16);
#pragma unroll
            for (int s = 0; s < kX; ++s)
                xf[j][s] = buf_load16(rx, t >= 0 && s * 32 + q * 8 < a.C ? (unsigned)(t * a.C + s * 32 + q * 8) * SZ : kOobOffset, 0);
        }
    };
    // the head's filter taps, through LDS (read from memory channel by channel, their 39 words cost as much address traffic as x)
    constexpr int kTapPieces = (L::kTapsA + L::kTapsB) / 16;
    static_assert(kTapPieces <= kSmallThreads, "one piece a thread");
    u32x4 tap_piece;
    if (threadIdx.x < kTapPieces) {
        if (threadIdx.x < L::kTapsA / 16) tap_piece = ((const u32x4*)((const T*)a.w_dw + (long)h * 48 * KSA * KSA))[threadIdx.x];
        else tap_piece = ((const u32x4*)(w_dw_b + (long)h * 48 * KSB * KSB))[threadIdx.x - L::kTapsA / 16];
    }
    if constexpr (kProject) {
        // the head's rows of w_qkv to LDS, 16-byte pieces; channels past C are zero.  Half of the waves bring them, so that
        // none of them queues behind the other half's x
        constexpr int kPieces = 48 * KC * 4, kWThreads = 256, kWPer = (kPieces + kWThreads - 1) / kWThreads;
        const T* w = (const T*)a.w_qkv + (long)h * 48 * a.C;
        u32x4 wp[kWPer];
#pragma unroll
        for (int j = 0; j < kWPer; ++j) {
            const int it = threadIdx.x + j * kWThreads, row = it / (KC * 4), c = it % (KC * 4) * 8;
            wp[j] = u32x4{0u, 0u, 0u, 0u};
            if (threadIdx.x < kWThreads && it < kPieces && c < a.C) wp[j] = *(const u32x4*)(w + (long)row * a.C + c);
        }
        fetch_x(0);
        __builtin_amdgcn_sched_barrier(0);
        if (threadIdx.x < kTapPieces) ((u32x4*)taps_lds)[threadIdx.x] = tap_piece;
#pragma unroll
        for (int j = 0; j < kWPer; ++j) {
            const int it = threadIdx.x + j * kWThreads;
            if (threadIdx.x < kWThreads && it < kPieces) *(u32x4*)(w_lds + it / (KC * 4) * L::kWPitch + it % (KC * 4) * 16) = wp[j];
        }
    } else {
        const unsigned q_tb = (unsigned)(a.q_ts * SZ), k_tb = (unsigned)(a.k_ts * SZ);
        const BufRsrc rq = make_rsrc((const T*)a.q + (long)h * a.q_hs + img_tok0 * a.q_ts, ((N - 1) * a.q_ts + 16) * (long)SZ);
        const BufRsrc rk = make_rsrc((const T*)a.k + (long)h * a.k_hs + img_tok0 * a.k_ts, ((N - 1) * a.k_ts + 32) * (long)SZ);
#pragma unroll
        for (int j = 0; j < L::kPer; ++j) {
            const int t = token(wave + kSmallWaves * j, x16);
            qf[j] = buf_load8(rq, t >= 0 ? (unsigned)t * q_tb + q * 4 * SZ : kOobOffset);
            xf[j][0] = buf_load16(rk, t >= 0 ? (unsigned)t * k_tb + q * 8 * SZ : kOobOffset, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (threadIdx.x < kTapPieces) ((u32x4*)taps_lds)[threadIdx.x] = tap_piece;
    }
    // everything else that comes from memory is requested here too
    Frag gpw[kScales][2];       // grouped 1x1 weights of Q and K as 16x16 operands: lane (o, q) holds w[o][4q..4q+3]
    Vec w_v[kScales][2];        // ... of V: row threadIdx.x % 16
    auto fetch_weights = [&](int i, const T* w_gpw) {
        const T* wgp = w_gpw + (long)h * 48 * 16;
#pragma unroll
        for (int t = 0; t < 2; ++t) gpw[i][t] = load_frag<T>(wgp + (t * 16 + x16) * 16 + q * 4);
#pragma unroll
        for (int v = 0; v < 2; ++v) w_v[i][v] = ((const Vec*)(wgp + (2 * 16 + x16) * 16))[v];
    };
    fetch_weights(0, (const T*)a.w_gpw);
    if constexpr (KSB > 0) fetch_weights(1, w_gpw_b);

    Frag ident, ones;
    Vec selk, selv;       // pick channel x16 out of the 32 contraction slots {K 0..15, V 0..15} of a K | V load
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        ident[r] = Tr::from_f32(x16 == q * 4 + r ? 1.0f : 0.0f);
        ones[r] = Tr::from_f32(1.0f);
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        selk[r] = Tr::from_f32(q * 8 + r == x16 ? 1.0f : 0.0f);
        selv[r] = Tr::from_f32(q * 8 + r == 16 + x16 ? 1.0f : 0.0f);
    }
    __syncthreads();        // filter taps and weights are in LDS

    auto toeplitz = [&](auto ks, auto& toep, const char* taps) {
        constexpr int K2 = decltype(ks)::value;
#pragma unroll
        for (int t = 0; t < 3; ++t)
            make_toeplitz<T, K2, (KS - K2) / 2>(load_taps<T, K2>((const T*)taps, t * 16 + sweep_channel(lane)), lane & 3, toep[t]);
    };
    constexpr std::integral_constant<int, KSA> ks_a;
    constexpr std::integral_constant<int, kB> ks_b;
    Frag toep_a[3][KSA][2];
    if constexpr (!kTwo) toeplitz(ks_a, toep_a, taps_lds);
    f32x4 kv_raw = z, ks_raw4 = z, kv_agg[kScales];
    float ks_agg[kScales];
#pragma unroll
    for (int i = 0; i < kScales; ++i) {
        kv_agg[i] = z;
        ks_agg[i] = 0.f;
    }
#pragma unroll
    for (int first = 0; first < L::kPer; first += kHalf) {
    // Q, K, V of a group: lane (channel x16, q), tokens 4q .. 4q + 3 of it
    f32x4 d_all[kHalf][3], dq_all[kHalf];       // (dq_all: Q the other way round, lane (token x16, q) with channels 4q .. 4q + 3)
    if constexpr (kProject) {
        if (first > 0) fetch_x(first);
        // (a weight operand is read once for all of a wave's groups)
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
#pragma unroll
            for (int t = 0; t < 3; ++t) d_all[j][t] = dq_all[j] = z;
#pragma unroll
        for (int s = 0; s < KC; ++s)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const Vec wf = *(const Vec*)(w_lds + (t * 16 + x16) * L::kWPitch + s * 64 + q * 16);
#pragma unroll
                for (int j = 0; j < kHalf; ++j)
                    if (first + j + 1 < L::kPer || wave + kSmallWaves * (first + j) < L::kGroups) {
                        d_all[j][t] = Tr::mma_vec(d_all[j][t], __builtin_bit_cast(Vec, xf[j][s]), wf);
                        if (t == 0) dq_all[j] = Tr::mma_vec(dq_all[j], wf, __builtin_bit_cast(Vec, xf[j][s]));
                    }
            }
        // the wait states between the last of these and whatever touches its registers next, written out: the compiler (ROCm 7.2) counts
        // one too many on the path on which a wave has no last group
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7");
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < kHalf; ++j) {
        const int g = wave + kSmallWaves * (first + j);
        if (g >= L::kGroups) break;
        f32x4(&d)[3] = d_all[j];
        if constexpr (!kProject) {
            const Vec kv = __builtin_bit_cast(Vec, xf[j][0]);
            d[0] = Tr::mma16(z, __builtin_bit_cast(Frag, qf[j]), ident);
            d[1] = Tr::mma_vec(z, kv, selk);
            d[2] = Tr::mma_vec(z, kv, selv);
        }
        const Frag dq = frag_from_f32<T>(d[0]), dk = frag_from_f32<T>(d[1]), dv = frag_from_f32<T>(d[2]);
        const int ly = at_row(g, 4 * q), lx = at_col(g, 4 * q);
        if (ly < L::LH) {
            char* dst = planar + x16 * L::kChanBytes + ly * kPlanarRowBytes + lx * SZ;
            store_frag<T>(dst, dq);
            store_frag<T>(dst + 16 * L::kChanBytes, dk);
            store_frag<T>(dst + 32 * L::kChanBytes, dv);
        }
        // the raw branch: the tile's own tokens
        Frag rk = frag_relu_bits<T>(dk);
        const bool own_row = ly >= P && ly < P + kTH;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (!own_row || lx + r < P || lx + r >= P + kTW) rk[r] = Tr::from_f32(0.f);
        if (kProject || a.do_raw) {
            ks_raw4 = Tr::mma16(ks_raw4, rk, ones);
            kv_raw = Tr::mma16(kv_raw, rk, dv);
        }
        if (kProject || a.copy_raw_q) {
            // raw Q, token-major: lane (token slot x16, q) with channels 4q .. 4q + 3
            const int t = own_token(g, x16);
            Frag out;
            if constexpr (kProject) out = frag_from_f32<T>(dq_all[j]);
            else out = __builtin_bit_cast(Frag, qf[j]);
            if (t >= 0) store_frag<T>(q_ms + (img_tok0 + t) * (long)a.S * Ct + h * 16 + q * 4, out);
        }
    }
    }
    if constexpr (kTwo) toeplitz(ks_a, toep_a, taps_lds);
    __syncthreads();        // the tile is staged
    // ---------------- the sweep: strip wave % 2, rows 2 * (wave / 2) and the next
    auto sweep = [&](auto ks, const auto& toep, int i, int branch) {
        constexpr int K2 = decltype(ks)::value, kOff = (KS - K2) / 2;
        const int strip = wave & 1, part = wave >> 1;
        const BufRsrc rout = make_rsrc(q_ms + img_tok0 * a.S * Ct + (long)branch * Ct + h * 16, ((N - 1) * a.S * Ct + 16) * (long)SZ);
        sweep_rows<T, K2, kRows, L::kChanBytes>(planar + (kRows * part + kOff) * kPlanarRowBytes + 16 * strip * SZ,
                                                w_lds + wave * 2 * kTransBytes, toep, gpw[i][0], gpw[i][1], a.H, a.W, ty0 + kRows * part,
                                                tx0 + 16 * strip, ty0 + kTH > a.H || tx0 + kTW > a.W, rout, q_ms_tb, kv_agg[i],
                                                ks_agg[i]);
    };
    sweep(ks_a, toep_a, 0, a.branch);
    if constexpr (KSB > 0) {
        Frag toep_b[3][kB][2];
        toeplitz(ks_b, toep_b, taps_lds + L::kTapsA);
        sweep(ks_b, toep_b, 1, branch_b);
    }

    // ---------------- workgroup partial state
#pragma unroll
    for (int i = 0; i < kScales; ++i) {
        ks_agg[i] += __shfl_xor(ks_agg[i], 16);
        ks_agg[i] += __shfl_xor(ks_agg[i], 32);
    }
    __syncthreads();   // tile memory is dead from here on
    float* const red = (float*)lds;
    // per wave: [which][lane] accumulator quads, then [which][16] Ksum; which 0, 1 = aggregated (V before
    // its grouped 1x1), the last = raw
    constexpr int kWhich = kScales + 1, kWaveFloats = kWhich * (256 + 16);
    float* const msum = red + kSmallWaves * kWaveFloats;        // [scale][16][16] summed pre-1x1 states of the aggregated branches
    static_assert((kSmallWaves * kWaveFloats + kScales * 256) * 4 <= L::kBytes, "reduction area");
    {
        float* mine = red + wave * kWaveFloats;
#pragma unroll
        for (int i = 0; i < kScales; ++i) {
            *(f32x4*)(mine + i * 256 + lane * 4) = kv_agg[i];
            if (q == 0) mine[kWhich * 256 + i * 16 + x16] = ks_agg[i];
        }
        *(f32x4*)(mine + kScales * 256 + lane * 4) = kv_raw;
        if (x16 == 0) *(f32x4*)(mine + kWhich * 256 + kScales * 16 + q * 4) = ks_raw4;
    }
    __syncthreads();
    auto put = [&](int which, int e, int f, float s) {
        const int branch = which == kScales ? 0 : which == 0 ? a.branch : branch_b;
        a.partials[((((long)b * a.S + branch) * a.heads + h) * a.nchunks + tile) * kStateSize + e * 17 + f] = s;
    };
    auto wave_sum = [&](int src) {      // fixed order
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) s += red[w * kWaveFloats + src];
        return s;
    };
    const int e = (threadIdx.x >> 4) & 15;
    {
        // Ksum beside the first of the thread's other sums, so that their reads are in flight together
        float s[(kWhich + 1) / 2], ksum = 0.f;
#pragma unroll
        for (int i = 0; i < (kWhich + 1) / 2; ++i) {
            const int which = 2 * i + (threadIdx.x >> 8);
            s[i] = wave_sum((which < kWhich ? which : 0) * 256 + ((e >> 2) * 16 + x16) * 4 + (e & 3));
        }
        if (threadIdx.x < kWhich * 16) ksum = wave_sum(kWhich * 256 + threadIdx.x);
#pragma unroll
        for (int i = 0; i < (kWhich + 1) / 2; ++i) {
            const int which = 2 * i + (threadIdx.x >> 8);
            if (which < kScales) msum[which * 256 + e * 16 + x16] = s[i];
            else if (which == kScales && a.do_raw) put(which, e, x16, s[i]);
        }
        const int which = threadIdx.x >> 4;
        if (which < kScales || (which == kScales && a.do_raw)) put(which, x16, 16, ksum);
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        // the grouped 1x1 of V, applied to the summed state: KV[e][f] = sum_c M[e][c] w_gpw[f][c]
#pragma unroll
        for (int i = 0; i < kScales; ++i) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < 16; ++c) s = fmaf(msum[i * 256 + e * 16 + c], Tr::to_f32(w_v[i][c >> 3][c & 7]), s);
            put(i, e, x16, s);
        }
    }
}

template <class T, int KSA, int KSB, int KC>
hipError_t run_small(const AggregateArgs& a, const AggregateArgs& second, hipStream_t stream) {
    constexpr int kLds = SLds<KSA, KSB, KC>::kBytes;
    const hipError_t e = allow_dynamic_lds<aggregate_small_kernel<T, KSA, KSB, KC>>(kLds);
    if (e != hipSuccess) return e;
    const long nblocks = ((long)a.B * a.heads * a.nchunks + 7) / 8 * 8;         // whole rounds over the XCDs
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((aggregate_small_kernel<T, KSA, KSB, KC>), dim3((unsigned)nblocks), dim3(kSmallThreads), kLds, stream, a,
                       (const T*)second.w_dw, (const T*)second.w_gpw, second.branch);
    return hipGetLastError();
}
template <class T, int KSA, int KSB>
hipError_t run_small_ks(const AggregateArgs& a, const AggregateArgs& second, hipStream_t stream) {
    if (a.w_qkv == nullptr) return run_small<T, KSA, KSB, 0>(a, second, stream);
    if (a.C <= 64) return run_small<T, KSA, KSB, 2>(a, second, stream);
    if (a.C <= 128) return run_small<T, KSA, KSB, 4>(a, second, stream);
    return run_small<T, KSA, KSB, 6>(a, second, stream);
}
// second: null for one scale
template <class T>
hipError_t run(const AggregateArgs& a, const AggregateArgs* second, hipStream_t stream) {
    const long tiles = (long)((a.H + kTH - 1) / kTH) * ((a.W + kTW - 1) / kTW);
    if (a.nchunks != tiles || a.tiles_per_chunk != 1) return hipErrorInvalidValue;
    // 32-bit byte offsets inside one image's maps
    long widest = (long)a.S * a.heads * 16;
    if (a.w_qkv != nullptr) {
        if (!a.do_raw || a.C <= 0 || a.C % 16 != 0 || a.C > kAggSmallMaxC) return hipErrorInvalidValue;
        widest = std::max(widest, (long)a.C);
    } else {
        // the kernel reads K and V of a token as one 32-channel run
        if ((const char*)a.v != (const char*)a.k + 16 * sizeof(T) || a.v_ts != a.k_ts || a.v_hs != a.k_hs) return hipErrorInvalidValue;
        widest = std::max(widest, std::max(a.q_ts, a.k_ts));
    }
    if ((long)a.H * a.W * widest * (long)sizeof(T) > 0x7fffffffL) return hipErrorNotSupported;
    if (second == nullptr) {
        if (a.ks == 3) return run_small_ks<T, 3, 0>(a, a, stream);
        if (a.ks == 5) return run_small_ks<T, 5, 0>(a, a, stream);
    } else {
        if (a.ks == 3 && second->ks == 5) return run_small_ks<T, 3, 5>(a, *second, stream);
        if (a.ks == 5 && second->ks == 3) return run_small_ks<T, 5, 3>(a, *second, stream);
    }
    return second ? hipErrorNotSupported : hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_aggregate_small(int dt, const AggregateArgs& a, const AggregateArgs* second, hipStream_t stream) {
    switch (dt) {
        case 1: return run<_Float16>(a, second, stream);
        case 2: return run<__bf16>(a, second, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace msla
