// The matrix-core aggregation's building blocks, shared by its kernels (k_aggregate_mfma.hip, k_aggregate_small.hip): the
// Toeplitz operands of the depthwise filters, and the sweep of a strip of a channel-planar halo tile down to aggregated Q tokens
// and the state.  What they compute and why it is done so is said at the top of k_aggregate_mfma.hip.
#pragma once
#include "msla_device.h"

namespace msla {

constexpr int kPlanarRowBytes = 72;                         // a tile row of one channel: 36 columns, 8-byte aligned
constexpr int kTransTokStride = 80;                         // transposition buffer: 16 tokens x 16 fp32 (+pad)
constexpr int kTransBytes = 16 * kTransTokStride;           // (a sweeping wave has two)

// Bytes from channel to channel of a halo tile of `rows` rows, an odd number of 8-byte slots (16 slots = all 32 banks).  A staging
// write puts 16 channels of one x-block side by side: 16 different slots mod 16.  A sweeping
// read covers, per 16 lanes, 4 x-blocks of the channels {g, g+4, g+8, g+12}: their strides are
// 0, 4, 8, 12 slots mod 16 (times an odd number), the x-blocks fill the gaps.
constexpr int planar_chan_bytes(int rows) { return rows * kPlanarRowBytes + (rows * kPlanarRowBytes / 8 % 2 == 0 ? 8 : 0); }

template <class T> struct M4;
template <> struct M4<_Float16> {
    static __device__ __forceinline__ f32x4 mma(f16x4 a, f16x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 0, 0, 0);
    }
};
template <> struct M4<__bf16> {
    static __device__ __forceinline__ f32x4 mma(bf16x4 a, bf16x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(i16x4, a), __builtin_bit_cast(i16x4, b), c,
                                                      0, 0, 0);
    }
};

// Compiler-level ordering of LDS traffic inside one wave (the hardware already
// executes a wave's LDS instructions in order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 4x4x4 block of a lane -> channel of the group: 16 consecutive lanes take channels 4 apart (LDS banks, see planar_chan_bytes)
__device__ __forceinline__ int sweep_channel(int lane) { return 4 * ((lane >> 2) & 3) + (lane >> 4); }

// One head's filter taps of a channel, KS * KS of them, as aligned words (channel `ch` of `wdw`, a copy in LDS; an odd channel starts
// in the middle of a word).  Word j of the result holds taps 2j and 2j + 1.
template <int KS>
struct TapWords {
    static constexpr int kTaps = KS, kWords = (KS * KS + 1) / 2;
    unsigned w[kWords];
};
template <class T, int KS>
__device__ __forceinline__ TapWords<KS> load_taps(const T* wdw, int ch) {
    typedef TapWords<KS> Tw;
    static_assert(Tw::kWords * 2 == KS * KS + 1, "an odd number of taps: the words of an odd channel end with it");
    const unsigned* p = (const unsigned*)(wdw + (ch * KS * KS & ~1));
    unsigned raw[Tw::kWords];
#pragma unroll
    for (int j = 0; j < Tw::kWords; ++j) raw[j] = p[j];
    Tw r;
    const unsigned pick = (ch & 1) ? 0x05040302u : 0x03020100u;
#pragma unroll
    for (int j = 0; j < Tw::kWords; ++j) r.w[j] = __builtin_amdgcn_perm(raw[j + 1 < Tw::kWords ? j + 1 : j], raw[j], pick);
    return r;
}

// Byte selector that puts taps 2j - s1 and 2j + 1 - s1 of a filter row into a word, out of the words par - 1 + j (the first
// tap of the row in its upper half if par) and the next; taps outside the row are 0.
constexpr unsigned band_selector(int KS, int par, int j, int s1) {
    unsigned sel = 0;
    for (int half = 0; half < 2; ++half) {
        const int tap = 2 * j + half - s1;
        unsigned two = 0x0c0cu;                                 // two zero bytes
        if (tap >= 0 && tap < KS) {
            const int word = (par + tap) / 2 - (par - 1 + j);   // 0 the earlier word, 1 the later
            const unsigned byte = 4u * word + 2u * ((par + tap) & 1);
            two = (byte + 1) << 8 | byte;
        }
        sel |= two << (16 * half);
    }
    return sel;
}

// The Toeplitz operands of one channel for output i = sub: toep[u][s][k] = w[u][4s + k - shift], shift = sub + kOff, i.e. each
// filter row shifted up by that many taps: by one in the byte selectors that cut the row out of the channel's words, by two and
// four in a choice of words.  kOff: the columns that the tile's halo has on each side beyond this filter's.
template <class T, int KS, int kOff = 0>
__device__ __forceinline__ void make_toeplitz(const TapWords<KS>& tw, int sub, typename Traits<T>::Frag (&toep)[KS][2]) {
    static_assert(KS + 2 * kOff <= 5, "a shifted row fits eight taps");
    const int shift = sub + kOff;
    const bool s1 = shift & 1, s2 = shift & 2, s4 = kOff > 0 && (shift & 4);
    static_for<0, KS>([&](auto uc) {
        constexpr int u = decltype(uc)::value, par = u * KS & 1, k = u * KS / 2;
        unsigned e[3];
        static_for<0, 3>([&](auto jc) {
            constexpr int j = decltype(jc)::value, lo = k + par - 1 + j, last = TapWords<KS>::kWords - 1;
            constexpr unsigned sel0 = band_selector(KS, par, j, 0), sel1 = band_selector(KS, par, j, 1);
            e[j] = sel0 == 0x0c0c0c0cu && sel1 == 0x0c0c0c0cu
                       ? 0u
                       : __builtin_amdgcn_perm(tw.w[lo + 1 < last ? lo + 1 : last], tw.w[lo < 0 ? 0 : lo < last ? lo : last], s1 ? sel1 : sel0);
        });
        const u32x2 f0 = {s2 ? 0u : e[0], s2 ? e[0] : e[1]}, f1 = {s2 ? e[1] : e[2], s2 ? e[2] : 0u};
        toep[u][0] = __builtin_bit_cast(typename Traits<T>::Frag, s4 ? u32x2{0u, 0u} : f0);
        toep[u][1] = __builtin_bit_cast(typename Traits<T>::Frag, s4 ? f0 : f1);
    });
}

// The sweep of one wave: 16 columns x R rows of a tile whose halo lies in LDS, channel by channel, Q, K, V.  (The zeros around
// a filter's taps are multiplied too: a Q that is not finite makes the aggregated Q of tokens up to five columns away NaN, in whose branch the
// rectifier then finds nothing, where the filter alone would reach KS / 2.)  `rows` points at
// the strip's first input row and column; gy0, gx_first are the image row and column of its first output; rout covers
// this head's channels of the branch in the image's Q map.  `ragged` (wave-uniform): some of the tile lies outside the image.
// Adds to the state: kv_agg (V before its grouped 1x1), ks_agg.
template <class T, int KS, int R, int kChanBytes>
__device__ __forceinline__ void sweep_rows(const char* rows, char* trans, const typename Traits<T>::Frag (&toep)[3][KS][2],
                                           typename Traits<T>::Frag gpw_q, typename Traits<T>::Frag gpw_k, int H, int W, int gy0,
                                           int gx_first, bool ragged, BufRsrc rout, unsigned q_ms_tb, f32x4& kv_agg, float& ks_agg) {
    typedef Traits<T> Tr;
    typedef typename Tr::Frag Frag;
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4;      // 16x16 MFMA view of the lane
    const int sub = lane & 3;      // 4x4x4 view: row/column inside a block
    const int chn = sweep_channel(lane);
    const int gx0 = gx_first + 4 * sub;               // image column of this lane's x-block
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    Frag aggK[R], aggK_lo[R];
    // The three passes (K, V, Q) form one flat, fully unrolled sequence of input rows.  A finished
    // output row goes through three stages in three consecutive iterations, so that no stage
    // waits for the one before it: (1) hand the row to LDS for transposition (K, Q) or to the
    // lane permutation (V); (2) pick it up in operand layout and issue the grouped-1x1 / state
    // MFMA; (3) rectify, pack, store.  Two transposition buffers alternate.
    constexpr int NR = R + KS - 1;
    f32x4 acc[KS];
    Frag s1v[2][2];                   // V (hi, lo) after the lane permutation
    f32x4 s2v[2];                     // MFMA results awaiting stage 3
    u32x2 q_held = {0u, 0u};          // an even Q row awaiting its partner
    auto pass_t = [](int pass) { return pass == 0 ? 1 : pass == 1 ? 2 : 0; };     // K, V, Q
    // A finished row sits as lane (channel chn, x-block sub) = 4 tokens of one channel.  It is
    // rounded to the operand type first (hi and lo halves for bf16), so everything that moves is
    // 8 bytes per lane.
    auto stage1 = [&](int it, f32x4 o) {
        const int t = pass_t(it / NR), y = it % NR - (KS - 1);
        const int gy = gy0 + y;
        // the wait states between a 4x4x4 matrix instruction and a reader of its result, written out: the compiler (ROCm
        // 7.2) leaves them out on the path that jumps over the masking below (bf16, paired launch)
        if (t == 1) asm volatile("s_nop 4" : "+v"(o));
        if (t == 1 && ragged) {
            // tokens outside the image contribute nothing: their aggregated K is made 0, which
            // also removes their V from the state; Q rows of such tokens are simply not stored.
            // (Only a tile that sticks out of the image has such tokens.)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (gy >= H || gx0 + i >= W) o[i] = 0.f;
        }
        Frag hi, lo;
        if constexpr (Tr::kHiLo) frag_split<T>(o, hi, lo);
        else hi = frag_from_f32<T>(o);
        if (t == 2) {
            // V: lane (channel c, q) <- the lane that swept channel c, x-block q: tokens (x-block q, i),
            // the K operand's order
            const int from = 4 * (4 * (x16 & 3) + (x16 >> 2)) + q;
            const u32x2 h2 = __builtin_bit_cast(u32x2, hi);
            s1v[it & 1][0] = __builtin_bit_cast(Frag, u32x2{(unsigned)__shfl((int)h2[0], from),
                                                            (unsigned)__shfl((int)h2[1], from)});
            if constexpr (Tr::kHiLo) {
                const u32x2 l2 = __builtin_bit_cast(u32x2, lo);
                s1v[it & 1][1] = __builtin_bit_cast(Frag, u32x2{(unsigned)__shfl((int)l2[0], from),
                                                                (unsigned)__shfl((int)l2[1], from)});
            }
        } else {
            // K, Q: the lane's 4 tokens of one channel go into a [token][channel] fp32 matrix; stage 2
            // picks up a token's 4 channels with one 16-byte read
            char* tb = trans + (it & 1) * kTransBytes;
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 4; ++i) *(float*)(tb + (4 * sub + i) * kTransTokStride + chn * 4) = o[i];
            wave_lds_fence();
        }
    };
    // Stage 2 is split: the transposed row is requested from LDS at the top of an iteration and
    // used after the iteration's depthwise MFMAs, which cover the LDS latency.
    auto stage2_read = [&](int it) {
        const char* tb = trans + (it & 1) * kTransBytes;
        return *(const f32x4*)(tb + x16 * kTransTokStride + q * 16);
    };
    auto stage2 = [&](int it, f32x4 tq) {
        const int t = pass_t(it / NR), y = it % NR - (KS - 1);
        if (t == 2) {
            if constexpr (Tr::kHiLo) {
                kv_agg = Tr::mma16(kv_agg, aggK[y], s1v[it & 1][0]);
                kv_agg = Tr::mma16(kv_agg, aggK[y], s1v[it & 1][1]);
                kv_agg = Tr::mma16(kv_agg, aggK_lo[y], s1v[it & 1][0]);
            } else {
                kv_agg = Tr::mma16(kv_agg, aggK[y], s1v[it & 1][0]);
            }
            return;
        }
        // The depthwise sums of Q always go to the grouped 1x1 as hi + lo pairs, whatever the
        // storage type: which components of the aggregated Q pass the rectifier of Eq. (2) is a
        // discrete decision, so that Q must carry the accuracy of its fp32 sums up to the one
        // rounding of its store (a sum rounded to 11 bits first moves a component that is small
        // against its 16 terms across zero).  K only feeds the sums of Eq. (3), which are
        // continuous in it: fp16 takes its depthwise sums rounded once.
        Frag dwf, dwf_lo;
        if (Tr::kHiLo || t == 0) frag_split<T>(tq, dwf, dwf_lo);
        else dwf = frag_from_f32<T>(tq);
        if (t == 1) {
            f32x4 kf = Tr::mma16(z, dwf, gpw_k);
            if constexpr (Tr::kHiLo) kf = Tr::mma16(kf, dwf_lo, gpw_k);
            s2v[it & 1] = kf;
        } else {
            f32x4 qq = Tr::mma16(z, gpw_q, dwf);
            qq = Tr::mma16(qq, gpw_q, dwf_lo);
            s2v[it & 1] = qq;
        }
    };
    auto stage3 = [&](int it) {
        const int t = pass_t(it / NR), y = it % NR - (KS - 1);
        if (t == 1) {
            const f32x4 kf = relu_bits_f32(s2v[it & 1]);       // Eq. (2): relu(K), one integer max per value
            ks_agg += (kf[0] + kf[1]) + (kf[2] + kf[3]);
            if constexpr (Tr::kHiLo) frag_split<T>(kf, aggK[y], aggK_lo[y]);
            else aggK[y] = frag_from_f32<T>(kf);
        } else if (t == 0) {
            // lane (token x16 = 4*xblock + i, q): channels 4q..4q+3 of image row gy0 + y, 8 bytes.
            // Two rows share one store (a store instruction costs the same whatever its width): an
            // even row waits for the next one, then the odd 16-lane groups of the one are swapped
            // with the even groups of the other, which leaves lane (x16, q) with channels
            // 8*(q/2) .. +7 of its token in row y - 1 + q % 2.
            static_assert(R % 2 == 0, "Q rows are stored in pairs");
            const u32x2 v = __builtin_bit_cast(u32x2, frag_from_f32<T>(s2v[it & 1]));
            if (y % 2 == 0) {
                q_held = v;
            } else {
                const u32x2 s0 = __builtin_amdgcn_permlane16_swap(q_held[0], v[0], false, false);
                const u32x2 s1 = __builtin_amdgcn_permlane16_swap(q_held[1], v[1], false, false);
                const int gy = gy0 + y - 1 + (q & 1);
                const int gx = gx_first + x16;
                const unsigned off = (unsigned)(gy * W + gx) * q_ms_tb + (q >> 1) * 8 * (unsigned)sizeof(T);
                buf_store16(rout, gy < H && gx < W ? off : kOobOffset, u32x4{s0[0], s1[0], s0[1], s1[1]});
            }
        }
    };
    // input row i of the flat sequence: 8 columns (two k-steps) of this lane's channel and x-block
    Frag din[2][2];
    auto fetch_row = [&](int i, Frag (&d)[2]) {
        const int t = pass_t(i / NR), r = i % NR;
        const char* src = rows + (t * 16 + chn) * kChanBytes + r * kPlanarRowBytes + sub * 8;
        d[0] = load_frag<T>(src);
        d[1] = load_frag<T>(src + 8);
    };
    fetch_row(0, din[0]);
    static_for<0, 3 * NR + 2>([&](auto it_c) {
        constexpr int it = decltype(it_c)::value;
        // iteration i finishes an output row iff it is the KS-th or a later input row of its pass
        constexpr auto has_row = [](int i) { return i >= 0 && i < 3 * NR && i % NR >= KS - 1; };
        constexpr bool kPickUp = has_row(it - 1) && ((it - 1) / NR != 1);     // K or Q row in the transposition buffer
        // LDS requests first: the next input row and the row handed over one iteration ago
        if constexpr (it + 1 < 3 * NR) fetch_row(it + 1, din[(it + 1) & 1]);
        f32x4 tq = z;
        if constexpr (kPickUp) tq = stage2_read(it - 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (it < 3 * NR) {
            const int pass = it / NR, r = it % NR;
            const int t = pass_t(pass);
            if (r == 0) {
#pragma unroll
                for (int i = 0; i < KS; ++i) acc[i] = z;
            }
#pragma unroll
            for (int u = 0; u < KS; ++u) {
                const int y = r - u;
                if (y < 0 || y >= R) continue;
                acc[y % KS] = M4<T>::mma(toep[t][u][0], din[it & 1][0], acc[y % KS]);
                acc[y % KS] = M4<T>::mma(toep[t][u][1], din[it & 1][1], acc[y % KS]);
            }
        }
        if constexpr (has_row(it - 1)) stage2(it - 1, tq);
        if constexpr (has_row(it - 2)) stage3(it - 2);
        if constexpr (has_row(it)) {
            // output row y of 16 channels x 16 tokens is complete: lane (channel chn, x-block sub)
            // holds the 4 tokens gx0..gx0+3 of image row gy0 + y
            const int y = it % NR - (KS - 1);
            const f32x4 o = acc[y % KS];
            acc[y % KS] = z;
            stage1(it, o);
        }
    });
}

}  // namespace msla
