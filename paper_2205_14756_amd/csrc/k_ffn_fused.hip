// The FFN+DWConv half of the building block (see k_ffn.hip for the operation) as ONE kernel, 16-bit storage types and up to
// 256 channels: the expanded map h = act(W1 y) is made where it is used and never reaches memory.
//
// A workgroup owns a block of TR x 16 tokens of one image and all output channels, and walks over slabs of 32 hidden channels.
// Its waves have three jobs, all of a step at once:
//   expand (4 waves)     h of slab i+2 on the block's halo of (TR + 2) x 18 tokens, whose y they hold as matrix operands in
//                        registers: matrix instructions, activation, one rounding -> halo planes in LDS
//   depthwise (8 or 4)   slab i+1 from its halo planes: vector ALU, activation, one rounding -> token tile in LDS
//   project (4 waves)    slab i: matrix instructions on the token tile, sums in registers; they also send out the loads of the
//                        weights, memory -> LDS, two steps ahead
// Halo planes and token tiles are double-buffered, one barrier ends a step.  The roundings and the order of every sum are those of
// the two launches, so results agree bit for bit.
//
// What it saves is the expanded map (134 MB written and 1.4 times read on the headline map) and a launch; what it pays is the
// expansion of the halo, 1.5 times (blocks of 128 tokens) or 2 times the products.  8 x 8192 tokens, 256 -> 1024 channels, fp16 132 ->
// 106 us on several input sets in turn, 110 -> 106 on one, whose expanded map stays in the memory-side cache, 122 -> 122 for a call
// alone on an idle GPU; 8192 tokens, 128 -> 512 channels 17.2 -> 14.4 (alone 19.8 -> 17.5).  Where it loses: see ffn_block_rows.
// Bound by the waves' own instruction streams: a wave alone on its SIMD's issue port sends a vector instruction every 8.5 cycles, and
// a step of the headline map (2500 cycles, of which 1280 of the matrix pipe) takes the depthwise waves 1400, the expanding ones 1160
// and the projecting ones 600 when each is alone.  Before the jobs were given to different waves the same map took 156 us (eight
// waves that did all three), with the weights through registers, requested one step ahead, 297.
#include "msla_device.h"
#include "msla_kernels.h"

namespace msla {
namespace {

// KC: 32-channel chunks of the input (C <= 32 * KC).  BR: output channels (C <= BR).  ND: depthwise waves (4 or 8).
template <int KC_, int TR_, int BR_, int ND_>
struct FfnFused {
    static constexpr int KC = KC_, TR = TR_, BR = BR_, ND = ND_;
    static constexpr int kThreads = (8 + ND) * 64;
    static constexpr int TB = TR * 16;                       // tokens of a block
    static constexpr int kHaloW = 18, kHaloH = TR + 2, kHaloTok = kHaloW * kHaloH;
    static constexpr int NG = (kHaloTok + 63) / 64;          // 16-token groups of the halo a wave expands (four quarters)
    static constexpr int BK = 32;                            // hidden channels of a slab
    static constexpr int kRing = 3;                          // slabs of weights in LDS
    static constexpr int kChunks1 = KC * 4;                  // 16-byte chunks of a W1 row
    static constexpr int kW1 = BK * kChunks1 * 16, kW1Vec = BK * kChunks1 / 256;      // vectors a staging thread
    static constexpr int kW2 = BR * 64, kW2Vec = BR * 4 / 256;
    static constexpr int CH = ND == 8 && TR == 4 ? 4 : 8;    // depthwise: channels and rows of a lane
    static constexpr int RPL = TR * 8 / (ND * CH);
    static constexpr int kPlane = NG * 64 * 16 + 16;         // one 8-channel vector of the halo (whole groups; padded for the banks)
    static constexpr int kHalo = 4 * kPlane;
    static constexpr int kTok = TB * 64;
    // LDS: the first slab of W2, the ring of W1, the rest of the ring of W2, halo planes, token tiles.  Before the first slab the
    // halo of y lies from the third slot of W1 on; in the end the sums lie over everything, one padded fp32 row a token.
    static constexpr int kW1At = kW2, kW2At = kW1At + kRing * kW1, kHaloAt = kW2At + (kRing - 1) * kW2;
    static constexpr int kYAt = kW1At + 2 * kW1, kYVec = kHaloTok * kChunks1;
    static constexpr int kSumRow = BR * 4 + 16;
    static constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
    // with four depthwise waves: each wave's filter taps of a slab, a ring of its own
    static constexpr int kTapVec = 9, kTapSlot = ND == 4 ? ND * kTapVec * 16 : 0;
    static constexpr int kTapAt = max3(kHaloAt + 2 * (kHalo + kTok), kYAt + (kYVec + 63) / 64 * 1024, 0);
    static constexpr int kLds = max3(kTapAt + kRing * kTapSlot, TB * kSumRow, 0);
    static constexpr int w2_slot(int slot) { return slot == 0 ? 0 : kW2At + (slot - 1) * kW2; }
    static constexpr int kInFlight = kW1Vec + kW2Vec;        // loads a project wave sends out in a step
    static constexpr int IO = BR / 64, JT = TB / 16;         // project: a wave has a quarter of the channels and all tokens
    // LDS chunk of a W1 row's chunk: sixteen rows of one chunk meet sixteen 16-byte slots mod 256
    static __device__ __forceinline__ int w1_at(int row, int chunk) { return row * (kChunks1 * 16) + (chunk ^ (row & 15)) * 16; }
    // ... and of the 64-byte rows of W2 and of the token tile
    static __device__ __forceinline__ int row64_at(int row, int chunk) { return row * 64 + (chunk ^ ((row >> 2) & 3)) * 16; }
    static_assert(kLds <= 160 * 1024 && KC % 4 == 0 && BR % 128 == 0 && (TR == 4 || TR == 8) && (ND == 4 || ND == 8), "");
};

// 16 bytes a lane from a buffer straight into LDS at lds_at + 16 * lane (a lane out of range writes zeros).  lds_at is
// wave-uniform.  The compiler does not know of these loads: whoever reads the data waits for them himself (wait_loads).  Nor
// does it see that they read scalar registers, which needs five wait states behind a vector instruction that wrote one (as where
// a spilled resource comes back) and one behind a write of m0: the s_nop is these.
typedef u32x4 RawRsrc;
__device__ __forceinline__ RawRsrc raw_rsrc(const void* base, long bytes) {
    const unsigned long a = (unsigned long)base;
    return RawRsrc{(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a),
                   (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)(a >> 32) & 0xffffu)),
                   (unsigned)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}
__device__ __forceinline__ void load_to_lds(RawRsrc r, unsigned voffset, unsigned lds_at) {
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voffset), "s"(r), "{m0}"(lds_at) : "memory");
}
// ... four of them for one such wait: v0 and v1 to lds_at and kStep further on, v2 and v3 of another buffer to lds_at2 and kStep further on
template <int kStep>
__device__ __forceinline__ void load_four_to_lds(RawRsrc r, unsigned v0, unsigned v1, unsigned lds_at, RawRsrc r2, unsigned v2, unsigned v3,
                                                 unsigned lds_at2) {
    asm volatile(
        "s_nop 4\n\tbuffer_load_dwordx4 %1, %5, 0 offen lds\n\ts_add_u32 m0, m0, %8\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %5, 0 offen lds\n\t"
        "s_mov_b32 m0, %7\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %6, 0 offen lds\n\ts_add_u32 m0, m0, %8\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %4, %6, 0 offen lds"
        : "+{m0}"(lds_at)
        : "v"(v0), "v"(v1), "v"(v2), "v"(v3), "s"(r), "s"(r2), "s"(lds_at2), "n"(kStep)
        : "memory", "scc");
}
template <int kLeft>
__device__ __forceinline__ void wait_loads_and_meet() {       // at most kLeft loads outstanding, LDS writes done, then the barrier
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kLeft) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void wait_lds_and_meet() {         // LDS reads and writes done, then the barrier
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// acc + t.half[TH] * h.half[HH] in fp32.  fp16 as the instruction that widens both halves itself: left to choose, the compiler
// converts some operands ahead and keeps them, and spills.
template <class T, bool kTapScalar, int TH, int HH>
__device__ __forceinline__ float fma_halves(uint32_t t, uint32_t h, float acc) {
    if constexpr (std::is_same<T, _Float16>::value) {
        if constexpr (kTapScalar)
            asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel:[%3,%4,0] op_sel_hi:[1,1,0]" : "+v"(acc) : "s"(t), "v"(h), "n"(TH), "n"(HH));
        else
            asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel:[%3,%4,0] op_sel_hi:[1,1,0]" : "+v"(acc) : "v"(t), "v"(h), "n"(TH), "n"(HH));
        return acc;
    } else {
        typedef T Pair __attribute__((ext_vector_type(2)));
        return fmaf(Traits<T>::to_f32(__builtin_bit_cast(Pair, t)[TH]), Traits<T>::to_f32(__builtin_bit_cast(Pair, h)[HH]), acc);
    }
}

template <class T, int ACT, class S>
__global__ __launch_bounds__(S::kThreads) void ffn_fused_kernel(const T* __restrict__ y, const T* __restrict__ w1,
                                                        const T* __restrict__ w_dw, const T* __restrict__ w2,
                                                        T* __restrict__ out, int H, int W, int C, int E, int tiles_x,
                                                        int tiles_y) {
    typedef Traits<T> Tr;
    typedef typename Tr::Vec Vec;
    constexpr int KC = S::KC, NG = S::NG, IO = S::IO, JT = S::JT, CH = S::CH, RPL = S::RPL, kHaloW = S::kHaloW;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* const ldsW1 = lds + S::kW1At;
    char* const ldsH = lds + S::kHaloAt;
    char* const ldsG = ldsH + 2 * S::kHalo;

    unsigned rest = xcd_remap(blockIdx.x, gridDim.x);
    const int tx = rest % tiles_x;
    rest /= tiles_x;
    const int ty = rest % tiles_y;
    const int b = rest / tiles_y;
    const int y0 = ty * S::TR, x0 = tx * 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4;
    const int n_slab = (E + 31) / 32;
    const unsigned c_bytes = (unsigned)C * 2u, e_bytes = (unsigned)E * 2u;
    // In step i W1 of slab i+2 and W2 of slab i are read; W1 of slab i+4 and W2 of slab i+2 are requested, two steps ahead of
    // their use, into the slots that were read in the step before.  Before step 0 come three shorter ones: the first loads,
    // slab 0 expanded, slab 1 expanded and the depthwise pass of slab 0.
    int s0 = 0, s1 = 1, s2 = 2;         // ring slots of slabs i, i+1, i+2
    auto next_slots = [&]() {
        const int t = s0;
        s0 = s1;
        s1 = s2;
        s2 = t;
    };

    const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) char*)lds;
    // All waves fetch the halo of y, rows as they lie in memory (as matrix operands straight from memory a load would cover sixteen
    // 64-byte pieces).  A token outside the image and channels past C read as zero.
    auto request_y = [&]() {
        const RawRsrc yres = raw_rsrc(y + (long)b * H * W * C, (long)H * W * c_bytes);
        for (int v0 = wave * 64; v0 < S::kYVec; v0 += S::kThreads) {
            const int t = (v0 + lane) / S::kChunks1, chunk = ((v0 + lane) % S::kChunks1) ^ (t & 15), hy = t / kHaloW, hx = t - hy * kHaloW;
            const int yy = y0 - 1 + hy, xx = x0 - 1 + hx;
            const bool ok = t < S::kHaloTok && yy >= 0 && yy < H && xx >= 0 && xx < W && chunk * 16 < (int)c_bytes;
            load_to_lds(yres, ok ? (unsigned)(yy * W + xx) * c_bytes + chunk * 16 : kOobOffset, lds0 + S::kYAt + v0 * 16);
        }
    };
    // The end, with the sums in LDS: the residual joins them, one rounding, whole rows leave.  A 16-token group is a row of the block.
    constexpr int kOutVec = S::TB * S::BR / 8, kOutIter = (kOutVec + S::kThreads - 1) / S::kThreads;
    const int rows = H - y0 < S::TR ? H - y0 : S::TR, cols = W - x0 < 16 ? W - x0 : 16;
    u32x4 res[kOutIter];
    auto out_at = [&](int j, int& tok, int& oc) {           // element offset of vector j of this thread, or -1
        const int v = (int)threadIdx.x + j * S::kThreads;
        tok = v / (S::BR / 8);
        oc = v % (S::BR / 8) * 8;
        if (v >= kOutVec || tok / 16 >= rows || tok % 16 >= cols || oc >= C) return -1L;
        return (((long)b * H + y0 + tok / 16) * W + x0 + tok % 16) * C + oc;
    };
    auto request_residual = [&]() {
#pragma unroll
        for (int j = 0; j < kOutIter; ++j) {
            int tok, oc;
            const long at = out_at(j, tok, oc);
            res[j] = u32x4{0u, 0u, 0u, 0u};
            if (at >= 0) res[j] = *(const u32x4*)(y + at);
        }
    };
    auto finish = [&]() {
#pragma unroll
        for (int j = 0; j < kOutIter; ++j) {
            int tok, oc;
            const long at = out_at(j, tok, oc);
            if (at < 0) continue;
            const f32x4 a0 = *(const f32x4*)(lds + tok * S::kSumRow + oc * 4), a1 = *(const f32x4*)(lds + tok * S::kSumRow + oc * 4 + 16);
            const Vec add = __builtin_bit_cast(Vec, res[j]);
            Vec o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] = Tr::from_f32(a0[e] + Tr::to_f32(add[e]));
                o[4 + e] = Tr::from_f32(a1[e] + Tr::to_f32(add[4 + e]));
            }
            *(u32x4*)(out + at) = __builtin_bit_cast(u32x4, o);
        }
    };

    if (wave < 4) {
        // ------------------------------------------------------------ expand
        request_y();
        wait_loads_and_meet<0>();
        // token group g of this wave's quarter of the halo, token (wave * NG + g) * 16 + x16, contraction slots 8q..8q+7 of each
        // chunk.  The h of a token outside the image is kept at zero (the convolution's padding).
        Vec xf[NG][KC];
        bool live[NG];
        int h_at[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int t = (wave * NG + g) * 16 + x16, hy = t / kHaloW, hx = t - hy * kHaloW;
            const int yy = y0 - 1 + hy, xx = x0 - 1 + hx, row = t < S::kHaloTok ? t : 0;
            live[g] = t < S::kHaloTok && yy >= 0 && yy < H && xx >= 0 && xx < W;
#pragma unroll
            for (int kk = 0; kk < KC; ++kk)
                xf[g][kk] = __builtin_bit_cast(Vec, *(const u32x4*)(lds + S::kYAt + S::w1_at(row, kk * 4 + q)));
            h_at[g] = (q >> 1) * S::kPlane + t * 16 + (q & 1) * 8;
        }
        wait_lds_and_meet();
        const bool inner = y0 > 0 && x0 > 0 && y0 + S::TR < H && x0 + 16 < W;      // (all of the halo is in the image)
        // a slab (W1 in `slot`) on this wave's halo tokens -> halo buffer `buf`
        auto expand = [&](int slot, int buf) {
            const char* wt = ldsW1 + slot * S::kW1;
            char* hd = ldsH + buf * S::kHalo;
            f32x4 h[2][NG];
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int g = 0; g < NG; ++g) h[o][g] = f32x4{0.f, 0.f, 0.f, 0.f};
            // weight fragments, read a few ahead of their use
            constexpr int kAhead = 3;
            Vec a[kAhead + 1];
            auto read = [&](auto n) {
                constexpr int kk = decltype(n)::value / 2, o = decltype(n)::value % 2;
                a[decltype(n)::value % (kAhead + 1)] = __builtin_bit_cast(Vec, *(const u32x4*)(wt + S::w1_at(o * 16 + x16, kk * 4 + q)));
            };
            static_for<0, kAhead>(read);
            static_for<0, 2 * KC>([&](auto n) {
                constexpr int kk = decltype(n)::value / 2, o = decltype(n)::value % 2;
                if constexpr (decltype(n)::value + kAhead < 2 * KC) read(std::integral_constant<int, decltype(n)::value + kAhead>{});
#pragma unroll
                for (int g = 0; g < NG; ++g) h[o][g] = Tr::mma_vec(h[o][g], a[decltype(n)::value % (kAhead + 1)], xf[g][kk]);
                __builtin_amdgcn_sched_barrier(0);
            });
            u32x2 v[2][NG];
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int g = 0; g < NG; ++g) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) h[o][g][r] = activate<ACT>(h[o][g][r]);
                    v[o][g] = __builtin_bit_cast(u32x2, frag_from_f32<T>(h[o][g]));
                }
            if (!inner)
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int g = 0; g < NG; ++g) v[o][g] = u32x2{live[g] ? v[o][g][0] : 0u, live[g] ? v[o][g][1] : 0u};
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int g = 0; g < NG; ++g) *(u32x2*)(hd + o * 2 * S::kPlane + h_at[g]) = v[o][g];
        };
        expand(0, 0);
        wait_loads_and_meet<0>();
        if (1 < n_slab) expand(1, 1);
        wait_loads_and_meet<0>();
        for (int i = 0; i < n_slab; ++i) {
            if (i + 2 < n_slab) expand(s2, i & 1);
            wait_loads_and_meet<0>();
            next_slots();
        }
        request_residual();
    } else if (wave < 8) {
        // ------------------------------------------------------------ project
        const int wp = wave - 4;
        // These waves also send out the loads of the weights: 16-byte vector v = wp * 64 + lane + 256 j of a tile of 32 rows of W1, of
        // BR rows' 64 bytes of W2.  Out of range (rows past the end, channels past C, hidden channels past E) reads as zero.
        const RawRsrc w1res = raw_rsrc(w1, (long)E * c_bytes), w2res = raw_rsrc(w2, (long)C * e_bytes);
        const unsigned lds_w = lds0 + wp * 1024;
        constexpr int kStep1 = 256 / S::kChunks1;       // W1 rows from one j to the next; 16 / kStep1 of them and the swizzle is back
        constexpr int kSame = 16 / kStep1 < S::kW1Vec ? 16 / kStep1 : S::kW1Vec;
        const int tid = wp * 64 + lane;
        unsigned g1[kSame];
#pragma unroll
        for (int j = 0; j < kSame; ++j) {
            const int v = tid + j * 256, row = v / S::kChunks1, chunk = (v % S::kChunks1) ^ (row & 15);
            g1[j] = chunk * 16 < (int)c_bytes ? (unsigned)row * c_bytes + chunk * 16 : kOobOffset;
        }
        const int k2 = ((tid & 3) ^ ((tid >> 4) & 3)) * 16;
        const unsigned g2 = (unsigned)(tid >> 2) * e_bytes + k2;
        auto at1 = [&](int slab, int j) { return g1[j % kSame] + (unsigned)(slab * 32 + j / kSame * 16) * c_bytes; };
        auto at2 = [&](int slab, int j) { return (slab * 64 + k2 < (int)e_bytes ? g2 + (unsigned)slab * 64u : kOobOffset) + (unsigned)(j * 64) * e_bytes; };
        auto request1 = [&](int slab, int slot) {
#pragma unroll
            for (int j = 0; j < S::kW1Vec; ++j) load_to_lds(w1res, at1(slab, j), lds_w + S::kW1At + slot * S::kW1 + j * 4096);
        };
        auto request2 = [&](int slab, int slot) {
#pragma unroll
            for (int j = 0; j < S::kW2Vec; ++j) load_to_lds(w2res, at2(slab, j), lds_w + S::w2_slot(slot) + j * 4096);
        };
        // W1 of one slab and W2 of another, a step's loads.  Up to 128 channels these are four and a step is short: one wait for all of them (the
        // building block of 8192 tokens, 128 channels, fp16 34.8-34.9 us, with no wait at all 34.9-35.0, with one each or one a pair 34.9-35.1;
        // the FFN alone 14.35, with none 14.25, with one each 14.4).
        auto request = [&](int slab1, int slot1, int slab2, int slot2) {
            if constexpr (S::kW1Vec == 2 && S::kW2Vec == 2) {
                load_four_to_lds<4096>(w1res, at1(slab1, 0), at1(slab1, 1), lds_w + S::kW1At + slot1 * S::kW1, w2res, at2(slab2, 0),
                                       at2(slab2, 1), lds_w + S::w2_slot(slot2));
            } else {
                request1(slab1, slot1);
                request2(slab2, slot2);
            }
        };
        request1(0, 0);
        request1(1, 1);
        request2(0, 0);
        request_y();
        f32x4 acc[IO][JT];
#pragma unroll
        for (int io = 0; io < IO; ++io)
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) acc[io][jt] = f32x4{0.f, 0.f, 0.f, 0.f};
        wait_loads_and_meet<0>();
        wait_loads_and_meet<0>();          // (the halo of y has been picked up)
        request1(2, 2);
        request2(1, 1);
        wait_loads_and_meet<S::kInFlight>();
        request1(3, 0);
        wait_loads_and_meet<S::kW1Vec>();
        for (int i = 0; i < n_slab; ++i) {
            request(i + 4, s1, i + 2, s2);
            const char* wt = lds + S::w2_slot(s0);
            const char* tok = ldsG + (i & 1) * S::kTok;
            Vec fa[IO];
#pragma unroll
            for (int io = 0; io < IO; ++io) fa[io] = __builtin_bit_cast(Vec, *(const u32x4*)(wt + S::row64_at((wp * IO + io) * 16 + x16, q)));
            constexpr int kAhead = 2;
            Vec fb[kAhead + 1];
            auto read = [&](auto jt) {
                fb[decltype(jt)::value % (kAhead + 1)] = __builtin_bit_cast(Vec, *(const u32x4*)(tok + S::row64_at(decltype(jt)::value * 16 + x16, q)));
            };
            static_for<0, kAhead>(read);
            static_for<0, JT>([&](auto jt) {
                constexpr int j = decltype(jt)::value;
                if constexpr (j + kAhead < JT) read(std::integral_constant<int, j + kAhead>{});
#pragma unroll
                for (int io = 0; io < IO; ++io) acc[io][j] = Tr::mma_vec(acc[io][j], fa[io], fb[j % (kAhead + 1)]);
                __builtin_amdgcn_sched_barrier(0);
            });
            wait_loads_and_meet<S::kInFlight>();
            next_slots();
        }
        wait_loads_and_meet<0>();          // (no load may reach the LDS any more)
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
            for (int io = 0; io < IO; ++io)
                *(f32x4*)(lds + (jt * 16 + x16) * S::kSumRow + ((wp * IO + io) * 16 + q * 4) * 4) = acc[io][jt];
        request_residual();
    } else {
        // ------------------------------------------------------------ depthwise
        // CH channels of RPL rows a lane, column x16.  The filter taps are the same for all lanes.  Eight waves keep them in scalar
        // registers, requested a slab ahead when the slab's LDS reads have arrived (any wait for an LDS read behind them would
        // wait for them as well; bf16 blocks of 128 tokens have too few of these registers, and the compiler keeps 102, with
        // hard-swish 38, in lanes of vector registers).  One wave a SIMD has no registers for two sets of eight channels, and no
        // other wave beside it to cover a request: those take them from LDS, where they arrive with the weights.
        constexpr bool kTapsInLds = S::kTapSlot > 0;
        const int wd = wave - 8, wq = wd & 3, part = wd >> 2;
        const int sub = CH == 4 ? part * 4 : 0, row0 = (CH == 4 ? 0 : part * 4) + q * RPL;
        const int ch0 = wq * 8 + sub;
        const RawRsrc tres = raw_rsrc(w_dw, (long)E * 18);
        auto request_taps = [&](int slab, int slot) {
            if (lane < S::kTapVec)
                load_to_lds(tres, (unsigned)(slab * 32 + ch0) * 18u + lane * 16, lds0 + S::kTapAt + slot * S::kTapSlot + wd * (S::kTapVec * 16));
        };
        constexpr int kTapWords = CH * 9 / 2;
        struct Taps {
            uint32_t w[kTapWords];
        };
        auto load_taps = [&](Taps& t, int s) {
            const int ch = s * 32 + ch0;
            const uint32_t* src = (const uint32_t*)(w_dw + (ch < E ? (long)ch * 9 : 0));       // (past E they are not used)
#pragma unroll
            for (int i = 0; i < kTapWords; ++i) t.w[i] = src[i];
        };
        const char* const h_lane = ldsH + wq * S::kPlane + (row0 * kHaloW + x16) * 16 + sub * 2;
        struct Px {
            uint32_t w[CH / 2];
        };
        // slab s, its taps in t, or in LDS at `slot`; `ahead` receives slab s+1's
        auto depthwise = [&](Taps& t, Taps& ahead, int slot, int s) {
            const char* hs = h_lane + (s & 1) * S::kHalo;
            Px f[RPL + 2][3], o[RPL];
#pragma unroll
            for (int r = 0; r < RPL + 2; ++r)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    __builtin_memcpy(&f[r][dx], __builtin_assume_aligned(hs + (r * kHaloW + dx) * 16, CH * 2), CH * 2);
            if constexpr (!kTapsInLds) {
                __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0)
                __builtin_amdgcn_sched_barrier(0);
                load_taps(ahead, s + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            // four channels at a time: with their taps in vector registers all eight do not fit
            constexpr int kPart = kTapsInLds ? 4 : CH;
#pragma unroll
            for (int j0 = 0; j0 < CH; j0 += kPart) {
                if constexpr (kTapsInLds) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = j0; i < j0 + 5; ++i)        // (words 0..17, then 18..35)
                        *(u32x4*)&t.w[4 * i] = *(const u32x4*)(lds + S::kTapAt + slot * S::kTapSlot + (wd * S::kTapVec + i) * 16);
                }
                float sum[RPL][kPart];
#pragma unroll
                for (int y = 0; y < RPL; ++y)
#pragma unroll
                    for (int j = 0; j < kPart; ++j) sum[y][j] = 0.f;
                static_for<0, (RPL + 2) * 3 * kPart>([&](auto n_c) {
                    constexpr int n = decltype(n_c)::value, j = n % kPart, dx = n / kPart % 3, r = n / kPart / 3;
                    static_for<0, RPL>([&](auto y_c) {
                        constexpr int y = decltype(y_c)::value;
                        if constexpr (r >= y && r < y + 3) {          // output row y: tap row r - y
                            constexpr int e = j * 9 + (r - y) * 3 + dx;      // (of this part's channels)
                            sum[y][j] = fma_halves<T, !kTapsInLds, e % 2, j % 2>(t.w[(j0 * 9 + e) / 2], f[r][dx].w[(j0 + j) / 2], sum[y][j]);
                        }
                    });
                });
#pragma unroll
                for (int y = 0; y < RPL; ++y)
#pragma unroll
                    for (int j = 0; j < kPart; j += 2) {
                        const typename Tr::elem pair[2] = {Tr::from_f32(activate<ACT>(sum[y][j])), Tr::from_f32(activate<ACT>(sum[y][j + 1]))};
                        __builtin_memcpy(&o[y].w[(j0 + j) / 2], pair, 4);
                    }
            }
#pragma unroll
            for (int y = 0; y < RPL; ++y) {
                if (s * 32 + ch0 >= E)
#pragma unroll
                    for (int j = 0; j < CH / 2; ++j) o[y].w[j] = 0u;
                char* to = ldsG + (s & 1) * S::kTok + S::row64_at((row0 + y) * 16 + x16, wq) + sub * 2;
                __builtin_memcpy(__builtin_assume_aligned(to, CH * 2), &o[y], CH * 2);
            }
        };
        Taps t0, t1;
        if constexpr (kTapsInLds) {
            request_taps(0, 0);
            request_taps(1, 1);
            request_taps(2, 2);
        } else {
            load_taps(t0, 0);
        }
        request_y();
        wait_loads_and_meet<0>();
        wait_loads_and_meet<0>();
        wait_loads_and_meet<0>();
        depthwise(t0, t1, 0, 0);
        wait_loads_and_meet<0>();
        for (int i = 0; i < n_slab; ++i) {
            if constexpr (kTapsInLds) {
                request_taps(i + 3, s0);
                if (i + 1 < n_slab) depthwise(t0, t0, s1, i + 1);
                wait_loads_and_meet<1>();
                next_slots();
            } else {
                if (i + 1 < n_slab) depthwise(t1, t0, 0, i + 1);
                wait_loads_and_meet<0>();
                if (++i >= n_slab) break;
                if (i + 1 < n_slab) depthwise(t0, t1, 0, i + 1);
                wait_loads_and_meet<0>();
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        request_residual();
    }
    if (wave < 4 || wave >= 8) wait_lds_and_meet();
    wait_lds_and_meet();
    finish();
}

template <class T, int ACT, class S>
hipError_t run_ffn_fused_as(const void* y, const void* w1, const void* w_dw, const void* w2, void* out, int B, int C, int H,
                            int W, int E, hipStream_t stream) {
    const int tiles_x = (W + 15) / 16, tiles_y = (H + S::TR - 1) / S::TR;
    const long nblocks = (long)B * tiles_x * tiles_y;
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    const hipError_t e = allow_dynamic_lds<ffn_fused_kernel<T, ACT, S>>(S::kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ffn_fused_kernel<T, ACT, S>), dim3((unsigned)nblocks), dim3(S::kThreads), S::kLds, stream, (const T*)y,
                       (const T*)w1, (const T*)w_dw, (const T*)w2, (T*)out, H, W, C, E, tiles_x, tiles_y);
    return hipGetLastError();
}

template <class T, int ACT>
hipError_t run_ffn_fused(bool small, const void* y, const void* w1, const void* w_dw, const void* w2, void* out, int B, int C, int H,
                         int W, int E, hipStream_t stream) {
    if (C <= 128)
        return small ? run_ffn_fused_as<T, ACT, FfnFused<4, 4, 128, 8>>(y, w1, w_dw, w2, out, B, C, H, W, E, stream)
                     : run_ffn_fused_as<T, ACT, FfnFused<4, 8, 128, 8>>(y, w1, w_dw, w2, out, B, C, H, W, E, stream);
    return small ? run_ffn_fused_as<T, ACT, FfnFused<8, 4, 256, 8>>(y, w1, w_dw, w2, out, B, C, H, W, E, stream)
                 : run_ffn_fused_as<T, ACT, FfnFused<8, 8, 256, 4>>(y, w1, w_dw, w2, out, B, C, H, W, E, stream);
}

}  // namespace

// One launch pays a round of workgroups, one a compute unit, and each slab in it, whatever share of its blocks' tokens and of their
// halo is in the image; the two launches pay for the expanded map -- its elements, and a pass over y for every 192 (256) of its
// channels -- and less a round.  So neither the number of rounds nor the fill of a block decides by itself: the time of the three
// forms is estimated.  The constants are fitted to 1100 shapes (32 tokens to 200 million elements of the expanded map, 16 to 256
// channels, 16 to 4096 hidden ones, rows of 1 to 4096 tokens), to calls in a row on several input sets in turn and on one: estimate /
// measured is 0.93 to 1.05 for nine shapes in ten, and the form taken is within 3 % of the best of the three at 99 in 100.
// Two launches / blocks of 64 tokens / of 128, us in turn (on one set):
//   full maps: fp16 8192 tokens, 128 -> 512 channels 17.2 / 14.4 / 19.0, 32768 29.9 / 28.4 / 20.6; 65536, 256 -> 1024 132 / 127 / 106
//     (110 / 126 / 106: the expanded map stays in the memory-side cache), bf16 136 / 134 / 115 (115 / 133 / 114);
//   blocks mostly outside the image: fp16 8 x 1 x 4096, 128 -> 512 71 / 101 / 138, 8 x 4096 x 1 228 / 413 / 284, 2048 images of 3 x 3
//     82 / 103 / 138; bf16 512 images of 7 x 7, 256 -> 1024 88 / 127 / 107;
//   many slabs for few workgroups: fp16 64 tokens, 128 -> 2048 35.6 / 42.1 / 57.3; bf16 1024, 128 -> 768 20.5 / 21.5 / 32.6;
//   more rounds of the smaller block: bf16 8 x 64 x 96, 256 -> 1024 (three or two) 118 / 102 / 112 (102 / 102 / 110).
// A call alone on an idle GPU runs before the clocks have risen, which costs this kernel more than the memory-bound two launches: 65536
// tokens, 256 -> 1024 take fp16 122 / 144 / 122 and bf16 127 / 157 / 136 there.
int ffn_block_rows(int dt, int B, int C, int H, int W, int E) {
    // 32-bit byte offsets into an image, each weight matrix and the filters
    const long lim = 0x7fffffffL;
    if (dt == 0 || C > 256 || (long)H * W * C * 2 >= lim || (long)C * E * 2 >= lim || (long)E * 18 >= lim) return 0;
    struct Form {
        // us: a call; a million tokens, a channel of y; a round; a slab in it (fp16, bf16), of 64 channels in the two launches, else of 32
        double call, channel, round, slab[2];
    };
    static const Form one4[2] = {{1.63, 0.43, 2.9, {0.593, 0.701}}, {1.64, 0.59, 3.4, {0.752, 0.851}}},      // up to 128 channels, more
                      one8[2] = {{1.24, 0.36, 4.2, {0.827, 1.13}}, {1.90, 0.58, 6.2, {1.20, 1.40}}},
                      two64[2] = {{6.1, 0.476, 1.7, {0.885, 1.07}}, {6.9, 0.879, 2.5, {1.05, 1.24}}},
                      two128[2] = {{6.1, 0.476, 3.0, {1.22, 1.45}}, {6.9, 0.879, 3.2, {1.61, 1.74}}},
                      two64_halves = {6.9, 0.879, 1.3, {0.97, 1.17}};        // (output channels in blocks of 128, see run_dw_project_split)
    const int wide = C > 128;
    const double m_tokens = 1e-6 * B * H * W;
    auto us = [&](const Form& f, long rounds, int slabs) { return f.call + f.channel * m_tokens * C + rounds * (f.round + slabs * f.slab[dt == 2]); };
    const FfnRounds r = ffn_rounds(B, H, W, 1);
    const double t4 = us(one4[wide], r.r4x16, (E + 31) / 32), t8 = us(one8[wide], r.r8x16, (E + 31) / 32);
    const int slabs64 = (E + 63) / 64, passes = E % 256 == 0 && E % 192 != 0 ? E / 256 : (E + 191) / 192;
    double two = m_tokens * (0.4 * E + 55.0 * passes);
    if (wide && 2 * r.b4x16 <= compute_units()) two += us(two64_halves, 1, slabs64);
    else if (r.r4x16 <= r.r8x16 && r.r4x16 <= r.r4x32) two += us(two64[wide], r.r4x16, slabs64);
    else two += us(two128[wide], r.r8x16 < r.r4x32 ? r.r8x16 : r.r4x32, slabs64);
    if (t4 > two && t8 > two) return 0;
    const int rows = t4 <= t8 ? 4 : 8;
    return (rows == 4 ? r.b4x16 : r.b8x16) * 1024 <= 0xffffffffL ? rows : 0;       // (a launch takes 32 bits of threads)
}

hipError_t launch_ffn_fused(int dt, const void* y, const void* w1, const void* w_dw, const void* w2, void* out, int B, int C,
                            int H, int W, int E, int act, hipStream_t stream) {
    const int rows = ffn_block_rows(dt, B, C, H, W, E);
    if (rows == 0) return hipErrorNotSupported;
    const bool small = rows == 4;
    if (dt == 1)
        return act == 0 ? run_ffn_fused<_Float16, 0>(small, y, w1, w_dw, w2, out, B, C, H, W, E, stream)
                        : run_ffn_fused<_Float16, 1>(small, y, w1, w_dw, w2, out, B, C, H, W, E, stream);
    return act == 0 ? run_ffn_fused<__bf16, 0>(small, y, w1, w_dw, w2, out, B, C, H, W, E, stream)
                    : run_ffn_fused<__bf16, 1>(small, y, w1, w_dw, w2, out, B, C, H, W, E, stream);
}

}  // namespace msla
