// Per-token normalise-and-apply of Eq. (3), last line:
//   att[n, m*16 + f] = relu(Q_n) . KV[:, f] / (relu(Q_n) . KV[:, 16] + eps)
// for every head-branch m = s*heads + h of the multi-scale Q map, either
// written out (the module without projections) or fed straight into the final
// 1x1 projection of the concatenated heads (Section 3.1, last sentence) so the
// attention map never reaches HBM.
//
// A 16-token x one-head-branch unit is two MFMAs: the state is the row operand
// (prepared by the finalize kernel, hi and lo halves stacked along the
// contraction for the 16-bit types), relu(Q) the column operand.  The second
// MFMA uses a row operand whose 16 rows all equal Ksum, so every lane gets the
// denominator of its own token without a shuffle.  The result has 4
// consecutive channels of one token per lane.
#include "gemm_tile.h"
#include "msla_kernels.h"

#ifndef MSLA_APPLY_W_AHEAD
#define MSLA_APPLY_W_AHEAD 3
#endif
#ifndef MSLA_APPLY_WR
#define MSLA_APPLY_WR 4
#define MSLA_APPLY_WC 2
#endif

namespace msla {
namespace {

// q: channels 4q..4q+3 of this lane's token (raw, not yet rectified).
// state: the 2048-byte operand block of (image, head-branch).  eps_s = eps * scale.
template <class T>
struct StateOps {
    u32x4 kv, ks;       // row operands: the state, and Ksum in every row
    float eps_s;
};
template <class T>
__device__ __forceinline__ StateOps<T> load_state_ops(const char* kvfrag, const float* kvscale, long sid, float eps,
                                                      bool live) {
    StateOps<T> s;
    s.kv = *(const u32x4*)(kvfrag + sid * 2048 + lane_id() * 16);
    s.ks = *(const u32x4*)(kvfrag + sid * 2048 + 1024 + lane_id() * 16);
    s.eps_s = live ? eps * kvscale[sid] : 0.f;
    return s;
}
template <class T>
__device__ __forceinline__ f32x4 att_unit(typename Traits<T>::Frag qf, const StateOps<T>& st) {
    typedef Traits<T> Tr;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    qf = frag_relu<T>(qf);
    f32x4 num, den;
    if constexpr (Tr::kSplit) {
        typedef typename Tr::Vec Vec;
        Vec b;
#pragma unroll
        for (int r = 0; r < 4; ++r) { b[r] = qf[r]; b[4 + r] = qf[r]; }   // pairs with {hi, lo}
        num = Tr::mma_vec(z, __builtin_bit_cast(Vec, st.kv), b);
        den = Tr::mma_vec(z, __builtin_bit_cast(Vec, st.ks), b);
    } else {
        num = Tr::mma16(z, __builtin_bit_cast(f32x4, st.kv), qf);
        den = Tr::mma16(z, __builtin_bit_cast(f32x4, st.ks), qf);
    }
    const float inv = 1.0f / (den[0] + st.eps_s);
    return f32x4{num[0] * inv, num[1] * inv, num[2] * inv, num[3] * inv};
}
// ------------------------------------------------------------------ att only
// A wave takes kApplyQuad neighbouring head-branches (128 contiguous bytes of a token's row in the 16-bit types: whole
// lines) of up to `gpw` groups of 16 tokens of one image; their state operands stay in registers and the next group's
// Q is requested before the current one is worked on.  Bound by memory (both maps once) where there are tokens
// enough; a wave that walked all head-branches of 16 tokens paid one load latency per head-branch instead (whole
// msla_core_forward: 2482 tokens, 54 head-branches, bf16 63.0 -> 37.4 us; 2204 tokens, 69, fp32 98.2 -> 45.7; 65536
// tokens, 32, fp16 123.4 -> 108.8; 1024 tokens, 8, fp16 18.8 -> 16.2).
constexpr int kApplyQuad = 4;
template <class T>
__global__ __launch_bounds__(256) void apply_kernel(const T* __restrict__ q_ms, const char* __restrict__ kvfrag,
                                                    const float* __restrict__ kvscale, T* __restrict__ att,
                                                    int N, int n_hb, int groups_per_image, int gpw, int runs_per_image,
                                                    long n_waves, float eps) {
    typedef typename Traits<T>::Frag Frag;
    const int n_quads = (n_hb + kApplyQuad - 1) / kApplyQuad;
    const long wid = (long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wid >= n_waves) return;
    const int quad = (int)(wid % n_quads);
    const long run = wid / n_quads;
    const int b = (int)(run / runs_per_image);
    const int g_begin = (int)(run % runs_per_image) * gpw;
    const int g_end = g_begin + gpw < groups_per_image ? g_begin + gpw : groups_per_image;
    const int x16 = lane_id() & 15, q = lane_id() >> 4;
    const int m0 = quad * kApplyQuad;
    const long ld = (long)n_hb * 16;
    const long col = (long)m0 * 16 + q * 4;

    StateOps<T> st[kApplyQuad];
#pragma unroll
    for (int j = 0; j < kApplyQuad; ++j) {
        const bool live = m0 + j < n_hb;
        st[j] = load_state_ops<T>(kvfrag, kvscale, (long)b * n_hb + (live ? m0 + j : 0), eps, live);
    }
    // (a token past the image's end reads its last one, a head-branch past the last the first: neither is stored)
    auto load = [&](int g, Frag (&f)[kApplyQuad]) {
        const int n = g * 16 + x16;
        const T* p = q_ms + ((long)b * N + (n < N ? n : N - 1)) * ld + col;
#pragma unroll
        for (int j = 0; j < kApplyQuad; ++j) f[j] = load_frag<T>(p + (m0 + j < n_hb ? j * 16 : -(long)m0 * 16));
    };
    Frag cur[kApplyQuad], next[kApplyQuad];
    load(g_begin, cur);
    for (int g = g_begin; g < g_end; ++g) {
        load(g + 1 < g_end ? g + 1 : g, next);
        const int n = g * 16 + x16;
        T* p = att + ((long)b * N + n) * ld + col;
#pragma unroll
        for (int j = 0; j < kApplyQuad; ++j) {
            const f32x4 o = att_unit<T>(cur[j], st[j]);
            if (n < N && m0 + j < n_hb) store_frag<T>(p + j * 16, frag_from_f32<T>(o));
            cur[j] = next[j];
        }
    }
}

// ------------------------------------------------- att fused into projection
// WC*64 tokens of one image x WR*64 output channels per workgroup, one wave per 64 x 64
// (128 tokens x 256 channels, 8 waves, unless the map is small).  Each
// iteration covers 128 contraction bytes = BK/16 head-branches; wave w makes
// the attention rows of token group w for them and writes them to the token
// tile in LDS while the weight tile arrives from the previous iteration's
// prefetch.  For bf16 the attention rows go to LDS as a hi and a lo tile (two
// MFMA passes), since 8 significant bits would cost half the error budget.
template <class T, int WR, int WC>
__global__ __launch_bounds__(WR * WC * 64) void apply_project_kernel(const T* __restrict__ q_ms,
                                                            const char* __restrict__ kvfrag,
                                                            const float* __restrict__ kvscale,
                                                            const T* __restrict__ w_proj, T* __restrict__ out,
                                                            int N, int n_hb, int c_out, int blocks_per_image,
                                                            int n_rb, float eps, const T* __restrict__ res) {
    typedef GemmTile<T, WR, WC> G;
    typedef typename Traits<T>::Frag Frag;
    constexpr int HB = G::BK / 16;   // head-branches per iteration
    constexpr int kWaves = G::kThreads / 64;
    constexpr int TG = (G::BC / 16) / kWaves;   // 16-token groups per wave for the attention rows
    static_assert(TG >= 1 && TG * kWaves * 16 == G::BC, "token groups must divide over the waves");
    constexpr bool kHiLo = Traits<T>::kHiLo;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* ldsR = lds;
    char* ldsC = lds + G::kLdsR;
    char* ldsC_lo = ldsC + G::kLdsC;   // only with kHiLo

    const unsigned L = xcd_remap(blockIdx.x, gridDim.x);
    const int rb = L % n_rb;
    const unsigned tb = L / n_rb;
    const int b = tb / blocks_per_image;
    const int n0 = (tb % blocks_per_image) * G::BC;
    const int oc0 = rb * G::BR;
    const int wave = threadIdx.x >> 6;
    const int wr = wave % WR, wc = wave / WR;
    const int x16 = lane_id() & 15, q = lane_id() >> 4;
    const int K = n_hb * 16;

    // this lane's tokens for the attention rows: token groups wave, wave + kWaves, ...
    bool ok[TG];
    const T* q_row[TG];
#pragma unroll
    for (int g = 0; g < TG; ++g) {
        const int n_mine = n0 + (g * kWaves + wave) * 16 + x16;
        ok[g] = n_mine < N;
        q_row[g] = q_ms + ((long)b * N + n_mine) * K + q * 4;
    }
    const long sid0 = (long)b * n_hb;

    f32x4 acc[4][4];
    G::zero(acc);
    u32x4 rw[G::kVecR];
    Frag qreg[TG][HB];
    // the state operands of a slab's head-branches are requested one slab ahead, like the weights
    StateOps<T> st[HB];
    auto fetch_states = [&](int m) {
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const bool live = m + j < n_hb;
            st[j] = load_state_ops<T>(kvfrag, kvscale, sid0 + (live ? m + j : 0), eps, live);
        }
    };
    G::load_global(rw, w_proj, oc0, c_out, K, 0, K);
    fetch_states(0);
#pragma unroll
    for (int g = 0; g < TG; ++g)
#pragma unroll
        for (int j = 0; j < HB; ++j)
            qreg[g][j] = (ok[g] && j < n_hb) ? load_frag<T>(q_row[g] + j * 16) : frag_zero<T>();

    for (int k0 = 0; k0 < K; k0 += G::BK) {
        G::store_lds_r(ldsR, rw);
        const int m0 = k0 >> 4;
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const bool live = m0 + j < n_hb;
#pragma unroll
            for (int g = 0; g < TG; ++g) {
                f32x4 o = {0.f, 0.f, 0.f, 0.f};
                if (live) o = att_unit<T>(qreg[g][j], st[j]);
                const int colb = (j * 16 + q * 4) * (int)sizeof(T);      // byte column inside the 128-byte slab
                const int off = ((g * kWaves + wave) * 16 + x16) * G::kRow + colb;
                if constexpr (kHiLo) {
                    Frag hi, lo;
                    frag_split<T>(o, hi, lo);
                    store_frag<T>(ldsC + off, hi);
                    store_frag<T>(ldsC_lo + off, lo);
                } else {
                    store_frag<T>(ldsC + off, frag_from_f32<T>(o));
                }
            }
        }
        __syncthreads();
        if (k0 + G::BK < K) {
            G::load_global(rw, w_proj, oc0, c_out, K, k0 + G::BK, K);
            const int m1 = m0 + HB;
            fetch_states(m1);
#pragma unroll
            for (int g = 0; g < TG; ++g)
#pragma unroll
                for (int j = 0; j < HB; ++j)
                    qreg[g][j] = (ok[g] && m1 + j < n_hb) ? load_frag<T>(q_row[g] + (m1 + j) * 16) : frag_zero<T>();
        }
        G::mma(acc, ldsR, ldsC, wr, wc);
        if constexpr (kHiLo) G::mma(acc, ldsR, ldsC_lo, wr, wc);
        __syncthreads();
    }
    const long tok0 = (long)b * N + n0;
    G::epilogue(acc, tok0, (long)b * N + N, oc0, c_out, wr, wc,
                [out, res, c_out](long tok, int oc, f32x4 v) {
                    if (res != nullptr) {
                        const f32x4 r = frag_to_f32<T>(load_frag<T>(res + tok * c_out + oc));
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += r[e];
                    }
                    store_frag<T>(out + tok * c_out + oc, frag_from_f32<T>(v));
                });
}

// ------------------------------------------- att fused into projection, weight-stationary
// The same fusion for a contraction of at most 512 slots (n_hb <= 2*KCH head-branches): a wave
// keeps the projection weights of its IO*16 output channels in registers for the whole kernel, and
// the (scaled) state operands of its own KCH/4 head-branches for as long as the image lasts.  A
// workgroup of 8 waves owns 8*IO*16 output channels and walks over tiles of 32 tokens of one image:
// every wave makes the attention rows of its head-branches for the tile -- two MFMAs per 16 tokens
// and head-branch -- and writes them to the tile in LDS; after the barrier every wave reads the
// whole tile as MFMA operands against its weights.
//
// fp16 runs this as one software pipeline with a single barrier per tile: while the matrix cores
// work through tile t (16 chunks of IO*2 MFMAs), the same instruction stream carries, dealt out
// between the chunks, the attention rows of tile t+1 (three stages per unit), the copy of the Q
// tile t+2 from registers to LDS, the request for Q tile t+3, and the stores of tile t-1's results.
// Measured with the shader clock, a period that keeps those jobs in blocks of their own around the
// MFMAs spends 60 % of its cycles outside the matrix instructions, all waves idling together.
// bf16 needs the LDS for the hi and lo tiles and keeps the phases apart (two barriers per tile).
//
// LDS tiles are [128-byte slab][token][128 bytes] without padding; the 16-byte chunk index of a row
// is XOR-ed with (row / 2) % 8, which keeps the 16-byte operand reads (16 consecutive rows of one
// chunk), the row-order copies (8 lanes per row) and the 8-byte attention accesses conflict-free.
template <class T, int KCH, int IO>
struct WsApply {
    static_assert(sizeof(T) == 2 && KCH % 4 == 0, "16-bit elements; whole head-branch quadruples");
    static constexpr bool kHiLo = Traits<T>::kHiLo;
    static constexpr int kWaves = 8, kThreads = 512;
    static constexpr int JT = 2, TB = JT * 16;           // tokens per tile
    static constexpr int HBW = KCH / 4;                  // head-branches per wave
    static constexpr int kUnits = JT * HBW;              // attention units per wave and tile
    static constexpr int kChanWave = IO * 16, kChanBlock = kWaves * kChanWave;
    static constexpr int NS = KCH / 2;                   // 128-byte slabs per attention row
    static constexpr int kRow = 128;
    static constexpr int kSlab = TB * kRow;
    static constexpr int kBuf = NS * kSlab;              // one attention tile or Q tile
    static constexpr int kQV = NS / 2;                   // 16-byte vectors per thread of a Q tile
    static constexpr int kWeightStage = kChanBlock * kRow;
    // bf16 keeps hi and lo attention tiles.  Where six tiles fit the LDS (up to 24 head-branches) it runs
    // the same single-barrier pipeline as fp16 with two hi, two lo and two Q tiles; beyond that, hi,
    // lo and one Q tile with the phases kept apart.
    static constexpr bool kPipeHiLo = kHiLo && 6 * kBuf <= 160 * 1024;
    static constexpr int kTiles = (kPipeHiLo ? 6 : 4) * kBuf;
    static constexpr int kLds = kTiles;
    static_assert(kWeightStage <= kTiles, "the weights are staged through the tile area");
    static_assert(NS % 2 == 0 && TB * 16 == kThreads, "the Q tile copy takes two slabs per pass");
    static_assert(KCH == 2 * kUnits, "one attention unit per two chunks of matrix instructions");
};

__device__ __forceinline__ int lds_swizzle(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// kOut: what becomes of the sums -- token-major rows, the same plus a residual, or a channel-planar map.  For the last the matrix
// instructions take their operands the other way round (tokens are the result's rows), so that a lane holds four tokens of one
// channel instead of four channels of one token: the module's result needs no transposition behind this kernel, and the
// sums are the same ones.
enum ApplyOut { kOutRows, kOutResidual, kOutPlanar };

template <class T, int KCH, int IO, ApplyOut kOut>
__global__ __launch_bounds__(512) void apply_project_ws_kernel(const T* __restrict__ q_ms,
                                                               const char* __restrict__ kvfrag,
                                                               const float* __restrict__ kvscale,
                                                               const T* __restrict__ w_proj, T* __restrict__ out,
                                                               int N, int n_hb, int c_out, int n_cg,
                                                               int tiles_per_image, long n_tt,
                                                               long tiles_per_block, float eps,
                                                               const T* __restrict__ res) {
    typedef WsApply<T, KCH, IO> S;
    typedef Traits<T> Tr;
    typedef typename Tr::Vec Vec;
    typedef typename Tr::Frag Frag;
    constexpr bool kHiLo = S::kHiLo, kPlanar = kOut == kOutPlanar;
    constexpr int kUnits = S::kUnits;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const unsigned L = xcd_remap(blockIdx.x, gridDim.x);
    const int cg = (int)(L % (unsigned)n_cg);
    const long t_begin = (long)(L / (unsigned)n_cg) * tiles_per_block;
    const long t_end = t_begin + tiles_per_block < n_tt ? t_begin + tiles_per_block : n_tt;
    if (t_begin >= t_end) return;
    const int n_mine = (int)(t_end - t_begin);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4;
    const int K = n_hb * 16;
    const unsigned row_bytes = (unsigned)K * 2u;
    const int ch0 = cg * S::kChanBlock + wave * S::kChanWave;

    // tile number -> (image, first token in it, that token's index in the whole map), walked with
    // counters: no division and no wide multiplication in the loop (the scalar unit runs a wave's
    // instructions one after the other, some eight cycles each)
    struct Origin {
        int b, n0;
        unsigned tok;
    };
    auto advance = [&](Origin o) {
        const int left = N - o.n0;                  // tokens of the image from this tile on
        o.tok += left < S::TB ? left : S::TB;
        if (left <= S::TB) { o.n0 = 0; ++o.b; }
        else o.n0 += S::TB;
        return o;
    };
    const Origin first = {(int)(t_begin / tiles_per_image), (int)(t_begin % tiles_per_image) * S::TB,
                          (unsigned)((t_begin / tiles_per_image) * N + (t_begin % tiles_per_image) * S::TB)};

    // ---- Q tile: copied in row order (8 lanes per 128-byte row segment; read as fragments straight
    // from memory every lane would touch its own row) into LDS.  Rows past the image's last token
    // and tiles past this workgroup's last read as zero.
    const int q_slab = threadIdx.x >> 8, q_row = (threadIdx.x >> 3) & 31, q_chunk = threadIdx.x & 7;
    const int q_lds = q_slab * S::kSlab + q_row * S::kRow + lds_swizzle(q_row, q_chunk) * 16;
    const unsigned q_glb = q_row * row_bytes + q_slab * 128 + q_chunk * 16;
    u32x4 qv[S::kQV];
    BufRsrc qres;
    auto aim_q = [&](Origin o, bool live) {
        const int rows = live ? (N - o.n0 < S::TB ? N - o.n0 : S::TB) : 0;
        qres = make_rsrc_small(q_ms + (size_t)o.tok * (unsigned)K, (unsigned)rows * row_bytes);
    };
    auto fetch_q1 = [&](int i) {
        qv[i] = buf_load16(qres, q_slab * 128 + q_chunk * 16 + i * 256 < row_bytes ? q_glb + i * 256 : kOobOffset, 0);
    };
    // Eq. (3) only ever sees relu(Q): the rectifier is applied here, once per element, as integer
    // maxima on the bit patterns (negative values and -0 have the sign bit set)
    auto park_q1 = [&](int qb, int i) {       // qb: byte offset of the Q tile in LDS
        typedef short i16x8 __attribute__((ext_vector_type(8)));
        const i16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        const i16x8 r = __builtin_elementwise_max(__builtin_bit_cast(i16x8, qv[i]), zero);
        *(u32x4*)(lds + qb + q_lds + 2 * i * S::kSlab) = __builtin_bit_cast(u32x4, r);
    };

    aim_q(first, true);      // requested ahead of the weights, so the first tile does not queue behind them
#pragma unroll
    for (int i = 0; i < S::kQV; ++i) fetch_q1(i);

    // ---- weights -> registers, copied in row order through LDS (fragment reads straight from
    // memory would touch one cache line per lane).  The registers the slabs wait in are the ones the
    // fragments move into.  The CU's address path needs longer for the 32 loads per thread than the
    // data takes to arrive, so the requests run kAheadW slabs ahead of the staging instead of all
    // being issued first: the staging of a slab then overlaps with the requests of the later ones.
    Vec wf[IO][KCH];
    const int g16 = (x16 >> 1) & 7;
    {
        const BufRsrc wres = make_rsrc(w_proj, (long)c_out * row_bytes);
        constexpr int kWV = S::kChanBlock * 8 / S::kThreads;      // vectors per thread and slab
        constexpr int kAheadW = S::NS < MSLA_APPLY_W_AHEAD ? S::NS : MSLA_APPLY_W_AHEAD;
        unsigned base[kWV];
        int wl[kWV];
#pragma unroll
        for (int i = 0; i < kWV; ++i) {
            const int r = (threadIdx.x + i * S::kThreads) >> 3;
            const int row = cg * S::kChanBlock + r;
            base[i] = row < c_out ? (unsigned)row * row_bytes + (threadIdx.x & 7) * 16 : kOobOffset;
            wl[i] = r * S::kRow + lds_swizzle(r, threadIdx.x & 7) * 16;
        }
        u32x4 wr[S::NS][kWV];
        auto request = [&](int sl) {
#pragma unroll
            for (int i = 0; i < kWV; ++i)
                wr[sl][i] = buf_load16(wres, (base[i] != kOobOffset && sl * 128 + (threadIdx.x & 7) * 16 < row_bytes)
                                                 ? base[i] + sl * 128 : kOobOffset, 0);
        };
#pragma unroll
        for (int sl = 0; sl < kAheadW; ++sl) request(sl);
#pragma unroll
        for (int sl = 0; sl < S::NS; ++sl) {
            if (sl) __syncthreads();
#pragma unroll
            for (int i = 0; i < kWV; ++i) *(u32x4*)(lds + wl[i]) = wr[sl][i];
            if (sl + kAheadW < S::NS) request(sl + kAheadW);
            __syncthreads();
#pragma unroll
            for (int io = 0; io < IO; ++io)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    wf[io][2 * sl + h] = __builtin_bit_cast(
                        Vec, *(const u32x4*)(lds + (wave * S::kChanWave + io * 16 + x16) * S::kRow + ((h * 4 + q) ^ g16) * 16));
        }
        __syncthreads();
    }

    // ---- this wave's head-branches: state operands and eps*scale, reloaded when the image changes
    Vec a_kv[S::HBW], a_ks[S::HBW];
    float eps_s[S::HBW];
    int img = -1;
    auto load_state = [&](int b) {
#pragma unroll
        for (int j = 0; j < S::HBW; ++j) {
            const int hb = wave * S::HBW + j;
            const long sid = (long)b * n_hb + (hb < n_hb ? hb : 0);
            a_kv[j] = __builtin_bit_cast(Vec, *(const u32x4*)(kvfrag + sid * 2048 + lane * 16));
            a_ks[j] = __builtin_bit_cast(Vec, *(const u32x4*)(kvfrag + sid * 2048 + 1024 + lane * 16));
            eps_s[j] = eps * kvscale[sid];
        }
        img = b;
    };

    // ---- attention rows of unit u = (jt, j) = 16 tokens x head-branch wave*HBW + j: Q tile ->
    // attention tile(s), a lane handling channels 4q..4q+3 of its token.  Three stages (request Q;
    // rectify and issue the two MFMAs; normalise and store) that the callers place in different
    // slots of their instruction stream, so no stage waits for the one before it.
    Frag att_q[2];
    f32x4 att_num, att_den;
    auto unit_off = [&](int u) {
        const int hb = wave * S::HBW + u % S::HBW;
        const int chunk = (hb & 3) * 2 + (q >> 1);
        return (hb >> 2) * S::kSlab + ((u / S::HBW) * 16 + x16) * S::kRow + (chunk ^ g16) * 16 + (q & 1) * 8;
    };
    auto att_a = [&](int qb, int u) { att_q[u & 1] = load_frag<T>((const T*)(lds + qb + unit_off(u))); };
    auto att_b = [&](int u) {
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        const Frag qf = att_q[u & 1];         // rectified when the tile was parked
        Vec b;
#pragma unroll
        for (int r = 0; r < 4; ++r) { b[r] = qf[r]; b[4 + r] = qf[r]; }   // pairs with {hi, lo} of the state
        att_num = Tr::mma_vec(z, a_kv[u % S::HBW], b);
        att_den = Tr::mma_vec(z, a_ks[u % S::HBW], b);
    };
    auto att_c = [&](int u, int hi_tile, int lo_tile) {
        const int hb = wave * S::HBW + u % S::HBW;
        const f32x4 num = att_num;
        const float inv = hb < n_hb ? __builtin_amdgcn_rcpf(att_den[0] + eps_s[u % S::HBW]) : 0.f;
        const f32x4 o = {num[0] * inv, num[1] * inv, num[2] * inv, num[3] * inv};
        const int off = unit_off(u);
        if constexpr (kHiLo) {
            Frag hi, lo;
            frag_split<T>(o, hi, lo);
            store_frag<T>(lds + hi_tile + off, hi);
            store_frag<T>(lds + lo_tile + off, lo);
        } else {
            store_frag<T>(lds + hi_tile + off, frag_from_f32<T>(o));
        }
    };
    // all units of a tile, the stages of neighbouring units overlapped
    auto att_all = [&](int qb, int hi_tile, int lo_tile) {
        att_a(qb, 0);
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            att_b(u);
            if (u + 1 < kUnits) att_a(qb, u + 1);
            att_c(u, hi_tile, lo_tile);
        }
    };

    // ---- projection: token-operand fragments are requested kAhead chunks ahead of their use (one
    // where the weights alone take half the register file)
    constexpr int kAhead = IO * KCH >= 32 ? 1 : 2;
    constexpr int kRing = kAhead + 1;
    f32x4 acc[IO][S::JT];
    const int frag_off = x16 * S::kRow + (q ^ g16) * 16;       // chunk (kk&1)*4 + q: the second half is ^ 64
    Vec bf[kRing][S::JT];
    Vec bl[S::kPipeHiLo ? kRing : 1][S::JT];          // the lo fragments of the pipelined hi/lo form
    auto read_b = [&](int tile, int kk) {
#pragma unroll
        for (int jt = 0; jt < S::JT; ++jt)
            bf[kk % kRing][jt] = __builtin_bit_cast(
                Vec, *(const u32x4*)(lds + tile + (frag_off ^ ((kk & 1) * 64)) + (kk >> 1) * S::kSlab + jt * 16 * S::kRow));
    };
    auto read_b_lo = [&](int tile, int kk) {
#pragma unroll
        for (int jt = 0; jt < S::JT; ++jt)
            bl[S::kPipeHiLo ? kk % kRing : 0][jt] = __builtin_bit_cast(
                Vec, *(const u32x4*)(lds + tile + (frag_off ^ ((kk & 1) * 64)) + (kk >> 1) * S::kSlab + jt * 16 * S::kRow));
    };
    auto mma = [&](int io, int jt, int kk, Vec tokens) {
        acc[io][jt] = kPlanar ? Tr::mma_vec(acc[io][jt], tokens, wf[io][kk]) : Tr::mma_vec(acc[io][jt], wf[io][kk], tokens);
    };
    auto mma_chunk = [&](int kk) {
#pragma unroll
        for (int io = 0; io < IO; ++io)
#pragma unroll
            for (int jt = 0; jt < S::JT; ++jt) mma(io, jt, kk, bf[kk % kRing][jt]);
    };
    auto mma_chunk_lo = [&](int kk) {
#pragma unroll
        for (int io = 0; io < IO; ++io)
#pragma unroll
            for (int jt = 0; jt < S::JT; ++jt) mma(io, jt, kk, bl[S::kPipeHiLo ? kk % kRing : 0][jt]);
    };
    auto zero_acc = [&]() {
#pragma unroll
        for (int io = 0; io < IO; ++io)
#pragma unroll
            for (int jt = 0; jt < S::JT; ++jt) acc[io][jt] = f32x4{0.f, 0.f, 0.f, 0.f};
    };

    // ---- results: finish() rounds a tile's accumulators into registers, a lane (token x16, q)
    // holding channels 4q..4q+3 of each 16-channel block: 8 bytes.  flush(p) writes piece p out with
    // one 16-byte store per lane: the odd 16-lane groups of one block are swapped with the even
    // groups of another, which leaves a lane with 8 consecutive channels -- of the two channel blocks
    // of 16 tokens (IO == 2: channels 16*(q%2) + 8*(q/2) .. +7 of token x16), or of one channel block
    // of both token groups (IO == 1: channels 8*(q/2) .. +7 of token 16*(q%2) + x16).  Planar: a lane (channel x16, q) holds
    // tokens 4q..4q+3 of each block, and the groups of both token blocks swapped leave it with tokens 16*(q%2) + 8*(q/2) .. +7.
    static_assert(IO == 1 || IO == 2, "two 8-byte halves per store");
    constexpr int kPieces = kPlanar ? IO : IO == 2 ? S::JT : S::JT / 2;
    Frag pend[IO][S::JT];
    BufRsrc ores;
    const unsigned out_row = (unsigned)c_out * 2u;
    // Planar: the map's rows start anywhere, which the stores take; a run of eight tokens that the image's end cuts leaves finish()
    // element by element.  (A branch between the matrix instructions made the widest variant spill 21 registers, and a module of
    // 8 x 53 x 67 tokens, 256 channels take 88.0 us instead of 84.9.)
    const int p_tok = (q & 1) * 16 + (q >> 1) * 8;
    const unsigned p_off = ((unsigned)x16 * (unsigned)N + p_tok) * 2u;
    int p_rows = 0;
    auto planar_at = [&](Origin o) { return out + ((size_t)(unsigned)o.b * (unsigned)c_out + ch0) * (unsigned)N + (unsigned)o.n0; };
    auto pair_up = [&](Frag a, Frag b) {
        const u32x2 even = __builtin_bit_cast(u32x2, a), odd = __builtin_bit_cast(u32x2, b);
        const u32x2 s0 = __builtin_amdgcn_permlane16_swap(even[0], odd[0], false, false);
        const u32x2 s1 = __builtin_amdgcn_permlane16_swap(even[1], odd[1], false, false);
        return u32x4{s0[0], s1[0], s0[1], s1[1]};
    };
    auto aim_out = [&](Origin o, bool live) {
        const int rows = live ? (N - o.n0 < S::TB ? N - o.n0 : S::TB) : 0;
        if constexpr (kPlanar) {
            const int live_io = ch0 >= c_out ? 0 : c_out - ch0 < IO * 16 ? 1 : IO;
            ores = make_rsrc_small(planar_at(o), (unsigned)live_io * 32u * (unsigned)N);      // (16 channels' rows each)
            p_rows = rows;
            return;
        }
        ores = make_rsrc_small(out + (size_t)o.tok * (unsigned)c_out, (unsigned)rows * out_row);
    };
    // (kOutResidual: out = res + ..., the residual joining the fp32 sums before their one rounding --
    // the block's y = x + MSLA(x); o is the origin of the tile the accumulators belong to)
    auto finish = [&](Origin o) {
#pragma unroll
        for (int io = 0; io < IO; ++io)
#pragma unroll
            for (int jt = 0; jt < S::JT; ++jt) {
                f32x4 v = acc[io][jt];
                if constexpr (kOut == kOutResidual) {
                    const int row = jt * 16 + x16, oc = ch0 + io * 16 + q * 4;
                    if (row < N - o.n0 && oc < c_out) {
                        const f32x4 r = frag_to_f32<T>(load_frag<T>(res + ((size_t)o.tok + row) * (unsigned)c_out + oc));
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += r[e];
                    }
                }
                pend[io][jt] = frag_from_f32<T>(v);
            }
        if constexpr (kPlanar) {
            const int rows = N - o.n0 < S::TB ? N - o.n0 : S::TB;
            if (rows % 8 != 0) {
                aim_out(o, true);
#pragma unroll
                for (int jt = 0; jt < S::JT; ++jt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int tok = jt * 16 + q * 4 + r;
                        const unsigned at = tok < rows && tok >= (rows & ~7) ? ((unsigned)x16 * (unsigned)N + tok) * 2u : kOobOffset;
#pragma unroll
                        for (int io = 0; io < IO; ++io)
                            buf_store2(ores, at + (unsigned)io * 32u * (unsigned)N, __builtin_bit_cast(u32x2, pend[io][jt])[r / 2] >> (r % 2 * 16));
                    }
            }
        }
    };
    auto flush = [&](int p) {
        if constexpr (kPlanar) {
            buf_store16(ores, p_tok + 8 <= p_rows ? p_off + (unsigned)p * 32u * (unsigned)N : kOobOffset, pair_up(pend[p][0], pend[p][1]));
            return;
        }
        const u32x4 v = IO == 2 ? pair_up(pend[0][p], pend[IO - 1][p]) : pair_up(pend[0][2 * p], pend[0][2 * p + 1]);
        const int row = IO == 2 ? p * 16 + x16 : (2 * p + (q & 1)) * 16 + x16;
        const int oc = ch0 + (IO == 2 ? (q & 1) * 16 : 0) + (q >> 1) * 8;
        buf_store16_stream(ores, oc < c_out ? (unsigned)row * out_row + oc * 2u : kOobOffset, v);
    };
    auto flush_all = [&](Origin o) {
        aim_out(o, true);
#pragma unroll
        for (int p = 0; p < kPieces; ++p) flush(p);
    };

    // the four tiles as byte offsets into LDS (plain numbers: a pointer chosen at run time would be
    // checked against null wherever something is added to it)
    constexpr int att0 = 0, att1 = S::kBuf, qb0 = 2 * S::kBuf, qb1 = 3 * S::kBuf;
    constexpr int lo0 = 4 * S::kBuf, lo1 = 5 * S::kBuf;      // (pipelined hi/lo form only)
    if constexpr (!kHiLo || S::kPipeHiLo) {
        // prologue: Q tiles 0 and 1 parked, Q tile 2 requested, attention rows of tile 0 made
        Origin o_att = first;                 // tile whose attention rows are made next
        Origin o_q = advance(first);          // tile whose Q is requested next
#pragma unroll
        for (int i = 0; i < S::kQV; ++i) park_q1(qb0, i);
        aim_q(o_q, 1 < n_mine);
#pragma unroll
        for (int i = 0; i < S::kQV; ++i) fetch_q1(i);
#pragma unroll
        for (int i = 0; i < S::kQV; ++i) park_q1(qb1, i);
        o_q = advance(o_q);
        aim_q(o_q, 2 < n_mine);
#pragma unroll
        for (int i = 0; i < S::kQV; ++i) fetch_q1(i);
        load_state(o_att.b);
        __syncthreads();
        att_all(qb0, att0, lo0);
        __syncthreads();
        Origin o_out = first;                 // tile whose results are written next
        o_att = advance(o_att);
        for (int t = 0; t < n_mine; ++t) {
            const bool odd = t & 1;
            const int here = odd ? att1 : att0;         // attention rows of tile t
            const int next = odd ? att0 : att1;         // ... of tile t+1, made now
            const int here_lo = odd ? lo1 : lo0, next_lo = odd ? lo0 : lo1;
            const int q_next = odd ? qb0 : qb1;         // Q of tile t+1
            const int q_park = odd ? qb1 : qb0;         // Q of tile t+2 goes where tile t's was
            if (t + 1 < n_mine && o_att.b != img) load_state(o_att.b);
            o_q = advance(o_q);
            aim_q(o_q, t + 3 < n_mine);                 // resource of Q tile t+3
            aim_out(o_out, t > 0);                      // ... and of the results of tile t-1 (none before the first)
            zero_acc();
            read_b(here, 0);
            if constexpr (S::kPipeHiLo) read_b_lo(here_lo, 0);
            if constexpr (kAhead > 1) {
                read_b(here, 1);
                if constexpr (S::kPipeHiLo) read_b_lo(here_lo, 1);
            }
            att_a(q_next, 0);
            // 16 slots of IO*2 matrix instructions; everything else rides between them.  Past the
            // last tile the extra jobs work on zeros that nobody reads.
            static_for<0, KCH>([&](auto kk_c) {
                constexpr int kk = decltype(kk_c)::value;
                if constexpr (kk + kAhead < KCH) {
                    read_b(here, kk + kAhead);
                    if constexpr (S::kPipeHiLo) read_b_lo(here_lo, kk + kAhead);
                }
                constexpr int u = kk / 2;
                if constexpr (kk % 2 == 0) {
                    att_b(u);
                    if constexpr (u + 1 < kUnits) att_a(q_next, u + 1);
                } else {
                    att_c(u, next, next_lo);
                }
                mma_chunk(kk);
                if constexpr (S::kPipeHiLo) mma_chunk_lo(kk);
                // Q tile t+2: registers -> LDS, then the same registers take the request for tile t+3
                constexpr int kParkAt = 1, kFetchAt = 3;
                if constexpr (kk >= kParkAt && kk < kParkAt + S::kQV) park_q1(q_park, kk - kParkAt);
                if constexpr (kk >= kFetchAt && kk < kFetchAt + S::kQV) fetch_q1(kk - kFetchAt);
                // results of tile t-1, a piece at a time
                static_assert(kFetchAt + S::kQV <= KCH && S::JT == 2, "slot plan");
                if constexpr (kk == KCH / 4) flush(0);
                if constexpr (kPieces > 1 && kk == 3 * KCH / 4) flush(1);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (t > 0) o_out = advance(o_out);
            finish(o_out);
            o_att = advance(o_att);
            __syncthreads();
        }
        flush_all(o_out);
    } else {
        Origin o = first, o_q = first, o_out = first;
        for (int t = 0; t < n_mine; ++t) {
            if (o.b != img) load_state(o.b);
#pragma unroll
            for (int i = 0; i < S::kQV; ++i) park_q1(qb0, i);
            if (t > 0) {
                flush_all(o_out);
                o_out = advance(o_out);
            }
            o_q = advance(o_q);
            aim_q(o_q, t + 1 < n_mine);
#pragma unroll
            for (int i = 0; i < S::kQV; ++i) fetch_q1(i);
            __syncthreads();           // Q tile complete; every wave is done with the previous tiles
            att_all(qb0, att0, att1);
            __syncthreads();
            zero_acc();
            read_b(att0, 0);
#pragma unroll
            for (int kk = 0; kk < KCH; ++kk) {
                // the hi fragments come through the ring, one chunk ahead; the lo ones are read here
                Vec lo[S::JT];
#pragma unroll
                for (int jt = 0; jt < S::JT; ++jt)
                    lo[jt] = __builtin_bit_cast(
                        Vec, *(const u32x4*)(lds + att1 + (frag_off ^ ((kk & 1) * 64)) + (kk >> 1) * S::kSlab + jt * 16 * S::kRow));
                if (kk + 1 < KCH) read_b(att0, kk + 1);
                mma_chunk(kk);
#pragma unroll
                for (int io = 0; io < IO; ++io)
#pragma unroll
                    for (int jt = 0; jt < S::JT; ++jt) mma(io, jt, kk, lo[jt]);
            }
            finish(o);
            o = advance(o);
        }
        flush_all(o_out);
    }
}

template <class T, int KCH, int IO>
hipError_t run_apply_project_ws(const void* q_ms, const void* kvfrag, const float* kvscale, const void* w_proj,
                                void* out, const void* res, long n_tokens, int N, int n_hb, int c_out, float eps,
                                bool planar, hipStream_t stream) {
    typedef WsApply<T, KCH, IO> S;
    const int n_cg = (c_out + S::kChanBlock - 1) / S::kChanBlock;
    const int tiles_per_image = (N + S::TB - 1) / S::TB;
    const long n_tt = (n_tokens / N) * tiles_per_image;
    if (n_tt <= 0 || n_tt * n_cg > 0x7fffffffL) return hipErrorInvalidValue;
    if ((long)c_out * n_hb * 32 >= 0x7fffffffL) return hipErrorInvalidValue;
    const long slots = compute_units();
    const long groups = slots / n_cg > 0 ? slots / n_cg : 1;
    const long tiles_per_block = (n_tt + groups - 1) / groups;
    const long nblocks = (n_tt + tiles_per_block - 1) / tiles_per_block * n_cg;
    // (compiled apart: the headline variant has no register to spare for a residual or another layout)
    auto launch = [&](auto out_c) {
        constexpr ApplyOut kOut = decltype(out_c)::value;
        const hipError_t e = allow_dynamic_lds<apply_project_ws_kernel<T, KCH, IO, kOut>>(S::kLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((apply_project_ws_kernel<T, KCH, IO, kOut>), dim3((unsigned)nblocks), dim3(S::kThreads), S::kLds,
                           stream, (const T*)q_ms, (const char*)kvfrag, kvscale, (const T*)w_proj, (T*)out, N, n_hb,
                           c_out, n_cg, tiles_per_image, n_tt, tiles_per_block, eps, (const T*)res);
        return hipGetLastError();
    };
    if (planar) return launch(std::integral_constant<ApplyOut, kOutPlanar>{});
    return res != nullptr ? launch(std::integral_constant<ApplyOut, kOutResidual>{}) : launch(std::integral_constant<ApplyOut, kOutRows>{});
}

// ------------------------------------------- att fused into projection, fp32, weight-stationary
// fp32 storage, contractions of at most 512 slots (n_hb <= 32).  The fp32 matrix instructions bound it (32 cycles for
// 16x16x4), as in the fp32 projection: small pieces, so that every SIMD has its share and nothing is padded.  A workgroup
// of W waves owns W*16 output channels -- a wave keeps its 16 channels' weights in registers, KCH fragments of 16 slots --
// and walks over tiles of JT*16 tokens of one image.  Per tile every wave makes attention rows: unit (16 tokens, head-branch
// m) is four matrix instructions with the state from LDS; the denominator is a dot product on the vector ALU, whose
// partial sums cross the lane groups in two register swaps (with the Ksum rows of channel 0 and of channel 8: they differ
// where a state is two heads of 8 side by side).  Rows go to one of two LDS tiles, so there is one barrier a
// tile; Q is requested a tile ahead.  (The tiled kernel's 256-channel x 64- or 128-token pieces leave most of the chip idle
// on small maps and compute channels that are not there; its denominators are matrix instructions as well.)
// Whole modules, this kernel against the tiled one: 1024 tokens, 64 channels, 8 head-branches 37.7 -> 27.7 us; 576, 256, 32
// 77 -> 39; 4 x 8192, 128, 16 126 -> 114; 2 x 4096, 256, 32 113 -> 99; 2 x 11550, 176, 22 156 -> 158.  Tiles of 32 tokens:
// 0.5-3 us more on the small ones, 1 us less on the largest.
// LDS tile: [token][KCH*16 slots], rows unpadded, the 16-byte chunk index XOR-ed with token % 8: an operand read (16 tokens,
// one chunk each) and an attention row's store (the same) touch every bank once per eight lanes.
template <int KCH, int W, int JT>
struct Ws32Apply {
    static constexpr int kThreads = W * 64, TB = JT * 16, kHb = KCH;
    static constexpr int kRow = KCH * 64;
    static constexpr int kTile = TB * kRow;
    static constexpr int kState = 1024 + 128;             // KV operand (64 lanes x 16 bytes), then two rows of 16 Ksum
    static constexpr int kStates = kHb * kState;
    static constexpr int kLds = 2 * kTile + kStates;
    static constexpr int kUnits = (JT * kHb + W - 1) / W; // attention units a wave, at most
    // resident waves a SIMD: what the registers (4 KCH of weights) and the LDS allow, in whole workgroups
    static constexpr int kByRegs = KCH <= 8 ? 4 : KCH <= 16 ? 3 : 2;
    static constexpr int kResident = 160 * 1024 / kLds < kByRegs * 4 / W ? 160 * 1024 / kLds : kByRegs * 4 / W;
    static_assert(kResident >= 1, "one workgroup fits a CU");
};

template <int KCH, int W, int JT, bool kPlanar>
__global__ __launch_bounds__(W * 64, (Ws32Apply<KCH, W, JT>::kResident * W / 4)) void apply_project_ws32_kernel(const float* __restrict__ q_ms,
                                                                    const char* __restrict__ kvfrag,
                                                                    const float* __restrict__ w_proj, float* __restrict__ out,
                                                                    int N, int n_hb, int c_out, int n_cg, int tiles_per_image,
                                                                    long n_tt, long tiles_per_block, float eps,
                                                                    const float* __restrict__ res) {
    typedef Ws32Apply<KCH, W, JT> S;
    typedef Traits<float> Tr;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* const states = lds + 2 * S::kTile;

    const unsigned L = xcd_remap(blockIdx.x, gridDim.x);
    const int cg = (int)(L % (unsigned)n_cg);
    const long t_begin = (long)(L / (unsigned)n_cg) * tiles_per_block;
    const long t_end = t_begin + tiles_per_block < n_tt ? t_begin + tiles_per_block : n_tt;
    if (t_begin >= t_end) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4;
    const int K = n_hb * 16;
    const int ch0 = cg * W * 16 + wave * 16;
    const bool live = ch0 < c_out;
    const int units = JT * n_hb;

    // this wave's Q fragments of a tile: units wave, wave + W, ... (unit = m * JT + jt).  A token past the image's end reads
    // the last one; it is never stored.
    f32x4 qv[S::kUnits];
    auto fetch_q = [&](long t) {
        const int b = (int)(t / tiles_per_image), n0 = (int)(t % tiles_per_image) * S::TB;
#pragma unroll
        for (int i = 0; i < S::kUnits; ++i) {
            const int u = wave + i * W;
            if (u < units) {
                const int n = n0 + (u % JT) * 16 + x16;
                qv[i] = *(const f32x4*)(q_ms + ((long)b * N + (n < N ? n : N - 1)) * K + (u / JT) * 16 + q * 4);
            }
        }
    };
    fetch_q(t_begin);

    // weights: lane (channel x16, q) holds slots 16 kk + 4q .. + 3 of its channel; slots past K are zero
    f32x4 wf[KCH];
    {
        const float* row = w_proj + (long)(ch0 + x16 < c_out ? ch0 + x16 : c_out - 1) * K + q * 4;
#pragma unroll
        for (int kk = 0; kk < KCH; ++kk) wf[kk] = kk < n_hb ? *(const f32x4*)(row + kk * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
    }

    int img = -1;
    auto load_states = [&](int b) {
        img = b;
        for (int i = threadIdx.x; i < n_hb * 72; i += S::kThreads) {
            const int m = i / 72, c = i % 72;
            const long sid = (long)b * n_hb + m;
            // (row f of the Ksum operand: quarter q sits in lane 16q + f)
            *(u32x4*)(states + m * S::kState + c * 16) =
                *(const u32x4*)(kvfrag + sid * 2048 + (c < 64 ? c * 16 : 1024 + (c & 3) * 256 + (c < 68 ? 0 : 128)));
        }
    };
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const int sw = x16 & 7;
    // attention rows of the tile whose Q is in qv -> LDS tile at byte offset `to`
    auto make_rows = [&](int b, int to) {
#pragma unroll
        for (int i = 0; i < S::kUnits; ++i) {
            const int u = wave + i * W;
            if (u < units) {
                const int m = u / JT, jt = u % JT;
                const char* st = states + m * S::kState;
                const f32x4 kv = *(const f32x4*)(st + lane * 16);
                const f32x4 ka = *(const f32x4*)(st + 1024 + q * 16), kb = *(const f32x4*)(st + 1024 + 64 + q * 16);
                const f32x4 qf = frag_relu<float>(qv[i]);
                const f32x4 num = Tr::mma16(z, kv, qf);
                // this lane's quarter of the dot products, then lanes 0..31 add up the first over the lane groups, lanes
                // 32..63 (channels 8..15) the second
                const float da = (qf[0] * ka[0] + qf[1] * ka[1]) + (qf[2] * ka[2] + qf[3] * ka[3]);
                const float db = (qf[0] * kb[0] + qf[1] * kb[1]) + (qf[2] * kb[2] + qf[3] * kb[3]);
                const u32x2 s32 = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, da),
                                                                   __builtin_bit_cast(unsigned, db), false, false);
                const unsigned a0 = s32[0], a1 = s32[1];
                const unsigned half = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1));
                const u32x2 s16 = __builtin_amdgcn_permlane16_swap(half, half, false, false);
                const unsigned b0 = s16[0], b1 = s16[1];
                const float den = __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
                const float inv = 1.0f / (den + eps);       // (fp32 states are not rescaled)
                *(f32x4*)(lds + to + (jt * 16 + x16) * S::kRow + ((m * 4 + q) ^ sw) * 16) =
                    f32x4{num[0] * inv, num[1] * inv, num[2] * inv, num[3] * inv};
            }
        }
    };

    // slots past K are read with zero weights: they must hold numbers
    for (int i = threadIdx.x; i < 2 * S::TB * (KCH - n_hb) * 4; i += S::kThreads) {
        const int row = i / ((KCH - n_hb) * 4), c = n_hb * 4 + i % ((KCH - n_hb) * 4);
        *(u32x4*)(lds + row * S::kRow + (c ^ (row & 7)) * 16) = u32x4{0u, 0u, 0u, 0u};
    }
    load_states((int)(t_begin / tiles_per_image));
    __syncthreads();
    make_rows(img, 0);
    for (long t = t_begin; t < t_end; ++t) {
        const int here = (int)((t - t_begin) & 1) * S::kTile, next = S::kTile - here;
        const bool more = t + 1 < t_end;
        if (more) fetch_q(t + 1);
        __syncthreads();                    // rows of tile t complete; nobody reads the other tile any more
        const int b = (int)(t / tiles_per_image), n0 = (int)(t % tiles_per_image) * S::TB;
        f32x4 acc[JT];
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) acc[jt] = z;
        if (live) {
#pragma unroll
            for (int kk = 0; kk < KCH; ++kk)
#pragma unroll
                for (int jt = 0; jt < JT; ++jt) {
                    const f32x4 tokens = *(const f32x4*)(lds + here + (jt * 16 + x16) * S::kRow + ((kk * 4 + q) ^ sw) * 16);
                    acc[jt] = kPlanar ? Tr::mma16(acc[jt], tokens, wf[kk]) : Tr::mma16(acc[jt], wf[kk], tokens);
                }
        }
        if (more) {
            const int b_next = (int)((t + 1) / tiles_per_image);
            if (b_next != img) {            // (the same for every wave; the old states were last read before the barrier above)
                load_states(b_next);
                __syncthreads();
            }
            make_rows(b_next, next);
        }
        if (live) {
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) {
                if constexpr (kPlanar) {            // (a lane has tokens 4q..4q+3 of channel x16)
                    const int n = n0 + jt * 16 + q * 4, oc = ch0 + x16;
                    if (oc < c_out) store_planar(out + ((size_t)b * c_out + oc) * N + n, n, N, __builtin_bit_cast(u32x4, acc[jt]));
                    continue;
                }
                const int n = n0 + jt * 16 + x16, oc = ch0 + q * 4;
                if (n < N) {
                    const long at = ((long)b * N + n) * c_out + oc;
                    f32x4 v = acc[jt];
                    if (res != nullptr) v += *(const f32x4*)(res + at);
                    *(f32x4*)(out + at) = v;
                }
            }
        }
    }
}

template <int KCH, int W, int JT>
hipError_t run_apply_project_ws32(const void* q_ms, const void* kvfrag, const void* w_proj, void* out,
                                  const void* res, long n_tokens, int N, int n_hb, int c_out, float eps, bool planar, hipStream_t stream) {
    typedef Ws32Apply<KCH, W, JT> S;
    const int n_cg = (c_out + W * 16 - 1) / (W * 16);
    const int tiles_per_image = (N + S::TB - 1) / S::TB;
    const long n_tt = (n_tokens / N) * tiles_per_image;
    if (n_tt <= 0 || n_tt * n_cg > 0x7fffffffL) return hipErrorInvalidValue;
    const long slots = (long)compute_units() * S::kResident;
    const long groups = slots / n_cg > 0 ? slots / n_cg : 1;
    const long tiles_per_block = (n_tt + groups - 1) / groups;
    const long nblocks = (n_tt + tiles_per_block - 1) / tiles_per_block * n_cg;
    auto launch = [&](auto planar_c) {
        constexpr bool kPlanar = decltype(planar_c)::value;
        const hipError_t e = allow_dynamic_lds<apply_project_ws32_kernel<KCH, W, JT, kPlanar>>(S::kLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((apply_project_ws32_kernel<KCH, W, JT, kPlanar>), dim3((unsigned)nblocks), dim3(S::kThreads), S::kLds, stream,
                           (const float*)q_ms, (const char*)kvfrag, (const float*)w_proj, (float*)out, N, n_hb, c_out, n_cg,
                           tiles_per_image, n_tt, tiles_per_block, eps, (const float*)res);
        return hipGetLastError();
    };
    return planar ? launch(std::true_type{}) : launch(std::false_type{});
}

template <int KCH>
hipError_t run_apply_project_f32(const void* q_ms, const void* kvfrag, const void* w_proj, void* out, const void* res,
                                 long n_tokens, int N, int n_hb, int c_out, float eps, bool planar, hipStream_t stream) {
    // 128 channels a workgroup (the attention rows are made once per channel group: 64 takes 122.8 instead of 114.0 us for
    // the module of 4 x 8192 tokens, 128 channels), except where that leaves half of the compute units without one and
    // there are channels to spread (576 tokens, 256 channels: 42.1 us with 128, 39.0 with 64)
    const long tiles = (n_tokens / N) * ((N + 15) / 16);
    if (c_out > 64 && 2 * tiles * ((c_out + 127) / 128) < compute_units())
        return run_apply_project_ws32<KCH, 4, 1>(q_ms, kvfrag, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
    return run_apply_project_ws32<KCH, 8, 1>(q_ms, kvfrag, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
}

template <class T>
hipError_t run_apply(const void* q_ms, const void* kvfrag, const float* kvscale, void* att, long n_tokens,
                     int N, int n_hb, float eps, hipStream_t stream) {
    const int gpi = (N + 15) / 16;
    const long images = n_tokens / N;
    const long quads = (n_hb + kApplyQuad - 1) / kApplyQuad;
    // as many groups a wave as leave 16 waves a compute unit, eight at most: its states (8 KB) are then an eighth of its Q
    long gpw = images * gpi * quads / (16L * compute_units());
    gpw = gpw < 1 ? 1 : gpw > 8 ? 8 : gpw;
    const long rpi = (gpi + gpw - 1) / gpw;
    const long n_waves = images * rpi * quads;
    const long nblocks = (n_waves + 3) / 4;
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((apply_kernel<T>), dim3((unsigned)nblocks), dim3(256), 0, stream, (const T*)q_ms,
                       (const char*)kvfrag, kvscale, (T*)att, N, n_hb, gpi, (int)gpw, (int)rpi, n_waves, eps);
    return hipGetLastError();
}

template <class T, int WR, int WC>
hipError_t run_apply_project_tiled(const void* q_ms, const void* kvfrag, const float* kvscale, const void* w_proj,
                                   void* out, const void* res, long n_tokens, int N, int n_hb, int c_out, float eps,
                                   hipStream_t stream) {
    typedef GemmTile<T, WR, WC> G;
    const int bpi = (N + G::BC - 1) / G::BC;
    const int n_rb = (c_out + G::BR - 1) / G::BR;
    const long nblocks = (n_tokens / N) * bpi * n_rb;
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    constexpr int kLds = G::kLdsR + G::kLdsC * (Traits<T>::kHiLo ? 2 : 1);
    if (kLds > 48 * 1024) {   // above the default dynamic-LDS limit (the CU has 160 KB)
        const hipError_t e = allow_dynamic_lds<apply_project_kernel<T, WR, WC>>(kLds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((apply_project_kernel<T, WR, WC>), dim3((unsigned)nblocks), dim3(G::kThreads), kLds, stream,
                       (const T*)q_ms, (const char*)kvfrag, kvscale, (const T*)w_proj, (T*)out, N, n_hb, c_out,
                       bpi, n_rb, eps, (const T*)res);
    return hipGetLastError();
}

// Whether an fp32 map of up to 32 head-branches is the tiled form's.  Its pieces are 256 channels x 64 tokens (128 where those
// give every compute unit one), all or nothing: what it computes is its rounds over the compute units.  The weight-stationary
// form computes no more than the map, but makes a token's attention rows once for every 128 channels, and is a quarter slower
// for each.  So the tiled form pays where its pieces are at least three quarters as full as the other's.  Whole modules, us tiled /
// weight-stationary: 16384 tokens of 256 channels (full pieces, both) 104 / 109, 2 x 16384 182 / 195, 8 x 16384 681 / 756; 12288
// (three quarters of the first round) 89.5 / 87.7, 4096 59 / 44; 16384 of 128 (half of each piece) 47.8 / 43.7; 8192 of 320 93.4 / 98.1,
// 20480 263 / 223.
bool tiled_fp32_pays(long images, int N, int c_out) {
    const long cus = compute_units(), rb = (c_out + 255) / 256;
    const long b64 = images * ((N + 63) / 64) * rb, b128 = images * ((N + 127) / 128) * rb;
    const long rounds = b128 < cus ? (b64 + cus - 1) / cus : (b128 + cus - 1) / cus * 2;        // of 64 tokens x 256 channels
    const long other = images * ((N + 15) / 16) * 16 * ((c_out + 127) / 128) * 128;             // tokens x channels
    return 4 * other >= 3 * rounds * cus * (64 * 256);
}

template <class T>
hipError_t run_apply_project(const void* q_ms, const void* kvfrag, const float* kvscale, const void* w_proj,
                             void* out, const void* res, long n_tokens, int N, int n_hb, int c_out, float eps,
                             bool planar, hipStream_t stream) {
#ifndef MSLA_APPLY_NO_WS
    if constexpr (sizeof(T) == 2) {
        // short contraction: weights and states stay in registers
        if (n_hb <= 32) {
            const bool narrow = c_out <= 128;
            if (n_hb <= 16)
                return narrow ? run_apply_project_ws<T, 8, 1>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream)
                              : run_apply_project_ws<T, 8, 2>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
            if (n_hb <= 24)
                return narrow ? run_apply_project_ws<T, 12, 1>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream)
                              : run_apply_project_ws<T, 12, 2>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
            return narrow ? run_apply_project_ws<T, 16, 1>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream)
                          : run_apply_project_ws<T, 16, 2>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
        }
    }
#endif
    if constexpr (sizeof(T) == 4) {
        if (n_hb <= 32 && !tiled_fp32_pays(n_tokens / N, N, c_out)) {
            if (n_hb <= 8) return run_apply_project_f32<8>(q_ms, kvfrag, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
            if (n_hb <= 16) return run_apply_project_f32<16>(q_ms, kvfrag, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
            if (n_hb <= 24) return run_apply_project_f32<24>(q_ms, kvfrag, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
            return run_apply_project_f32<32>(q_ms, kvfrag, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, planar, stream);
        }
    }
    if (planar) return hipErrorInvalidValue;            // (see apply_project_writes_planar)
    // Tiled form: 64 x 64 per wave, 256 channels x 128 tokens per workgroup; a map too small to give
    // every CU such a tile takes 64-token tiles (measured on the 2048- and 1024-token workloads: 33
    // against 45 us and 17 against 25 us; still smaller workgroups were slower again)
    const long blocks = (n_tokens / N) * ((N + 64 * MSLA_APPLY_WC - 1) / (64 * MSLA_APPLY_WC)) *
                        ((c_out + 64 * MSLA_APPLY_WR - 1) / (64 * MSLA_APPLY_WR));
    if (MSLA_APPLY_WC == 2 && blocks < compute_units())
        return run_apply_project_tiled<T, MSLA_APPLY_WR, 1>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, stream);
    return run_apply_project_tiled<T, MSLA_APPLY_WR, MSLA_APPLY_WC>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, N, n_hb, c_out, eps, stream);
}

}  // namespace

hipError_t launch_apply(int dt, const void* q_ms, const void* kvfrag, const float* kvscale, void* att,
                        long n_tokens, int tokens_per_image, int n_hb, float eps, hipStream_t stream) {
    switch (dt) {
        case 0: return run_apply<float>(q_ms, kvfrag, kvscale, att, n_tokens, tokens_per_image, n_hb, eps, stream);
        case 1: return run_apply<_Float16>(q_ms, kvfrag, kvscale, att, n_tokens, tokens_per_image, n_hb, eps, stream);
        case 2: return run_apply<__bf16>(q_ms, kvfrag, kvscale, att, n_tokens, tokens_per_image, n_hb, eps, stream);
    }
    return hipErrorInvalidValue;
}

static bool small_apply_project(int dt, long n_tokens, int tokens_per_image, int n_hb, int c_out) {
    // more head-branches than the register-resident form holds: the long-contraction kernel, which makes a token's attention
    // rows once per 128 output channels and keeps the weights, where the tiled form makes them once per 256 and fetches the
    // weights for every tile.  For few tokens, or up to three such channel groups (8 x 4096 tokens, 320 channels, 60
    // head-branches, fp16: 190 us a module tiled, 172; 6 x 7055, 288, 54, bf16: 264, 246; with four, 8 x 4096, 512, 64: fp16 224,
    // 229, bf16 239, 270)
    const int K = n_hb * 16;
    // Beyond 1024 slots, in parts, while there are at most two pieces of 32 tokens x 128 channels a compute unit and a workgroup walks at most
    // two of them (each fetches its weights; 896 channels leave four units idle, and 73 tiles would be three for some).  Us a
    // module, tiled / in parts, 512 channels, 3x3 + 5x5: 512 tokens fp16 65.0 / 34.7, bf16 74.3 / 37.9; 2048 bf16 (256 pieces) 78.8 / 44.1,
    // 2 x 2048 fp16 (512) 76.4 / 63.6, 4 x 2048 (1024) 89.2 / 105.7; 3 x 45 x 45 of 352, bf16 (576) 87.4 / 93.0.
    const long tiles = (n_tokens / tokens_per_image) * ((tokens_per_image + 31) / 32), pieces = tiles * ((c_out + 127) / 128);
    if (dt != 0 && K > 1024 && K <= 4096 && pieces <= 2L * compute_units() && small_tiles_a_workgroup(tiles, c_out) <= 2) return true;
    return n_hb > 32 && (small_product(dt, n_tokens, K, c_out) || (dt != 0 && K <= 1024 && c_out <= 384));
}

// out channel-planar, [images, c_out, tokens_per_image]: all forms but the tiled one, whose epilogue goes through LDS row by row.
// Modules with planar x and out, us with a transposition / without: fp16 1 x 64 x 128 tokens, 128 channels 25.9 / 23.1, 6 x 128 x
// 129, 128 102.9 / 85.9 (of which 4 are x's), 8 x 64 x 96, 256 105.8 / 101.2, 8 x 53 x 67, 256 84.7 / 84.9 (rows that start anywhere: the widest
// form gains least), bf16 3 x 37 x 53, 192, two scales 46.6 / 43.6, 8 x 64 x 96, 256 115.4 / 105.9, fp32 1600 tokens, 32 21.5 / 18.1,
// 4 x 64 x 128, 128 115.0 / 107.4.
bool apply_project_writes_planar(int dt, long n_tokens, int tokens_per_image, int n_hb, int c_out) {
    if (tokens_per_image > 0x1ffffff) return false;         // (31 bits of bytes over 32 channels' rows)
    if (small_apply_project(dt, n_tokens, tokens_per_image, n_hb, c_out)) return true;
#ifdef MSLA_APPLY_NO_WS
    if (dt != 0) return false;              // (the tiled form takes them all)
#endif
    // fp16's widest form has no registers left for this (it spills), and its stores lose most where rows start at odd elements: there, beyond
    // three million elements, the transposition's launch weighs less (10 x 47 x 49 tokens, 320 channels, 26 head-branches 81.1 / 86.2, 8 x 53 x
    // 67, 256, 32 82.5 / 84.9, 2 x 219 x 39, 304, 26 68.1 / 69.6, but 3 x 81 x 19, 208, 30 34.8 / 33.4, 9 x 46 x 65, 240, 28 73.8 / 71.8).
    if (dt == 1 && n_hb > 24 && c_out > 128 && tokens_per_image % 2 != 0 && n_tokens * c_out > (3L << 20)) return false;
    return n_hb <= 32 && !(dt == 0 && tiled_fp32_pays(n_tokens / tokens_per_image, tokens_per_image, c_out));
}

hipError_t launch_apply_project(int dt, const void* q_ms, const void* kvfrag, const float* kvscale,
                                const void* w_proj, void* out, const void* res, long n_tokens, int tokens_per_image,
                                int n_hb, int c_out, float eps, hipStream_t stream, bool planar) {
    if (small_apply_project(dt, n_tokens, tokens_per_image, n_hb, c_out))
        return launch_small_apply_project(dt, q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, tokens_per_image, n_hb, c_out,
                                          eps, stream, planar);
    switch (dt) {
        case 0: return run_apply_project<float>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, tokens_per_image, n_hb, c_out, eps, planar, stream);
        case 1: return run_apply_project<_Float16>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, tokens_per_image, n_hb, c_out, eps, planar, stream);
        case 2: return run_apply_project<__bf16>(q_ms, kvfrag, kvscale, w_proj, out, res, n_tokens, tokens_per_image, n_hb, c_out, eps, planar, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace msla
