// Multi-scale token aggregation fused with the state of Eq. (3) for heads of 32 channels, 16-bit storage
// (Section 3.1, last paragraph, with d = 32: depthwise k x k, grouped 1x1 with 3*heads groups of 32
// channels, then KV = sum_n relu(K_n)^T [V_n, 1] per image / branch / head).
//
// The form of the general head-size-16 kernel (k_aggregate.hip) with every 16 x 16 block doubled: one
// workgroup owns one (image, head) and a run of 8 x 32-token tiles; per tile it stages the halo tile of the
// head's raw K, V and Q channels in LDS, one map at a time (the next one on its way while the current one is
// swept), and each of its 4 waves takes 2 tile rows.  A lane (strip, q) owns 4
// consecutive tokens and channels 4q..4q+3 of one 16-channel block of Q, K or V and slides the k x k window
// along its strip in registers (fp32 sums), block after block.  The grouped 1x1 is a 2 x 2 arrangement of
// 16x16x16 matrix instructions, relu(K)^T V a 2 x 2 arrangement of accumulators contracted over the tokens;
// aggregated K and V never leave registers, aggregated Q is written with a lane storing 4 consecutive
// channels of its own token, and the raw branch rides along through an identity matrix, which is exact.
// Operand precision as in the head-size-16 kernel: depthwise sums and aggregated K/V as hi + lo pairs for
// bf16; for fp16 the Q sums as hi + lo, the K and V operands rounded once.
// What bounds it is the vector ALU (two thirds of a SIMD's cycles with two waves on it).  Two waves a SIMD is what the
// register plan is for, with 3x3 and 5x5 filters: the grouped 1x1 operands and the raw tokens are read from LDS where they are
// used, a filter row's pixels and taps are not read ahead, matrix results go to ordinary registers (compiler flag).  8 x 8
// heads, 64 x 128 tokens, fp16, 5x5: this kernel 136 -> 85 us, the module 239 -> 193; with one wave a SIMD and 388 registers, half of
// them on their way between register files, the reads ahead did not hide what a second wave does.  The LDS holds one
// workgroup with a 7x7 filter (92 KB in fp16, 101 in bf16), so one wave a SIMD it is there (kAhead): 24 heads, 4 x 64 x 64 tokens, the
// module 380 -> 352 us in fp16, 414 -> 397 in bf16 (361 and 417 without the reads ahead).
// Per-workgroup partial states [32][33] go to the buffer that the plain finalize kernel sums in a fixed order.
#include "msla_device.h"
#include "msla_kernels.h"

namespace msla {
namespace {

constexpr int TH = kAggTileH, TW = kAggTileW;
constexpr int kThreads32 = 256;
constexpr int D32 = 32, NB = 2;                      // head size; 16-channel blocks per Q, K or V
constexpr int kState32 = D32 * (D32 + 1);

template <class T, int KS>
struct Agg32Lds {
    static constexpr int P = (KS - 1) / 2;
    static constexpr int LH = TH + 2 * P, LW = TW + 2 * P;
    // One map (Q, K or V: 32 channels = eight quads) of the halo tile at a time, two buffers: the next map is fetched while
    // the current one is swept.
    typedef HaloPlanes<LH, LW, (int)sizeof(T), 2> Planes;
    static constexpr int kMapBytes = 2 * 4 * Planes::kPlane;
    static constexpr int kTileBytes = 2 * kMapBytes;
    // filter taps [t][tap][32 ch]: fp16 as they are (the multiply-add takes them), bf16 widened
    typedef typename std::conditional<std::is_same<T, _Float16>::value, _Float16, float>::type Tap;
    static constexpr int kWtsBytes = 3 * KS * KS * D32 * (int)sizeof(Tap);
    static constexpr int kGpwBytes = 3 * NB * NB * 64 * 8;           // grouped 1x1 operands [t][out block][in block][lane]
    // per wave: [branch][K block][V block][lane] accumulator quads, then [branch][32] Ksum
    static constexpr int kWaveFloats = 2 * NB * NB * 256 + 2 * D32;
    static constexpr int kRedBytes = 4 * kWaveFloats * 4;
    static constexpr int kBytes = (kTileBytes > kRedBytes ? kTileBytes : kRedBytes) + kWtsBytes + kGpwBytes;
    // waves a SIMD: two workgroups a CU where the LDS allows it
    static constexpr int kWaves = 2 * kBytes <= 160 * 1024 ? 2 : 1;
};

// kRaw: the raw branch rides along (its state and the copy of its Q).  A template argument and not a run-time branch: with
// the branch, the compiler (ROCm 7.2) left out the wait states between a matrix instruction before it and the conversion of
// its result behind it, on the path that skips the raw branch, and the second V block of the state came out wrong.
template <class T, int KS, bool kRaw>
__global__ __launch_bounds__(kThreads32, (Agg32Lds<T, KS>::kWaves)) void aggregate32_kernel(AggregateArgs a) {
    static_assert(sizeof(T) == 2, "16-bit storage types");
    typedef Traits<T> Tr;
    typedef typename Tr::Frag Frag;
    typedef Agg32Lds<T, KS> L;
    // One wave a SIMD: every read of a filter row is sent out before the first result is used -- with the raw branch, whose
    // compiled code otherwise waits for each tap (8 x 64 x 128 tokens, 8 heads, 7x7, the module: fp16 279 -> 270 us, bf16 328 -> 309);
    // without it (a module's second scale) the compiler's own order is the better one (3x3 and 7x7, fp16 358 and 365).
    constexpr bool kAhead = L::kWaves == 1 && kRaw;
    constexpr int P = L::P;
    constexpr int SZ = (int)sizeof(T);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* tile = lds;
    typedef typename L::Tap Tap;
    Tap* wts = (Tap*)(lds + (L::kBytes - L::kWtsBytes - L::kGpwBytes));
    char* gpw_lds = lds + (L::kBytes - L::kGpwBytes);
    float* red = (float*)lds;   // reused after the last tile

    const unsigned Lid = xcd_remap(blockIdx.x, gridDim.x);
    const int h = Lid % a.heads;
    const int chunk = (Lid / a.heads) % a.nchunks;
    const int b = Lid / (a.heads * a.nchunks);
    const int Ct = a.heads * D32;
    const long N = (long)a.H * a.W;
    const long img_tok0 = (long)b * N;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int x16 = lane & 15, q = lane >> 4;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};

    // depthwise filters of this head -> LDS as [t][tap][32]
    {
        const T* wdw = (const T*)a.w_dw + (long)h * 3 * D32 * KS * KS;
        for (int it = threadIdx.x; it < 3 * D32 * KS * KS; it += kThreads32) {
            const int ch = it / (KS * KS), tap = it - ch * (KS * KS);
            wts[((ch / D32) * KS * KS + tap) * D32 + (ch % D32)] = (Tap)wdw[it];
        }
    }
    // grouped 1x1 weights of (h, t), block (out ob, in ib), as an MFMA operand: lane (o, q) holds
    // w[ob*16 + o][ib*16 + 4q .. 4q+3].  They wait in LDS: in registers they would cost the second wave of the SIMD.
    for (int it = wave; it < 3 * NB * NB; it += 4) {
        const int t = it / (NB * NB), ob = (it / NB) % NB, ib = it % NB;
        store_frag<T>(gpw_lds + (it * 64 + lane) * 8,
                      load_frag<T>((const T*)a.w_gpw + ((long)(h * 3 + t) * D32 + ob * 16 + x16) * D32 + ib * 16 + q * 4));
    }
    auto gpw = [&](int t, int ob, int ib) { return load_frag<T>(gpw_lds + (((t * NB + ob) * NB + ib) * 64 + lane) * 8); };
    Frag ident;
#pragma unroll
    for (int r = 0; r < 4; ++r) ident[r] = Tr::from_f32(x16 == q * 4 + r ? 1.0f : 0.0f);

    const T* maps[3] = {(const T*)a.q + (long)h * a.q_hs, (const T*)a.k + (long)h * a.k_hs, (const T*)a.v + (long)h * a.v_hs};
    const long map_ts[3] = {a.q_ts, a.k_ts, a.v_ts};
    T* q_ms = (T*)a.q_ms;
    const long q_ms_ts = (long)a.S * Ct;

    f32x4 kv_agg[NB][NB], kv_raw[NB][NB];
    float ks_agg[NB], ks_raw[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        ks_agg[i] = ks_raw[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) kv_agg[i][j] = kv_raw[i][j] = z;
    }

    const int tiles_x = (a.W + TW - 1) / TW, tiles_y = (a.H + TH - 1) / TH;
    const int n_tiles = tiles_x * tiles_y;
    const int tile_begin = chunk * a.tiles_per_chunk;
    const int tile_end = min(n_tiles, tile_begin + a.tiles_per_chunk);
    // this lane's strip inside the tile
    const int srow = wave * 2 + (x16 >> 3);
    const int scol = (x16 & 7) * 4;
    // byte offset of its pixels 4j .. 4j+3 (columns scol + 4j ..) in a tile row of its quad's plane
    constexpr int kQuads = (4 + KS - 1 + 3) / 4;
    int lane_at[kQuads];
#pragma unroll
    for (int j = 0; j < kQuads; ++j) lane_at[j] = q * L::Planes::kPlane + L::Planes::at(srow, scol + 4 * j);
    auto pixel = [&](const char* map, int ib, int u, int c) {       // block ib of row srow + u, column scol + c
        return load_frag<T>(map + ib * 4 * L::Planes::kPlane + lane_at[c >> 2] + (u * L::Planes::kRowSlots + (c & 3)) * L::Planes::kSlot);
    };

    // Stages: (tile, pass) with the passes in the order K, V, Q.  A stage's map goes global -> registers while
    // the stage before it is swept, registers -> LDS after that sweep, one barrier a stage.
    constexpr int VPT = D32 * SZ / 16;
    constexpr int kItems = L::LH * L::LW * VPT;                    // 16-byte vectors of one map's halo tile
    constexpr int kPer = (kItems + kThreads32 - 1) / kThreads32;
    u32x4 pre[kPer];
    auto map_of = [](int pass) { return pass == 0 ? 1 : pass == 1 ? 2 : 0; };
    // this thread's pixels of a halo tile: row and column in it (a row no image has for those past the last)
    int item_yx[kPer];
    const int item_v = threadIdx.x % VPT;
    static_assert(kThreads32 % VPT == 0, "a thread keeps its channels");
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int it = threadIdx.x + j * kThreads32, pix = it / VPT;
        item_yx[j] = it < kItems ? (pix / L::LW) << 8 | (pix % L::LW) : 0x7f << 8;
    }
    static_assert(L::LW < 256 && L::LH < 0x7f, "a pixel's place is packed");
    auto fetch = [&](int tile_id, int pass) {
        const int ty0 = (tile_id / tiles_x) * TH, tx0 = (tile_id % tiles_x) * TW;
        const int t = map_of(pass);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int gy = ty0 - P + (item_yx[j] >> 8), gx = tx0 - P + (item_yx[j] & 255);
            u32x4 val = {0u, 0u, 0u, 0u};
            if (item_yx[j] < (L::LH << 8) && (unsigned)gy < (unsigned)a.H && (unsigned)gx < (unsigned)a.W)
                val = *(const u32x4*)(maps[t] + (img_tok0 + (long)gy * a.W + gx) * map_ts[t] + item_v * Tr::kVec);
            pre[j] = val;
        }
    };
    auto stash = [&](char* buf) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (item_yx[j] < (L::LH << 8)) {
                char* dst = buf + item_v * 2 * L::Planes::kPlane + L::Planes::at(item_yx[j] >> 8, item_yx[j] & 255);
                *(u32x2*)dst = u32x2{pre[j][0], pre[j][1]};
                *(u32x2*)(dst + L::Planes::kPlane) = u32x2{pre[j][2], pre[j][3]};
            }
        }
    };
    int cur = 0;
    if (tile_begin < tile_end) {
        fetch(tile_begin, 0);
        stash(tile);
    }
    __syncthreads();   // first map staged, wts written

    for (int tile_id = tile_begin; tile_id < tile_end; ++tile_id) {
        const int ty0 = (tile_id / tiles_x) * TH, tx0 = (tile_id % tiles_x) * TW;
        const int gy = ty0 + srow, gx0 = tx0 + scol;
        bool valid[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) valid[r] = (gy < a.H) && (gx0 + r < a.W);
        const long tok0 = img_tok0 + (long)gy * a.W + gx0;

        Frag aggK[NB][4], aggK_lo[NB][4], rawK[NB][4];
        // order K, V, Q: K's operands are kept for the V pass; Q only stores
#pragma unroll
        for (int pass = 0; pass < 3; ++pass) {
            const int t = (pass == 0) ? 1 : (pass == 1) ? 2 : 0;
            // Q's sums always as hi + lo: the sign of an aggregated Q component decides what passes the
            // rectifier of Eq. (2), so it keeps its fp32 accuracy up to its store
            const bool wide = Tr::kHiLo || t == 0;
            const bool more = pass < 2 || tile_id + 1 < tile_end;
            if (more) fetch(pass < 2 ? tile_id : tile_id + 1, pass < 2 ? pass + 1 : 0);
            const char* map = tile + cur * L::kMapBytes;
            Frag dwf[NB][4], dwl[NB][4];
            // the strip's raw tokens (the centre tap), for the raw branch and the raw-Q copy
            auto center = [&](int ib, int r) {
                const Frag f = pixel(map, ib, P, r + P);
                return valid[r] ? f : frag_zero<T>();
            };
#pragma unroll
            for (int ib = 0; ib < NB; ++ib) {
                float acc[4][4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[r][c] = 0.f;
                const Tap* wt = wts + t * KS * KS * D32 + ib * 16 + q * 4;
                // one filter row at a time: 4+KS-1 pixels feed 4 tokens x KS taps x 4 channels
#pragma unroll 1
                for (int u = 0; u < KS; ++u) {
                    Frag px[4 + KS - 1];
#pragma unroll
                    for (int c = 0; c < 4 + KS - 1; ++c) px[c] = pixel(map, ib, u, c);
                    typedef typename std::conditional<sizeof(Tap) == 2, Frag, f32x4>::type Taps;
                    auto taps = [&](int v) { return *(const Taps*)(wt + (u * KS + v) * D32); };
                    Taps ahead[kAhead ? KS : 1];
                    if constexpr (kAhead) {
#pragma unroll
                        for (int v = 0; v < KS; ++v) ahead[v] = taps(v);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int v = 0; v < KS; ++v) {
                        const Taps w = kAhead ? ahead[kAhead ? v : 0] : taps(v);
                        f32x4 w4;
                        if constexpr (sizeof(Tap) == 2) w4 = frag_to_f32<T>(w);
                        else w4 = w;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const f32x4 d4 = frag_to_f32<T>(px[r + v]);
#pragma unroll
                            for (int c = 0; c < 4; ++c) acc[r][c] = fmaf(w4[c], d4[c], acc[r][c]);
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    f32x4 a4 = {acc[r][0], acc[r][1], acc[r][2], acc[r][3]};
                    if (!valid[r]) a4 = z;       // tokens outside the image contribute nothing
                    if (wide) frag_split<T>(a4, dwf[ib][r], dwl[ib][r]);
                    else dwf[ib][r] = frag_from_f32<T>(a4);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (t == 1) {
#pragma unroll
                    for (int ob = 0; ob < NB; ++ob) {
                        // lane (c, q) <- channel ob*16 + c of the r-th token of strips 4q..4q+3
                        f32x4 kf = z;
#pragma unroll
                        for (int ib = 0; ib < NB; ++ib) {
                            kf = Tr::mma16(kf, dwf[ib][r], gpw(1, ob, ib));
                            if constexpr (Tr::kHiLo) kf = Tr::mma16(kf, dwl[ib][r], gpw(1, ob, ib));
                        }
#pragma unroll
                        for (int c = 0; c < 4; ++c) kf[c] = fmaxf(kf[c], 0.f);      // Eq. (2): relu(K)
                        ks_agg[ob] += (kf[0] + kf[1]) + (kf[2] + kf[3]);
                        if constexpr (Tr::kHiLo) frag_split<T>(kf, aggK[ob][r], aggK_lo[ob][r]);
                        else aggK[ob][r] = frag_from_f32<T>(kf);
                        if constexpr (kRaw) {
                            const Frag rk = frag_relu<T>(frag_from_f32<T>(Tr::mma16(z, center(ob, r), ident)));
                            rawK[ob][r] = rk;
                            const f32x4 rf = frag_to_f32<T>(rk);
                            ks_raw[ob] += (rf[0] + rf[1]) + (rf[2] + rf[3]);
                        }
                    }
                } else if (t == 2) {
#pragma unroll
                    for (int ov = 0; ov < NB; ++ov) {
                        f32x4 vf = z;
#pragma unroll
                        for (int ib = 0; ib < NB; ++ib) {
                            vf = Tr::mma16(vf, dwf[ib][r], gpw(2, ov, ib));
                            if constexpr (Tr::kHiLo) vf = Tr::mma16(vf, dwl[ib][r], gpw(2, ov, ib));
                        }
                        // KV[e][f] += sum_n relu(K_n[e]) V_n[f], block (K block ok, V block ov)
                        Frag vh, vl;
                        if constexpr (Tr::kHiLo) frag_split<T>(vf, vh, vl);
                        else vh = frag_from_f32<T>(vf);
                        Frag rv;
                        if constexpr (kRaw) rv = frag_from_f32<T>(Tr::mma16(z, center(ov, r), ident));
#pragma unroll
                        for (int ok = 0; ok < NB; ++ok) {
                            kv_agg[ok][ov] = Tr::mma16(kv_agg[ok][ov], aggK[ok][r], vh);
                            if constexpr (Tr::kHiLo) {
                                kv_agg[ok][ov] = Tr::mma16(kv_agg[ok][ov], aggK[ok][r], vl);
                                kv_agg[ok][ov] = Tr::mma16(kv_agg[ok][ov], aggK_lo[ok][r], vh);
                            }
                            if constexpr (kRaw) kv_raw[ok][ov] = Tr::mma16(kv_raw[ok][ov], rawK[ok][r], rv);
                        }
                    }
                } else {
#pragma unroll
                    for (int ob = 0; ob < NB; ++ob) {
                        // transposed: lane (strip, q) <- output channels ob*16 + 4q..4q+3 of its own token r
                        f32x4 qq = z;
#pragma unroll
                        for (int ib = 0; ib < NB; ++ib) {
                            qq = Tr::mma16(qq, gpw(0, ob, ib), dwf[ib][r]);
                            qq = Tr::mma16(qq, gpw(0, ob, ib), dwl[ib][r]);
                        }
                        if (valid[r]) {
                            T* dst = q_ms + (tok0 + r) * q_ms_ts + h * D32 + ob * 16 + q * 4;
                            store_frag<T>(dst + (long)a.branch * Ct, frag_from_f32<T>(qq));
                            if constexpr (kRaw) store_frag<T>(dst, center(ob, r));
                        }
                    }
                }
            }
            // the next stage's map: registers -> the other buffer (free since the barrier of the stage before)
            if (more) stash(tile + (cur ^ 1) * L::kMapBytes);
            __syncthreads();
            cur ^= 1;
        }
    }

    // ---- workgroup partial state: combine the 4 q-groups of Ksum, then the 4 waves
#pragma unroll
    for (int ob = 0; ob < NB; ++ob) {
        ks_agg[ob] += __shfl_xor(ks_agg[ob], 16);
        ks_agg[ob] += __shfl_xor(ks_agg[ob], 32);
        ks_raw[ob] += __shfl_xor(ks_raw[ob], 16);
        ks_raw[ob] += __shfl_xor(ks_raw[ob], 32);
    }
    __syncthreads();   // tile memory is dead from here on
    {
        float* mine = red + wave * L::kWaveFloats;
#pragma unroll
        for (int ok = 0; ok < NB; ++ok)
#pragma unroll
            for (int ov = 0; ov < NB; ++ov) {
                *(f32x4*)(mine + ((0 * NB + ok) * NB + ov) * 256 + lane * 4) = kv_agg[ok][ov];
                *(f32x4*)(mine + ((1 * NB + ok) * NB + ov) * 256 + lane * 4) = kv_raw[ok][ov];
            }
        if (q == 0) {
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) {
                mine[2 * NB * NB * 256 + ob * 16 + x16] = ks_agg[ob];
                mine[2 * NB * NB * 256 + D32 + ob * 16 + x16] = ks_raw[ob];
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < 2 * kState32; j += kThreads32) {
        const int which = j / kState32, idx = j - which * kState32;   // 0: aggregated, 1: raw
        if (which == 1 && !kRaw) continue;
        const int e = idx / (D32 + 1), f = idx - e * (D32 + 1);
        // KV[e][f] sits in block (e / 16, f / 16), lane (f % 16, (e % 16) / 4), element e % 4
        const int src = f < D32 ? ((which * NB + (e >> 4)) * NB + (f >> 4)) * 256 + ((((e & 15) >> 2) * 16) + (f & 15)) * 4 + (e & 3)
                                : 2 * NB * NB * 256 + which * D32 + e;
        const float s = (red[src] + red[L::kWaveFloats + src]) + (red[2 * L::kWaveFloats + src] + red[3 * L::kWaveFloats + src]);
        const int branch = which == 0 ? a.branch : 0;
        a.partials[((((long)b * a.S + branch) * a.heads + h) * a.nchunks + chunk) * kState32 + idx] = s;
    }
}

template <class T, int KS, bool kRaw>
hipError_t run_ks32_raw(const AggregateArgs& a, unsigned nblocks, hipStream_t stream) {
    constexpr int kLds = Agg32Lds<T, KS>::kBytes;
    static_assert(kLds <= 160 * 1024, "the halo tile of a head of 32 channels fits the LDS");
    const hipError_t e = allow_dynamic_lds<aggregate32_kernel<T, KS, kRaw>>(kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((aggregate32_kernel<T, KS, kRaw>), dim3(nblocks), dim3(kThreads32), kLds, stream, a);
    return hipGetLastError();
}
template <class T, int KS>
hipError_t run_ks32(const AggregateArgs& a, unsigned nblocks, hipStream_t stream) {
    if ((a.do_raw != 0) != (a.copy_raw_q != 0)) return hipErrorInvalidValue;
    return a.do_raw ? run_ks32_raw<T, KS, true>(a, nblocks, stream) : run_ks32_raw<T, KS, false>(a, nblocks, stream);
}

template <class T>
hipError_t run32(const AggregateArgs& a, hipStream_t stream) {
    const long nblocks = (long)a.B * a.heads * a.nchunks;
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    if (a.ks == 3) return run_ks32<T, 3>(a, (unsigned)nblocks, stream);
    if (a.ks == 5) return run_ks32<T, 5>(a, (unsigned)nblocks, stream);
    if (a.ks == 7) return run_ks32<T, 7>(a, (unsigned)nblocks, stream);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_aggregate32(int dt, const AggregateArgs& a, hipStream_t stream) {
    switch (dt) {
        case 1: return run32<_Float16>(a, stream);
        case 2: return run32<__bf16>(a, stream);
    }
    return hipErrorNotSupported;
}

}  // namespace msla
