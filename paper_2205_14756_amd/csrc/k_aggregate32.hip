// Multi-scale token aggregation fused with the state of Eq. (3) for heads of 32 channels, 16-bit storage
// (Section 3.1, last paragraph, with d = 32: depthwise k x k, grouped 1x1 with 3*heads groups of 32
// channels, then KV = sum_n relu(K_n)^T [V_n, 1] per image / branch / head).
//
// Two kernels.  3x3 and 5x5 filters take the second (aggregate32_mfma_kernel, depthwise on the matrix cores); 7x7 filters, whose Toeplitz
// operands would span more than eight input columns, and maps of 2 GiB and more the first (aggregate32_kernel):
//
// the form of the general head-size-16 kernel (k_aggregate.hip) with every 16 x 16 block doubled: one
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
#include <algorithm>

#include "aggregate_sweep.h"
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

// ---------------------------------------------------------------- 3x3 and 5x5 filters: depthwise on the matrix cores
// The head-size-16 kernel's form (k_aggregate_mfma.hip) for heads of 32: four waves stage, eight sweep tiles of 16 x 32 tokens, the
// depthwise convolution is a Toeplitz product on 4x4x4 matrix instructions.  A head's three maps of 32 channels do not fit the
// LDS twice, so the pipeline steps from map to map (K, V, Q) with two buffers of one map; a step's map is two blocks of 16
// channels, swept one after the other.  What that changes: the Toeplitz operands of all six blocks wait in LDS (a wave needs
// another 20 registers of them every half step); the first block's depthwise sums wait in registers for the second's, and the
// grouped 1x1 contracts over all 32 in one instruction; a staging wave reads its rows' raw K back in the V step for the raw state.
// Aggregated K stays in registers from its step to V's; V's grouped 1x1 is applied to the summed state at the end.
// A Q that is not finite (an fp16 overflow of one token) must not pass the zeros that surround a filter's taps in its operand, or
// the selecting products of the staging: times them it would be NaN in tokens outside the filter's reach.  A tile that has one is staged
// again with zeros in its place, and the sweeping waves mark what it reaches.  (In K or V it makes the image's states
// of that head useless, wherever it goes.)  With the grouped 1x1 operands of Q and K in LDS (registers for the rest) this costs nothing: a module
// of 8 x 8192 tokens, 8 heads, fp16 143.1 -> 142.0 us, bf16 145.4 -> 144.0; 128 x 128, 2 heads, 3x3 + 5x5, bf16 45.4 -> 44.1.
// Us a module, the first kernel / this: 8 x 8192 tokens, 8 heads, 5x5 fp16 182.9 / 152.8, bf16 199.8 / 154.6; 2048 tokens, 8 heads
// 41.4 / 32.7; 2 x 4096, 4 heads, 3x3 35.8 / 27.8; 16384 tokens, 2 heads, 3x3 + 5x5 64.0 / 42.4.  The first of these, this kernel 91.8 ->
// 58.6 (vector ALU 44 % of a SIMD's cycles, matrix pipe 36 %, LDS 52 %); errors as before or smaller (V is rounded once less).
template <int KS>
struct Mfma32Lds {
    static constexpr int P = (KS - 1) / 2;
    static constexpr int LH = kAggMfmaTileH + 2 * P, LW = kAggMfmaTileW + 2 * P;
    static constexpr int kChanBytes = planar_chan_bytes(LH);
    static constexpr int kMapBytes = D32 * kChanBytes;
    static constexpr int kToepBytes = 6 * KS * 2 * 64 * 8;              // [map][block][filter row][k-step][lane]
    static constexpr int kWvBytes = D32 * D32 * 2;                      // V's grouped 1x1
    static constexpr int kWork = 2 * kMapBytes + 8 * 2 * kTransBytes;   // two maps in flight, the sweeping waves' transposition buffers
    static constexpr int kGpwBytes = 2 * NB * 64 * 16;                  // grouped 1x1 of Q and K as operands: [map][output block][lane]
    static constexpr int kLostBytes = LH * 8;                           // [tile row] columns whose raw Q is not finite
    static constexpr int kBytes = kWork + kToepBytes + kWvBytes + kGpwBytes + kLostBytes;
    static constexpr int kWaveFloats = NB * NB * 256 + D32;             // per wave: accumulator quads of its state, Ksum
    static_assert(kMapBytes % 16 == 0 && LW <= 36 && kBytes <= 160 * 1024 && (12 * kWaveFloats + D32 * D32) * 4 <= kWork, "LDS layout");
};

// One map's sweep of one wave: 16 columns x 4 rows.  kMap: 0 Q, 1 K, 2 V.
template <class T, int KS, int kMap, int kChanBytes>
__device__ __forceinline__ void sweep32(const char* rows, char* trans, const char* toep_lds, const typename Traits<T>::Vec (&gpw)[NB], int H,
                                        int W, int gy0, int gx_first, bool ragged, BufRsrc rout, unsigned q_ms_tb,
                                        typename Traits<T>::Frag (&aggK)[NB][4], typename Traits<T>::Frag (&aggK_lo)[NB][4],
                                        f32x4 (&kv_agg)[NB][NB], float (&ks_agg)[NB]) {
    typedef Traits<T> Tr;
    typedef typename Tr::Frag Frag;
    typedef typename Tr::Vec Vec;
    constexpr int R = 4, NR = R + KS - 1;
    constexpr bool kWide = Tr::kHiLo || kMap == 0;      // depthwise sums as hi + lo pairs
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4, sub = lane & 3;
    const int chn = sweep_channel(lane);
    const int gx0 = gx_first + 4 * sub;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[KS];
    Frag s1v[2][2], dw0[R], dw0_lo[R];      // the first block's depthwise sums of each row
    f32x4 s2v[2][NB];
    u32x2 q_held[NB];
    auto stage1 = [&](int it, f32x4 o) {
        const int y = it % NR - (KS - 1);
        // (the wait states between a 4x4x4 matrix instruction and a reader of its result: see sweep_rows)
        if (kMap == 1) asm volatile("s_nop 4" : "+v"(o));
        if (kMap == 1 && ragged) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (gy0 + y >= H || gx0 + i >= W) o[i] = 0.f;
        }
        if constexpr (kMap == 2) {
            Frag hi, lo;
            if constexpr (Tr::kHiLo) frag_split<T>(o, hi, lo);
            else hi = frag_from_f32<T>(o);
            const int from = 4 * (4 * (x16 & 3) + (x16 >> 2)) + q;
            const u32x2 h2 = __builtin_bit_cast(u32x2, hi);
            s1v[it & 1][0] = __builtin_bit_cast(Frag, u32x2{(unsigned)__shfl((int)h2[0], from), (unsigned)__shfl((int)h2[1], from)});
            if constexpr (Tr::kHiLo) {
                const u32x2 l2 = __builtin_bit_cast(u32x2, lo);
                s1v[it & 1][1] = __builtin_bit_cast(Frag, u32x2{(unsigned)__shfl((int)l2[0], from), (unsigned)__shfl((int)l2[1], from)});
            }
        } else {
            char* tb = trans + (it & 1) * kTransBytes;
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 4; ++i) *(float*)(tb + (4 * sub + i) * kTransTokStride + chn * 4) = o[i];
            wave_lds_fence();
        }
    };
    auto both = [](Frag a, Frag b) {
        Vec v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = a[r];
            v[4 + r] = b[r];
        }
        return v;
    };
    auto stage2 = [&](int it, f32x4 tq) {
        const int ib = it / NR, y = it % NR - (KS - 1);
        if constexpr (kMap == 2) {
#pragma unroll
            for (int ok = 0; ok < NB; ++ok) {
                kv_agg[ok][ib] = Tr::mma16(kv_agg[ok][ib], aggK[ok][y], s1v[it & 1][0]);
                if constexpr (Tr::kHiLo) {
                    kv_agg[ok][ib] = Tr::mma16(kv_agg[ok][ib], aggK[ok][y], s1v[it & 1][1]);
                    kv_agg[ok][ib] = Tr::mma16(kv_agg[ok][ib], aggK_lo[ok][y], s1v[it & 1][0]);
                }
            }
        } else {
            Frag hi, lo;
            if constexpr (kWide) frag_split<T>(tq, hi, lo);
            else hi = frag_from_f32<T>(tq);
            if (ib == 0) {
                dw0[y] = hi;
                if constexpr (kWide) dw0_lo[y] = lo;
                return;
            }
            const Vec vh = both(dw0[y], hi);
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) {
                s2v[it & 1][ob] = kMap == 1 ? Tr::mma_vec(z, vh, gpw[ob]) : Tr::mma_vec(z, gpw[ob], vh);
                if constexpr (kWide) {
                    const Vec vl = both(dw0_lo[y], lo);
                    s2v[it & 1][ob] = kMap == 1 ? Tr::mma_vec(s2v[it & 1][ob], vl, gpw[ob]) : Tr::mma_vec(s2v[it & 1][ob], gpw[ob], vl);
                }
            }
        }
    };
    auto stage3 = [&](int it) {
        const int y = it % NR - (KS - 1);
        if (it / NR == 0) return;
        if constexpr (kMap == 1) {
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) {
                const f32x4 kf = relu_bits_f32(s2v[it & 1][ob]);
                ks_agg[ob] += (kf[0] + kf[1]) + (kf[2] + kf[3]);
                if constexpr (Tr::kHiLo) frag_split<T>(kf, aggK[ob][y], aggK_lo[ob][y]);
                else aggK[ob][y] = frag_from_f32<T>(kf);
            }
        } else if constexpr (kMap == 0) {
            const int gy = gy0 + y - 1 + (q & 1), gx = gx_first + x16;
            const unsigned off = gy < H && gx < W ? (unsigned)(gy * W + gx) * q_ms_tb + (q >> 1) * 16 : kOobOffset;
#pragma unroll
            for (int ob = 0; ob < NB; ++ob) {
                const u32x2 v = __builtin_bit_cast(u32x2, frag_from_f32<T>(s2v[it & 1][ob]));
                if (y % 2 == 0) {
                    q_held[ob] = v;
                } else {
                    const u32x2 s0 = __builtin_amdgcn_permlane16_swap(q_held[ob][0], v[0], false, false);
                    const u32x2 s1 = __builtin_amdgcn_permlane16_swap(q_held[ob][1], v[1], false, false);
                    buf_store16(rout, off + ob * 32, u32x4{s0[0], s1[0], s0[1], s1[1]});
                }
            }
        }
    };
    Frag toep[KS][2], din[2][2];
    auto fetch_row = [&](int i, Frag (&d)[2]) {
        const char* src = rows + (i / NR * 16 + chn) * kChanBytes + i % NR * kPlanarRowBytes + sub * 8;
        d[0] = load_frag<T>(src);
        d[1] = load_frag<T>(src + 8);
    };
    auto fetch_toep = [&](int ib) {
#pragma unroll
        for (int u = 0; u < KS; ++u)
#pragma unroll
            for (int s = 0; s < 2; ++s) toep[u][s] = load_frag<T>(toep_lds + (((kMap * NB + ib) * KS + u) * 2 + s) * 512 + lane * 8);
    };
    fetch_toep(0);
    fetch_row(0, din[0]);
    static_for<0, 2 * NR + 2>([&](auto it_c) {
        constexpr int it = decltype(it_c)::value;
        constexpr auto has_row = [](int i) { return i >= 0 && i < 2 * NR && i % NR >= KS - 1; };
        if constexpr (it + 1 < 2 * NR) fetch_row(it + 1, din[(it + 1) & 1]);
        f32x4 tq = z;
        if constexpr (has_row(it - 1) && kMap != 2) tq = *(const f32x4*)(trans + ((it - 1) & 1) * kTransBytes + x16 * kTransTokStride + q * 16);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (it < 2 * NR) {
            constexpr int r = it % NR;
            if constexpr (it == NR) fetch_toep(1);
            if constexpr (r == 0) {
#pragma unroll
                for (int i = 0; i < KS; ++i) acc[i] = z;
            }
#pragma unroll
            for (int u = 0; u < KS; ++u) {
                const int y = r - u;
                if (y < 0 || y >= R) continue;
                acc[y % KS] = M4<T>::mma(toep[u][0], din[it & 1][0], acc[y % KS]);
                acc[y % KS] = M4<T>::mma(toep[u][1], din[it & 1][1], acc[y % KS]);
            }
        }
        if constexpr (has_row(it - 1)) stage2(it - 1, tq);
        if constexpr (has_row(it - 2)) stage3(it - 2);
        if constexpr (has_row(it)) {
            constexpr int y = it % NR - (KS - 1);
            const f32x4 o = acc[y % KS];
            acc[y % KS] = z;
            stage1(it, o);
        }
    });
}

constexpr int kMfma32Threads = 12 * 64;
template <class T, int KS, bool kRaw>
__global__ __launch_bounds__(kMfma32Threads) void aggregate32_mfma_kernel(AggregateArgs a) {
    typedef Traits<T> Tr;
    typedef typename Tr::Frag Frag;
    typedef typename Tr::Vec Vec;
    typedef Mfma32Lds<KS> L;
    constexpr int P = L::P, SZ = (int)sizeof(T), MTH = kAggMfmaTileH, MTW = kAggMfmaTileW;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* const toep_lds = lds + L::kWork;
    char* const wv_lds = toep_lds + L::kToepBytes;
    char* const gpw_lds = wv_lds + L::kWvBytes;
    unsigned long long* const lost = (unsigned long long*)(gpw_lds + L::kGpwBytes);
    float* const red = (float*)lds;             // reused after the last tile

    const unsigned Lid = xcd_remap(blockIdx.x, gridDim.x);
    const int tiles_x = (a.W + MTW - 1) / MTW, n_tiles = tiles_x * ((a.H + MTH - 1) / MTH);
    const int filled = (n_tiles + a.tiles_per_chunk - 1) / a.tiles_per_chunk;      // (of nchunks)
    if (Lid >= (unsigned)a.B * a.heads * filled) return;
    const int h = Lid % a.heads;
    const int chunk = (Lid / a.heads) % filled;
    const int b = Lid / (a.heads * filled);
    const int Ct = a.heads * D32;
    const long N = (long)a.H * a.W, img_tok0 = (long)b * N;
    const int lane = lane_id(), x16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const T* wgp = (const T*)a.w_gpw + (long)h * 3 * D32 * D32;
    T* q_ms = (T*)a.q_ms;
    const unsigned q_ms_tb = (unsigned)(a.S * Ct * SZ);

    const int tile_begin = chunk * a.tiles_per_chunk;
    const int tile_end = min(n_tiles, tile_begin + a.tiles_per_chunk);
    const int n_my = tile_end - tile_begin;
    struct TileAt {
        int ty0, tx0;
    };
    auto tile_after = [&](TileAt t) {
        t.tx0 += MTW;
        if (t.tx0 >= tiles_x * MTW) { t.tx0 = 0; t.ty0 += MTH; }
        return t;
    };
    TileAt here = {tile_begin / tiles_x * MTH, tile_begin % tiles_x * MTW};
    // this wave's state: a staging wave's raw, a sweeping wave's aggregated
    f32x4 kv[NB][NB], ks4[NB];
    float ks[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        ks4[i] = z;
        ks[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) kv[i][j] = z;
    }

    if (wave < 4) {
        // ---------------- staging: as in the head-size-16 kernel, a lane's 16-byte load being 8 of the 32 channels of one map
        const char* base[3] = {(const char*)((const T*)a.k + (long)h * a.k_hs + img_tok0 * a.k_ts),
                               (const char*)((const T*)a.v + (long)h * a.v_hs + img_tok0 * a.v_ts),
                               (const char*)((const T*)a.q + (long)h * a.q_hs + img_tok0 * a.q_ts)};
        const long ts[3] = {a.k_ts, a.v_ts, a.q_ts};
        Vec sel[NB];
        Frag ones;
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int i = 0; i < NB; ++i) sel[i][r] = Tr::from_f32(q * 8 + r == 16 * i + x16 ? 1.0f : 0.0f);
#pragma unroll
        for (int r = 0; r < 4; ++r) ones[r] = Tr::from_f32(1.0f);
        struct Batch {
            u32x4 v[2][2], tail;
        };
        auto tail_jbase = [](int it) { return it == 2 ? 0 : 4; };
        auto issue = [&](TileAt at, int m, int it, Batch& bt, bool live) {
            const BufRsrc r = make_rsrc(base[m], ((N - 1) * ts[m] + D32) * (long)SZ);
            const unsigned tb = (unsigned)(ts[m] * SZ);
#pragma unroll
            for (int rr = 0; rr < 2; ++rr) {
                const int ly = wave + 4 * (it + rr), gy = at.ty0 - P + ly;
                const bool row_ok = live && ly < L::LH && gy >= 0 && gy < a.H;
#pragma unroll
                for (int cg = 0; cg < 2; ++cg) {
                    const int gx = at.tx0 - P + cg * 16 + x16;
                    bt.v[rr][cg] = buf_load16(r, row_ok && gx >= 0 && gx < a.W ? (unsigned)(gy * a.W + gx) * tb + q * 16 : kOobOffset, 0);
                }
            }
            if (it != 0) {
                const int j = tail_jbase(it) + (x16 >> 2), ly = wave + 4 * j, lx = 32 + (x16 & 3);
                const int gy = at.ty0 - P + ly, gx = at.tx0 - P + lx;
                const bool ok = live && j <= 4 && ly < L::LH && lx < L::LW && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
                bt.tail = buf_load16(r, ok ? (unsigned)(gy * a.W + gx) * tb + q * 16 : kOobOffset, 0);
            }
        };
        const BufRsrc rraw = make_rsrc(q_ms + img_tok0 * a.S * Ct + h * D32, ((N - 1) * a.S * Ct + D32) * (long)SZ);
        // 0 while all of this wave's Q is finite (the selected values are sums over a token's channels: one that is not finite is in all)
        float finite = 0.f;
        auto check = [&](f32x4 d) { finite = fmaf((d[0] + d[1]) + (d[2] + d[3]), 0.f, finite); };
        // This wave's rows of a Q map that is not: stored again, value by value, without the products and with zeros for what is not
        // finite, and the columns of those tokens noted.
        auto restage = [&](TileAt at, char* planar) {
            const BufRsrc r = make_rsrc(base[2], ((N - 1) * ts[2] + D32) * (long)SZ);
            const unsigned tb = (unsigned)(ts[2] * SZ), top = std::is_same<T, _Float16>::value ? 0x7c00u : 0x7f80u;
            const int l = lane_id_again();      // (nothing of this is worth a register while maps are staged)
            const int x = l & 15, c8 = (l >> 4) * 8;
            wave_lds_fence();
#pragma unroll 1
            for (int ly = wave; ly < L::LH; ly += 4) {
                const int gy = at.ty0 - P + ly;
                unsigned long long cols = 0;
#pragma unroll 1
                for (int cg = 0; cg < 3; ++cg) {
                    const int lx = cg * 16 + x, gx = at.tx0 - P + lx;
                    const bool in = lx < L::LW && gy >= 0 && gy < a.H && gx >= 0 && gx < a.W;
                    const u32x4 v = buf_load16(r, in ? (unsigned)(gy * a.W + gx) * tb + c8 * 2 : kOobOffset, 0);
                    bool bad = false;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const unsigned bits = (v[i >> 1] >> (16 * (i & 1))) & 0xffffu;
                        const bool this_bad = (bits & top) == top;
                        bad = bad || this_bad;
                        if (lx < L::LW)
                            *(unsigned short*)(planar + (c8 + i) * L::kChanBytes + ly * kPlanarRowBytes + lx * SZ) = (unsigned short)(this_bad ? 0u : bits);
                    }
                    unsigned long long m = __ballot(bad);
                    m |= m >> 32;
                    cols |= ((m | m >> 16) & 0xffffu) << (cg * 16);
                }
                if (l == 0) lost[ly] = cols;
            }
        };
        auto consume = [&](TileAt at, auto mc, auto itc, const Batch& bt, char* planar, const char* planar_k) {
            constexpr int m = decltype(mc)::value, it = decltype(itc)::value;
            // What a group of 16 tokens (this lane: tokens 4q .. 4q + 3 of channels x16 and 16 + x16) adds to the raw state, in the V step;
            // its K is where the lane put it a step ago.  own: which of the four tokens are the tile's.
            auto raw = [&](const Frag (&v)[NB], const char* k, bool own0, bool own1, bool own2, bool own3) {
                if constexpr (kRaw && m == 1) {
                    Frag rk[NB];
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        rk[i] = frag_relu_bits<T>(load_frag<T>(k + i * 16 * L::kChanBytes));
                        if (!own0) rk[i][0] = Tr::from_f32(0.f);
                        if (!own1) rk[i][1] = Tr::from_f32(0.f);
                        if (!own2) rk[i][2] = Tr::from_f32(0.f);
                        if (!own3) rk[i][3] = Tr::from_f32(0.f);
                    }
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        ks4[i] = Tr::mma16(ks4[i], rk[i], ones);
#pragma unroll
                        for (int j = 0; j < NB; ++j) kv[i][j] = Tr::mma16(kv[i][j], rk[i], v[j]);
                    }
                }
            };
#pragma unroll
            for (int rr = 0; rr < 2; ++rr) {
                const int ly = wave + 4 * (it + rr), gy = at.ty0 - P + ly;
                if (ly >= L::LH) break;
                const bool own_row = ly >= P && ly < P + MTH;
                f32x4 d[2][NB];
#pragma unroll
                for (int cg = 0; cg < 2; ++cg)
#pragma unroll
                    for (int i = 0; i < NB; ++i) d[cg][i] = Tr::mma_vec(z, __builtin_bit_cast(Vec, bt.v[rr][cg]), sel[i]);
                __builtin_amdgcn_sched_barrier(0);
                const int at_lds = x16 * L::kChanBytes + ly * kPlanarRowBytes + q * 8;
#pragma unroll
                for (int cg = 0; cg < 2; ++cg) {
                    if constexpr (m == 2) check(d[cg][0]);
                    Frag f[NB];
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        f[i] = frag_from_f32<T>(d[cg][i]);
                        store_frag<T>(planar + at_lds + i * 16 * L::kChanBytes + cg * 32, f[i]);
                    }
                    const int c0 = cg * 16 + 4 * q;     // (the first P columns are halo; the last are the tail's)
                    if (own_row) raw(f, planar_k + at_lds + cg * 32, c0 >= P, c0 + 1 >= P, c0 + 2 >= P, c0 + 3 >= P);
                    if constexpr (kRaw && m == 2) {
                        const int gx = at.tx0 - P + cg * 16 + x16;
                        buf_store16(rraw, own_row && cg * 16 + x16 >= P && gy < a.H && gx < a.W ? (unsigned)(gy * a.W + gx) * q_ms_tb + q * 16 : kOobOffset,
                                    bt.v[rr][cg]);
                    }
                }
            }
            if constexpr (it != 0) {
                const int j = tail_jbase(it) + q, ly = wave + 4 * j;
                const bool row_ok = j <= 4 && ly < L::LH, own_row = row_ok && ly >= P && ly < P + MTH;
                f32x4 d[NB];
                Frag f[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) d[i] = Tr::mma_vec(z, __builtin_bit_cast(Vec, bt.tail), sel[i]);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (m == 2) check(d[0]);
                const int at_lds = x16 * L::kChanBytes + (row_ok ? ly : 0) * kPlanarRowBytes + 64;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    f[i] = frag_from_f32<T>(d[i]);
                    if (row_ok) store_frag<T>(planar + at_lds + i * 16 * L::kChanBytes, f[i]);
                }
                raw(f, planar_k + at_lds, own_row && 32 < P + MTW, own_row && 33 < P + MTW, own_row && 34 < P + MTW, own_row && 35 < P + MTW);
                if constexpr (kRaw && m == 2) {
                    const int js = tail_jbase(it) + (x16 >> 2), lys = wave + 4 * js, lxs = 32 + (x16 & 3);
                    const int gys = at.ty0 - P + lys, gxs = at.tx0 - P + lxs;
                    buf_store16(rraw, js <= 4 && lys >= P && lys < P + MTH && lxs < P + MTW && gys < a.H && gxs < a.W
                                          ? (unsigned)(gys * a.W + gxs) * q_ms_tb + q * 16 : kOobOffset, bt.tail);
                }
            }
        };
        Batch ring[3];
        static_for<0, 3>([&](auto i) {
            issue(here, 0, 2 * decltype(i)::value, ring[decltype(i)::value], true);
            __builtin_amdgcn_sched_barrier(0);
        });
        int buf = 0;
        for (int i = 0; i < n_my; ++i) {
            const TileAt next = tile_after(here);
            const bool more = i + 1 < n_my;
            static_for<0, 3>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                char* planar = lds + buf * L::kMapBytes;
                static_for<0, 3>([&](auto i3) {
                    constexpr int n = decltype(i3)::value;
                    consume(here, mc, std::integral_constant<int, 2 * n>{}, ring[n], planar, lds + (buf ^ 1) * L::kMapBytes);
                    issue(m < 2 ? here : next, (m + 1) % 3, 2 * n, ring[n], m < 2 || more);
                });
                if constexpr (m == 2) {
                    const int l = lane_id_again();
                    if (wave + 4 * l < L::LH) lost[wave + 4 * l] = 0;
                    if (__any(!(finite == 0.f))) restage(here, planar);
                    finite = 0.f;
                }
                buf ^= 1;
                __syncthreads();
            });
            here = next;
        }
        __syncthreads();
    } else {
        // ---------------- sweeping; before the first map is staged, waves 0 .. 5 make the Toeplitz operands of a block each (map, block of
        // 16 channels) and wave 6 brings V's grouped 1x1
        const int sw = wave - 4;
        if (sw < 6) {
            Frag toep[KS][2];
            make_toeplitz<T, KS>(load_taps<T, KS>((const T*)a.w_dw + (long)h * 3 * D32 * KS * KS, sw * 16 + sweep_channel(lane)), lane & 3, toep);
#pragma unroll
            for (int u = 0; u < KS; ++u)
#pragma unroll
                for (int s = 0; s < 2; ++s) store_frag<T>(toep_lds + ((sw * KS + u) * 2 + s) * 512 + lane * 8, toep[u][s]);
        } else if (sw == 6) {
#pragma unroll
            for (int i = 0; i < 2; ++i) ((u32x4*)wv_lds)[i * 64 + lane] = ((const u32x4*)(wgp + 2 * D32 * D32))[i * 64 + lane];
        } else {
            // grouped 1x1 of Q and K, contraction slots {4q .. 4q + 3} and {16 + 4q ..}: lane (o, q) of output block ob.  A sweep reads its own
            // (16 registers that the others have for themselves)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int ob = 0; ob < NB; ++ob) {
                    const T* row = wgp + (t * D32 + ob * 16 + x16) * D32 + q * 4;
                    const u32x2 lo = *(const u32x2*)row, hi = *(const u32x2*)(row + 16);
                    *(u32x4*)(gpw_lds + (t * NB + ob) * 1024 + lane * 16) = u32x4{lo[0], lo[1], hi[0], hi[1]};
                }
        }
        const int strip = sw & 1, part = sw >> 1;
        const BufRsrc rout = make_rsrc(q_ms + img_tok0 * a.S * Ct + (long)a.branch * Ct + h * D32, ((N - 1) * a.S * Ct + D32) * (long)SZ);
        char* const trans = lds + 2 * L::kMapBytes + sw * 2 * kTransBytes;
        Frag aggK[NB][4], aggK_lo[NB][4];
        int buf = 0;
        for (int c = chunk + filled; c < a.nchunks; c += filled)       // chunks without tiles: empty sums
            for (int j = threadIdx.x - 256; j < kState32; j += kMfma32Threads - 256) {
                float* to = a.partials + (((long)b * a.S * a.heads + h) * a.nchunks + c) * kState32 + j;
                to[(long)a.branch * a.heads * a.nchunks * kState32] = 0.f;
                if constexpr (kRaw) to[0] = 0.f;
            }
        __syncthreads();
        for (int i = 0; i < n_my; ++i) {
            const int gy0 = here.ty0 + 4 * part, gx = here.tx0 + 16 * strip;
            const bool ragged = here.ty0 + MTH > a.H || here.tx0 + MTW > a.W;
            auto sweep = [&](auto mapc) {
                Vec g[NB] = {};
                if constexpr (decltype(mapc)::value < 2) {
#pragma unroll
                    for (int ob = 0; ob < NB; ++ob) g[ob] = *(const Vec*)(gpw_lds + (decltype(mapc)::value * NB + ob) * 1024 + lane_id_again() * 16);
                }
                sweep32<T, KS, decltype(mapc)::value, L::kChanBytes>(lds + buf * L::kMapBytes + 4 * part * kPlanarRowBytes + 16 * strip * SZ, trans,
                                                                     toep_lds, g, a.H, a.W, gy0, gx, ragged, rout, q_ms_tb, aggK, aggK_lo, kv, ks);
                if constexpr (decltype(mapc)::value == 0) {
                    // tokens with a Q that is not finite in the filter's reach: not a number, in all channels (lane: one token)
                    const int l = lane_id_again();          // (nothing of this is worth a register during the sweeps)
                    if (__any(lost[4 * part + (l < 4 + KS - 1 ? l : 0)] != 0)) {
                        const int y = l >> 4, x = l & 15;
                        unsigned long long hit = 0;
#pragma unroll 1
                        for (int u = 0; u < KS; ++u) hit |= lost[4 * part + y + u];
                        const bool mine = (hit >> (16 * strip + x) & ((1u << KS) - 1)) != 0 && gy0 + y < a.H && gx + x < a.W;
                        const unsigned nan = std::is_same<T, _Float16>::value ? 0x7e007e00u : 0x7fc07fc0u;
                        __builtin_amdgcn_s_waitcnt(0);      // (the stores of these tokens above come first)
#pragma unroll 1
                        for (int i = 0; i < 4; ++i)
                            buf_store16(rout, mine ? (unsigned)((gy0 + y) * a.W + gx + x) * q_ms_tb + i * 16 : kOobOffset, u32x4{nan, nan, nan, nan});
                    }
                }
                buf ^= 1;
                __syncthreads();
            };
            sweep(std::integral_constant<int, 1>{});
            sweep(std::integral_constant<int, 2>{});
            sweep(std::integral_constant<int, 0>{});
            here = tile_after(here);
        }
    }

    // ---------------- workgroup partial state: per wave [K block][V block][lane] accumulator quads, then [32] Ksum
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        ks[i] += __shfl_xor(ks[i], 16);
        ks[i] += __shfl_xor(ks[i], 32);
    }
    __syncthreads();   // tile memory is dead from here on
    float* const msum = red + 12 * L::kWaveFloats;              // [32][32] summed pre-1x1 state of the aggregated branch
    {
        float* mine = red + wave * L::kWaveFloats;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
#pragma unroll
            for (int j = 0; j < NB; ++j) *(f32x4*)(mine + (i * NB + j) * 256 + lane * 4) = kv[i][j];
            if (wave < 4) {
                if (x16 == 0) *(f32x4*)(mine + NB * NB * 256 + i * 16 + q * 4) = ks4[i];
            } else if (q == 0) {
                mine[NB * NB * 256 + i * 16 + x16] = ks[i];
            }
        }
    }
    __syncthreads();
    auto sum = [&](int src, bool of_raw) {      // fixed order
        float s = 0.f;
        if (of_raw) {
#pragma unroll
            for (int w = 0; w < 4; ++w) s += red[w * L::kWaveFloats + src];
        } else {
#pragma unroll
            for (int w = 4; w < 12; ++w) s += red[w * L::kWaveFloats + src];
        }
        return s;
    };
    auto put = [&](int branch, int e, int f, float s) {
        a.partials[((((long)b * a.S + branch) * a.heads + h) * a.nchunks + chunk) * kState32 + e * (D32 + 1) + f] = s;
    };
    for (int j = threadIdx.x; j < D32 * D32; j += kMfma32Threads) {
        const int e = j >> 5, c = j & 31, src = ((e >> 4) * NB + (c >> 4)) * 256 + (((e & 15) >> 2) * 16 + (c & 15)) * 4 + (e & 3);
        msum[j] = sum(src, false);
        if constexpr (kRaw) put(0, e, c, sum(src, true));
    }
    if (threadIdx.x < D32) {
        put(a.branch, threadIdx.x, D32, sum(NB * NB * 256 + threadIdx.x, false));
        if constexpr (kRaw) put(0, threadIdx.x, D32, sum(NB * NB * 256 + threadIdx.x, true));
    }
    __syncthreads();
    for (int j = threadIdx.x; j < D32 * D32; j += kMfma32Threads) {
        // the grouped 1x1 of V, applied to the summed state: KV[e][f] = sum_c M[e][c] w_gpw[f][c]
        const int e = j >> 5, f = j & 31;
        float s = 0.f;
#pragma unroll
        for (int c8 = 0; c8 < D32 / 8; ++c8) {
            const Vec w = *(const Vec*)(wv_lds + (f * D32 + c8 * 8) * SZ);
#pragma unroll
            for (int c = 0; c < 8; ++c) s = fmaf(msum[e * D32 + c8 * 8 + c], Tr::to_f32(w[c]), s);
        }
        put(a.branch, e, f, s);
    }
}

template <class T, int KS, bool kRaw>
hipError_t run_mfma32(const AggregateArgs& a, hipStream_t stream) {
    constexpr int kLds = Mfma32Lds<KS>::kBytes;
    const hipError_t e = allow_dynamic_lds<aggregate32_mfma_kernel<T, KS, kRaw>>(kLds);
    if (e != hipSuccess) return e;
    const long tiles = (long)((a.H + kAggMfmaTileH - 1) / kAggMfmaTileH) * ((a.W + kAggMfmaTileW - 1) / kAggMfmaTileW);
    const long filled = (tiles + a.tiles_per_chunk - 1) / a.tiles_per_chunk;
    if (filled > a.nchunks) return hipErrorInvalidValue;
    const long nblocks = ((long)a.B * a.heads * filled + 7) / 8 * 8;         // whole rounds over the XCDs
    if (nblocks <= 0 || nblocks > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((aggregate32_mfma_kernel<T, KS, kRaw>), dim3((unsigned)nblocks), dim3(kMfma32Threads), kLds, stream, a);
    return hipGetLastError();
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
    if (aggregate32_on_matrix_cores(a.ks, (long)a.H * a.W, std::max(std::max(a.q_ts, a.k_ts), std::max(a.v_ts, (long)a.S * a.heads * D32)))) {
        if ((a.do_raw != 0) != (a.copy_raw_q != 0)) return hipErrorInvalidValue;
        AggregateArgs g = a;        // tiles of 16 rows
        const long tiles = (long)((a.H + kAggMfmaTileH - 1) / kAggMfmaTileH) * ((a.W + kAggMfmaTileW - 1) / kAggMfmaTileW);
        // The chunks may have been counted for a 7x7 scale beside it, more than this kernel has tiles or compute units for: its workgroups
        // are counted by themselves and clear the states of the chunks that are left over.  (With a workgroup for every chunk, the empty ones
        // were whole XCDs: 131 x 167 tokens, 6 heads, 3x3 + 7x7, fp16 176.3 us a module, now 159.7; 3 x 151 x 11, 9 heads, 5x5 + 7x7, bf16 156.4, 139.0.)
        const long want = chunks_in_rounds((long)a.B * a.heads, tiles, std::min((long)a.nchunks, tiles), compute_units());
        g.tiles_per_chunk = (int)((tiles + want - 1) / want);
        if (a.ks == 3) return a.do_raw ? run_mfma32<T, 3, true>(g, stream) : run_mfma32<T, 3, false>(g, stream);
        return a.do_raw ? run_mfma32<T, 5, true>(g, stream) : run_mfma32<T, 5, false>(g, stream);
    }
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
