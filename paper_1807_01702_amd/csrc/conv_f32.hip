// conv_f32.hip -- float32 CONV (1x1 and 3x3, forward and data gradient) on the
// float32 matrix cores with the BN fission/fusion prologues and epilogues.
//
// A workgroup (four waves) computes BM pixels x 16 WN output channels; a wave
// owns 16 of the channels and all (WN = 4) or half (WN = 2) of the pixels.
//   * A: the pixel rows of a chunk of K (64 channels; 3x3: 16, plus a W + 1
//     row halo on each side) are staged in LDS, transformed by the prologue, in
//     two buffers: the next chunk is loaded to registers before the matrix-core
//     work on the current one and written after it, one barrier per chunk.
//   * Weights: read from the caller's array straight into matrix-core
//     fragments, two or three steps ahead (they stay in L2); no packing launch and no LDS.
//   * A 16x16x4 product takes one k per lane group; the groups take k = 4 q + s
//     in step s = 0..3 of 16 consecutive k, so one 16-byte LDS read per 16
//     pixels feeds four products.
//   * The weights are the first operand: a lane's accumulators are four
//     consecutive channels of one pixel, so the epilogue works on the
//     accumulators with 16-byte global accesses and no output staging.
// What bounds it: the round trips of a workgroup's prologue and epilogue and
// the float32 matrix cores (157 TFLOP/s).  32 images of 28 x 28, against the
// tiled kernel with its packing launch: 3x3 data gradient 32 -> 128 channels
// 65 + 5 -> 33 us, 3x3 forward 128 -> 32 channels 41 + 3 -> 35 us, 1x1 forward
// 160 -> 128 channels 22 + 5 -> 21 us.  A run-time branch on the weights' layout
// in the products' loop cost 2-4 us a launch; five steps of weights in flight
// instead of two nothing.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "tiles.hpp"
#include "trace.hpp"

namespace bnr {

constexpr int kF32BM = 64;
constexpr int f32_bk(int taps) { return taps == 9 ? 16 : 64; }      // K channels of a chunk
// Row pitch of the staged rows (floats).  1x1: no padding, the sixteen 16-byte
// blocks of a row are permuted by the row number instead (f32_at), which leaves
// room for four workgroups per CU up to K = 1024: with padded rows and four
// coefficient arrays three fitted past K = 384, and 40 images of 28 x 28 took
// 58.4 us forward at 416 -> 128 channels (39.3 at 320 -> 128), 46.4 this way.
constexpr int f32_pitch(int taps) { return taps == 9 ? f32_bk(taps) + 4 : f32_bk(taps); }
template <int TAPS> __device__ __forceinline__ int f32_at(int row, int c)
{
    return row * f32_pitch(TAPS) + (TAPS == 9 ? c : c ^ (4 * (row & 15)));
}
// per-channel coefficients in LDS (floats): c0, c1, (deferred gradient) c2 and the
// centre, where there is none four zeros
static size_t f32_coefs(const RowsParams &p) { return (size_t)(p.pro == PRO_BNGRAD ? 3 : 2) * p.K + (p.p_ctr ? p.K : 4); }
// prologue kinds: FP_ONE (none, BN+ReLU, ReLU or the pooling gradient, chosen
// at run time), FP_BNGRAD and FP_BNADD (a second operand: the deferred BN input
// gradient; BN + identity + ReLU), FP_POOL (four input pixels a row).  With a
// side view (FP_ONE with BN+ReLU, FP_BNADD) the transformed rows are stored too.
enum { FP_ONE = 0, FP_BNGRAD = 1, FP_POOL = 2, FP_BNADD = 3 };
// the BN-backward epilogue on the stored z (p.e_zsrc)
constexpr int EKF_BNBWD_Z = 7;

// Waves per SIMD the registers are held to: four (a workgroup spends as long on
// its prologue and epilogue round trips as on its products, so several per CU
// have to overlap) where that does not spill.
constexpr int f32_waves(int taps, int wn, int fp, bool wt)
{
    if (fp == FP_POOL) return 2;
    if (fp == FP_BNADD || (taps == 9 && wn == 4 && !wt)) return 3;
    return 4;
}

// WT: the data gradient's weights W[n][k] (else the forward's W[k][n])
template <int TAPS, int WN, int FP, int EK, bool WT>
__global__ __launch_bounds__(kThreads, f32_waves(TAPS, WN, FP, WT)) void k_conv_f32(RowsParams p)
{
    using M = Mfma<float>;
    constexpr int BK = f32_bk(TAPS), PITCH = f32_pitch(TAPS);
    constexpr int WM = 4 / WN, TM = kF32BM / 16 / WM;
    constexpr int HALO = TAPS == 9 ? kRowsMaxW3 + 1 : 0;
    constexpr int VPR = BK / 4, RPS = kThreads / VPR;         // vectors per staged row; rows per pass
    constexpr int NA = (kF32BM + 2 * HALO + RPS - 1) / RPS;
    constexpr int PF = FP == FP_POOL ? 4 : 1;
    constexpr bool TWO = FP == FP_BNGRAD || FP == FP_BNADD, ZK = EK == EKF_BNBWD_Z;
    constexpr int NB2 = TWO ? NA : 1;
    constexpr bool BNB = ZK || EK == EK_BNBWD || EK == EK_BNBWD_SC || EK == EK_BNBWD_SCACC;
    constexpr bool READX = BNB || EK == EK_RELUMASK, READY = EK == EK_STORE_ACC || EK == EK_BNBWD_SCACC;
    constexpr int STEPS = TAPS * (BK / 16);                       // 16-channel products of a chunk
    // weight fragments in flight (buffers; a step is 128 TM matrix-core clocks,
    // an L2 read several hundred)
    constexpr int ND = TAPS == 9 ? 3 : 4;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN, q4 = lane >> 4, l16 = lane & 15;
    const int K = p.K, N = p.N, H = p.h, W = p.w;
    const int m = (int)p.m;                                       // launcher: every span below 2^31 bytes
    const int mt = xcd_remap(blockIdx.x, gridDim.x);
    const int p0 = mt * kF32BM, n0 = blockIdx.y * 16 * WN;
    const int halo = TAPS == 9 ? W + 1 : 0, arows = kF32BM + 2 * halo;
    float *As = reinterpret_cast<float *>(smem);                  // [2][arows][PITCH]
    float *coef = As + 2 * arows * PITCH;                     // [f32_coefs][K]: c0, c1, c2, centre
    constexpr bool C2 = FP == FP_BNGRAD;
    float *cen = coef + (C2 ? 3 : 2) * K;
    const bool bnr = FP == FP_POOL || FP == FP_BNADD || (FP == FP_ONE && p.pro == PRO_BNRELU);
    const bool pool = FP == FP_ONE && p.pro == PRO_POOLUP, relu = FP == FP_ONE && p.pro == PRO_RELU;

    // ---- operand views ----
    const int a_ldc = (int)p.a_ldc, a2_ldc = (int)p.a2_ldc, y_ldc = (int)p.y_ldc, ex_ldc = (int)p.ex_ldc;
    const int srows = pool ? m / 4 : (FP == FP_POOL ? 4 * m : m);
    const __amdgpu_buffer_rsrc_t abuf = buf_view(p.a, (uint32_t)(((int64_t)(srows - 1) * a_ldc + K) * 4));
    const __amdgpu_buffer_rsrc_t a2buf = buf_view(TWO ? p.a2 : p.a,
                                                  TWO ? (uint32_t)(((int64_t)(m - 1) * a2_ldc + K) * 4) : 0u);
    const bool side = (FP == FP_BNADD || FP == FP_ONE) && p.side && blockIdx.y == 0;
    const __amdgpu_buffer_rsrc_t sbuf = buf_view(side ? p.side : p.y,
                                                 side ? (uint32_t)(((int64_t)(m - 1) * p.side_ldc + K) * 4) : 0u);
    const __amdgpu_buffer_rsrc_t wbuf = buf_view(p.wraw, (uint32_t)(TAPS * K * N * 4));
    const __amdgpu_buffer_rsrc_t ybuf = buf_view(p.y, (uint32_t)(((int64_t)(m - 1) * y_ldc + N) * 4));
    const __amdgpu_buffer_rsrc_t xbuf = buf_view(READX ? p.ex : p.y,
                                                 READX ? (uint32_t)(((int64_t)(m - 1) * ex_ldc + N) * 4) : 0u);

    // ---- staged rows of this thread: channel vector av of rows tid / VPR + j RPS ----
    const int av = (tid % VPR) * 4, ar0 = tid / VPR;
    uint32_t aoff[NA], a2off[NB2];                                // byte offsets of channel av (kBufOff: zeros)
    #pragma unroll
    for (int j = 0; j < NA; j++) {
        const int r = ar0 + j * RPS, pp = p0 - halo + r;
        const bool ok = r < arows && pp >= 0 && pp < m;
        int q = ok ? pp : 0;
        if (pool) {
            const int img = q / (H * W), rem = q - img * H * W, y = rem / W, x = rem - y * W;
            q = (img * (H / 2) + y / 2) * (W / 2) + x / 2;
        } else if (FP == FP_POOL) {
            const int ho = H / 2, wo = W / 2, img = q / (ho * wo), rem = q - img * ho * wo, y = rem / wo, x = rem - y * wo;
            q = (img * H + 2 * y) * W + 2 * x;
        }
        aoff[j] = ok ? (uint32_t)(q * a_ldc + av) * 4u : kBufOff;
        if (TWO) a2off[j < NB2 ? j : 0] = ok ? (uint32_t)(q * a2_ldc + av) * 4u : kBufOff;
    }
    vec16 ra[NA * PF], rb[NB2];
    auto load_chunk = [&](int ch) __attribute__((always_inline)) {
        const int c = ch * BK;
        const bool cok = c + av < K;
        #pragma unroll
        for (int j = 0; j < NA; j++) {
            const bool ok = cok && aoff[j] != kBufOff;
            #pragma unroll
            for (int f = 0; f < PF; f++) {
                const uint32_t d = FP == FP_POOL ? (uint32_t)(((f >> 1) * W + (f & 1)) * a_ldc) * 4u : 0u;
                ra[j * PF + f] = bld16(abuf, ok ? aoff[j] + d + (uint32_t)c * 4u : kBufOff);
            }
            if (TWO) rb[j < NB2 ? j : 0] = bld16(a2buf, ok ? a2off[j < NB2 ? j : 0] + (uint32_t)c * 4u : kBufOff);
        }
    };
    // rows outside the tensor are zeros (not bn(0)); channels past K have zero weights
    auto store_chunk = [&](int ch, float *dst) __attribute__((always_inline)) {
        const int c = ch * BK + av, cc = c < K ? c : 0;
        const bool kin = c < K;
        float k0[4], k1[4], k2[4], kc[4];
        if (bnr || FP == FP_BNGRAD)
            #pragma unroll
            for (int e = 0; e < 4; e++) {
                k0[e] = coef[cc + e]; k1[e] = coef[K + cc + e];
                k2[e] = C2 ? coef[2 * K + cc + e] : 0.f;
                kc[e] = cen[(p.p_ctr ? cc : 0) + e];
            }
        #pragma unroll
        for (int j = 0; j < NA; j++) {
            float f[4];
            Elem<float>::unpack(ra[j * PF], f);
            const bool ok = kin && aoff[j] != kBufOff;
            if (FP == FP_POOL) {                      // mean over the window of max(x c0 + c1, 0)
                float s[4] = {0.f, 0.f, 0.f, 0.f};
                #pragma unroll
                for (int u = 0; u < PF; u++) {
                    Elem<float>::unpack(ra[j * PF + u], f);
                    #pragma unroll
                    for (int e = 0; e < 4; e++) s[e] += __builtin_fmaxf(bn_lin(f[e] - kc[e], k0[e], k1[e]), 0.f);
                }
                #pragma unroll
                for (int e = 0; e < 4; e++) f[e] = ok ? s[e] * 0.25f : 0.f;
            } else if (FP == FP_BNGRAD) {             // d = c0 dy + c1 x + c2
                float x[4];
                Elem<float>::unpack(rb[j < NB2 ? j : 0], x);
                #pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float d = __builtin_fmaf(k0[e], f[e], __builtin_fmaf(k1[e], x[e] - kc[e], k2[e]));
                    f[e] = ok ? d : 0.f;
                }
            } else if (FP == FP_BNADD) {              // max(x c0 + c1 + identity, 0)
                float id[4];
                Elem<float>::unpack(rb[j < NB2 ? j : 0], id);
                #pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float t = __builtin_fmaxf(bn_lin(f[e] - kc[e], k0[e], k1[e]) + id[e], 0.f);
                    f[e] = ok ? t : 0.f;
                }
            } else if (bnr) {
                #pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float t = bn_lin(f[e] - kc[e], k0[e], k1[e]);
                    f[e] = ok && t > 0.f ? t : 0.f;
                }
            } else if (relu) {
                #pragma unroll
                for (int e = 0; e < 4; e++) f[e] = f[e] > 0.f ? f[e] : 0.f;
            } else if (pool) {
                #pragma unroll
                for (int e = 0; e < 4; e++) f[e] *= 0.25f;
            }
            if (side) {                               // by the first column tile, the tile's own rows
                const int r = ar0 + j * RPS - halo;
                bst16(sbuf, ok && r >= 0 && r < kF32BM ? (uint32_t)((p0 + r) * (int)p.side_ldc + c) * 4u : kBufOff,
                      Elem<float>::pack(f));
            }
            if (TAPS == 1 || ar0 + j * RPS < arows)
                *reinterpret_cast<vec16 *>(dst + f32_at<TAPS>(ar0 + j * RPS, av)) = Elem<float>::pack(f);
        }
    };

    // ---- weight fragments: step s of a chunk is tap s % TAPS of 16-channel
    // group s / TAPS; lane (q4, l16) holds k = 4 q4 + e of column l16 ----
    const int wcol = n0 + wn * 16 + l16;
    auto load_w = [&](int ch, int s, float *b) __attribute__((always_inline)) {
        const int tap = s % TAPS, k = ch * BK + s / TAPS * 16 + 4 * q4;
        const bool ok = wcol < N && k < K;
        if (WT) {                                     // W[TAPS - 1 - tap][n][k]
            const vec16 v = bld16(wbuf, ok ? (uint32_t)(((TAPS - 1 - tap) * N + wcol) * K + k) * 4u : kBufOff);
            Elem<float>::unpack(v, b);
        } else {                                      // W[tap][k][n]
            const uint32_t o = (uint32_t)((tap * K + k) * N + wcol) * 4u;
            #pragma unroll
            for (int e = 0; e < 4; e++)
                b[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wbuf, ok ? o + (uint32_t)(e * N) * 4u : kBufOff, 0, 0));
        }
    };

    // prologue: the first chunk's rows and weights are in flight while the
    // per-channel coefficients are read
    load_chunk(0);
    float wb[ND][4];
    #pragma unroll
    for (int s = 0; s + 1 < ND; s++) load_w(0, s, wb[s]);
    if (bnr || FP == FP_BNGRAD) {
        const float inv_m = 1.0f / (float)m;
        if (!p.p_ctr && tid < 4) cen[tid] = 0.f;
        for (int c = tid; c < K; c += kThreads) {
            float c0, c1, c2 = 0.f;
            const float kc = bn_centre<float>(p.p_ctr, c);
            if (FP == FP_BNGRAD) {
                const float mu = p.p_mean[c], rs = p.p_rstd[c];
                const float g = p.p_split ? p.p_alpha[c] : p.p_gamma[c], dg = p.p_split ? p.p_betap[c] : p.p_dgamma[c];
                const float db = p.p_split ? 0.f : p.p_dbeta[c];
                deferred_coef_of(p.p_split, inv_m, g, mu, rs, dg, db, c0, c1, c2);
            } else {
                bn_coef(p.p_gamma[c], p.p_beta[c], p.p_mean[c], p.p_rstd[c], c0, c1);
            }
            coef[c] = c0; coef[K + c] = c1;
            if (C2) coef[2 * K + c] = c2;
            if (p.p_ctr) cen[c] = kc;
        }
    }
    // pixels of this lane's accumulators, and (3x3) the taps inside the image
    int pix[TM];
    uint32_t taps_in[TM];
    #pragma unroll
    for (int rbk = 0; rbk < TM; rbk++) {
        pix[rbk] = p0 + (wm * TM + rbk) * 16 + l16;
        taps_in[rbk] = 0x1ffu;
        if (TAPS == 9) {
            const int t = pix[rbk] / W, x = pix[rbk] - t * W, y = t % H;
            uint32_t in = 0;
            #pragma unroll
            for (int s = 0; s < 9; s++)
                if ((unsigned)(y + s / 3 - 1) < (unsigned)H && (unsigned)(x + s % 3 - 1) < (unsigned)W) in |= 1u << s;
            taps_in[rbk] = in;
        }
    }
    f32x4 acc[TM];
    #pragma unroll
    for (int i = 0; i < TM; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    store_chunk(0, As);
    __syncthreads();

    const int nch = (K + BK - 1) / BK;
    const int arow = wm * TM * 16 + l16 + halo;
    for (int ch = 0; ch < nch; ch++) {
        const float *src = As + (ch & 1) * arows * PITCH;
        if (ch + 1 < nch) load_chunk(ch + 1);
        // a step's fragments are read while the step before it is multiplied,
        // its weights ND - 1 steps ahead (the scheduler would sink both to
        // their use: the barriers keep the order)
        float4 a[2][TM];
        auto load_a = [&](int s, float4 *dst) __attribute__((always_inline)) {
            const int tap = s % TAPS, kg = s / TAPS;
            const int off = TAPS == 9 ? (tap / 3 - 1) * W + tap % 3 - 1 : 0;
            const float *ap = src + f32_at<TAPS>(arow + off, 4 * q4 + kg * 16);       // (16 rows on: the same permutation)
            #pragma unroll
            for (int i = 0; i < TM; i++)
                dst[i] = *reinterpret_cast<const float4 *>(ap + i * 16 * PITCH);
        };
        load_a(0, a[0]);
        #pragma unroll
        for (int s = 0; s < STEPS; s++) {
            if (TAPS == 1 && ch * BK + s * 16 >= K) break;            // (uniform: no products past K)
            const int sn = s + ND - 1;
            load_w(sn < STEPS ? ch : ch + 1, sn < STEPS ? sn : sn - STEPS, wb[sn % ND]);
            if (s + 1 < STEPS) load_a(s + 1, a[(s + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            float4 (&av4)[TM] = a[s & 1];
            if (TAPS == 9)
                #pragma unroll
                for (int i = 0; i < TM; i++) {
                    const bool in = (taps_in[i] >> (s % TAPS)) & 1u;
                    av4[i].x = in ? av4[i].x : 0.f; av4[i].y = in ? av4[i].y : 0.f;
                    av4[i].z = in ? av4[i].z : 0.f; av4[i].w = in ? av4[i].w : 0.f;
                }
            #pragma unroll
            for (int i = 0; i < TM; i++) M::mma(acc[i], wb[s % ND][0], av4[i].x);
            #pragma unroll
            for (int i = 0; i < TM; i++) M::mma(acc[i], wb[s % ND][1], av4[i].y);
            #pragma unroll
            for (int i = 0; i < TM; i++) M::mma(acc[i], wb[s % ND][2], av4[i].z);
            #pragma unroll
            for (int i = 0; i < TM; i++) M::mma(acc[i], wb[s % ND][3], av4[i].w);
        }
        if (ch + 1 < nch) store_chunk(ch + 1, As + ((ch + 1) & 1) * arows * PITCH);
        __syncthreads();
    }
    static_assert(STEPS % ND == 0 && ND <= STEPS, "weight buffers alternate across chunks too");

    // ---- epilogue on the accumulators: lane = channels n .. n + 3 of TM pixels ----
    const int n = n0 + wn * 16 + 4 * q4;
    const bool col_ok = n < N;
    // ZK: z, or x for a channel vector that holds a gamma = 0 channel (a load at
    // a clamped pixel from this lane's source)
    bool zs = ZK && col_ok;
    if (ZK)
        #pragma unroll
        for (int e = 0; e < 4; e++) zs = zs && p.e_gamma[col_ok ? n + e : 0] != 0.f;
    const float *zsrc = reinterpret_cast<const float *>(ZK && !zs ? p.ex2 : p.ex) + (col_ok ? n : 0);
    const int64_t zld = ZK && !zs ? p.ex2_ldc : p.ex_ldc;
    vec16 xv[READX ? TM : 1], yv[READY ? TM : 1];
    uint32_t yoff[TM];
    #pragma unroll
    for (int i = 0; i < TM; i++) {
        const bool ok = col_ok && pix[i] < m;
        yoff[i] = ok ? (uint32_t)(pix[i] * y_ldc + n) * 4u : kBufOff;
        if (ZK) xv[READX ? i : 0] = ldg16(zsrc + (ok ? pix[i] : 0) * zld);
        else if (READX) xv[READX ? i : 0] = bld16(xbuf, ok ? (uint32_t)(pix[i] * ex_ldc + n) * 4u : kBufOff);
        if (READY) yv[READY ? i : 0] = bld16(ybuf, yoff[i]);
    }
    float mu[4], rs[4], c0[4], c1[4], kc[4], s1[4], s2[4];
    #pragma unroll
    for (int e = 0; e < 4; e++) {
        const int c = col_ok ? n + e : 0;
        s1[e] = s2[e] = 0.f;
        mu[e] = 0.f;
        if (EK == EK_STATS && p.e_shift) mu[e] = p.e_shift[c];
        if (BNB) {
            mu[e] = p.e_mean[c]; rs[e] = p.e_rstd[c]; kc[e] = bn_centre<float>(p.e_ctr, c);
            bn_coef(p.e_gamma[c], p.e_beta[c], mu[e], rs[e], c0[e], c1[e]);
            if (zs) {                                 // mask fma(z, 1, 0) > 0, xhat = (z - beta) / gamma
                mu[e] = p.e_beta[c]; rs[e] = 1.0f / p.e_gamma[c]; kc[e] = 0.f; c0[e] = 1.f; c1[e] = 0.f;
            }
        }
    }
    #pragma unroll
    for (int i = 0; i < TM; i++) {
        const bool ok = yoff[i] != kBufOff;
        float f[4], x[4], old[4];
        #pragma unroll
        for (int e = 0; e < 4; e++) f[e] = acc[i][e];
        if (READX) Elem<float>::unpack(xv[READX ? i : 0], x);
        if (READY) Elem<float>::unpack(yv[READY ? i : 0], old);
        #pragma unroll
        for (int e = 0; e < 4; e++) {
            if (EK == EK_STORE_ACC) f[e] += old[e];
            else if (EK == EK_RELUMASK) f[e] = x[e] > 0.f ? f[e] : 0.f;
            else if (EK == EK_STATS) {
                const float d = ok ? f[e] - mu[e] : 0.f;
                s1[e] += d;
                s2[e] += d * d;
            } else if (BNB) {
                // (a row past the tensor adds zeros, whatever it was read from)
                const float xc = x[e] - kc[e], xh = ok ? (xc - mu[e]) * rs[e] : 0.f;
                const float d = ok && bn_lin(xc, c0[e], c1[e]) > 0.f ? f[e] : 0.f;
                s1[e] += d;
                s2[e] += d * xh;
                // summed-gradient form: gamma rstd dy, stored or added
                f[e] = EK == EK_BNBWD || ZK ? d : (EK == EK_BNBWD_SCACC ? __builtin_fmaf(d, c0[e], old[e]) : d * c0[e]);
            }
        }
        bst16(ybuf, yoff[i], Elem<float>::pack(f));
    }
    if (EK == EK_STATS || BNB) {
        constexpr int ROWS = 16 * WM, LD = 16 * WN;
        float *red = As;                              // (every wave is past its last read of the staged rows)
        #pragma unroll
        for (int e = 0; e < 4; e++) {
            red[(wm * 16 + l16) * LD + wn * 16 + 4 * q4 + e] = s1[e];
            red[(ROWS + wm * 16 + l16) * LD + wn * 16 + 4 * q4 + e] = s2[e];
        }
        lds_colsum2(red, ROWS, LD, LD, kThreads, tid, p.part + (int64_t)mt * 2 * N + n0,
                    p.part + (int64_t)mt * 2 * N + N + n0, N - n0);
    }
}

// ------------------------------------------------------------- launchers ---
// Every operand span below 2^31 bytes (raw-buffer offsets); larger tensors
// take the tiled kernel.
bool conv_f32_supported(const RowsParams &p)
{
    const int64_t lim = (int64_t)1 << 31;
    const bool poolf = p.pro == PRO_BNRELU_POOL;
    if (p.dtype != DT_F32 || (p.taps == 9 && (poolf || p.pro == PRO_BNADDRELU || p.w > kRowsMaxW3))) return false;
    if ((p.side && (p.m * p.side_ldc + p.K) * 4 >= lim) || (p.ex2 && (p.m * p.ex2_ldc + p.N) * 4 >= lim)) return false;
    if (p.pro == PRO_BNADDRELU && (p.m * p.a2_ldc + p.K) * 4 >= lim) return false;
    const int64_t srows = poolf ? 4 * p.m : p.m;
    return (srows * p.a_ldc + p.K) * 4 < lim && (p.pro != PRO_BNGRAD || (p.m * p.a2_ldc + p.K) * 4 < lim) &&
           (p.m * p.y_ldc + p.N) * 4 < lim && (!p.ex || (p.m * p.ex_ldc + p.N) * 4 < lim) &&
           (int64_t)p.taps * p.K * p.N * 4 < lim && p.m <= (lim >> 2) - kF32BM;
}

template <int TAPS, int WN, int FP, int EK, bool WT>
static hipError_t run_f32(const RowsParams &p, hipStream_t s)
{
    const int arows = kF32BM + (TAPS == 9 ? 2 * (p.w + 1) : 0);
    // statistics scratch: two arrays of 16 WM rows of 16 WN floats (8 KB)
    const size_t lds = ((size_t)2 * arows * f32_pitch(TAPS) + f32_coefs(p)) * sizeof(float);
    const double m = (double)p.m, e = 4.0;
    double a = m * p.K;
    if (FP == FP_BNGRAD || p.side) a *= 2.0;
    if (FP == FP_BNADD) a *= 1.5;                     // y and the identity read, the result written
    if (FP == FP_POOL) a *= 4.0;
    if (p.pro == PRO_POOLUP) a /= 4.0;
    double out = m * p.N;
    if (EK == EK_STORE_ACC || EK == EK_RELUMASK || EK == EK_BNBWD || EK == EKF_BNBWD_Z || EK == EK_BNBWD_SC) out *= 2.0;
    if (EK == EK_BNBWD_SCACC) out *= 3.0;
    if (WT != (p.wtrans != 0)) return hipErrorInvalidValue;
    auto kern = k_conv_f32<TAPS, WN, FP, EK, WT>;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t er = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (er != hipSuccess) return er;
        attr_set = true;
    }
    TraceScope tr(KC_CONV, TAPS == 9 ? KID_CONV_3X3 : KID_CONV_1X1, s, e * (a + out + (double)TAPS * p.K * p.N),
                  2.0 * m * TAPS * p.K * p.N);
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(p.m, kF32BM), (unsigned)ceil_div(p.N, 16 * WN)), dim3(kThreads), lds,
                       s, p);
    return hipGetLastError();
}

template <int TAPS, int WN, int FP>
static hipError_t run_f32_ek(const RowsParams &p, hipStream_t s)
{
    const int ek = epilogue_kind(p.epi, p.accumulate, p.e_scale);
    if constexpr (FP == FP_POOL || FP == FP_BNADD) {
        if (ek == EK_STATS) return run_f32<TAPS, WN, FP, EK_STATS, false>(p, s);
        if (ek == EK_STORE) return run_f32<TAPS, WN, FP, EK_STORE, false>(p, s);
        return hipErrorInvalidValue;
    } else {
        // (statistics: the forward; everything else but a plain store: the data gradient)
        if constexpr (FP == FP_ONE) {
            if (ek == EK_STATS) return run_f32<TAPS, WN, FP, EK_STATS, false>(p, s);
            if (ek == EK_STORE && !p.wtrans) return run_f32<TAPS, WN, FP, EK_STORE, false>(p, s);
        }
        switch (ek) {
        case EK_STORE: return run_f32<TAPS, WN, FP, EK_STORE, true>(p, s);
        case EK_STORE_ACC: return run_f32<TAPS, WN, FP, EK_STORE_ACC, true>(p, s);
        case EK_RELUMASK: return run_f32<TAPS, WN, FP, EK_RELUMASK, true>(p, s);
        case EK_BNBWD_SC: return run_f32<TAPS, WN, FP, EK_BNBWD_SC, true>(p, s);
        case EK_BNBWD_SCACC: return run_f32<TAPS, WN, FP, EK_BNBWD_SCACC, true>(p, s);
        case EK_STATS: return hipErrorInvalidValue;
        default:
            return p.e_zsrc ? run_f32<TAPS, WN, FP, EKF_BNBWD_Z, true>(p, s) : run_f32<TAPS, WN, FP, EK_BNBWD, true>(p, s);
        }
    }
}

hipError_t launch_conv_f32(const RowsParams &p, hipStream_t s)
{
    if (!conv_f32_supported(p) || !p.a || !p.wraw || !p.y || p.m < 1) return hipErrorInvalidValue;
    const bool poolf = p.pro == PRO_BNRELU_POOL;
    const bool bnadd = p.pro == PRO_BNADDRELU;
    if (p.side && ((p.pro != PRO_BNRELU && !bnadd) || p.wtrans || (p.epi != EPI_STORE && p.epi != EPI_STATS) || p.accumulate))
        return hipErrorInvalidValue;
    if (bnadd && (!p.a2 || !p.side)) return hipErrorInvalidValue;
    if (p.e_zsrc && (p.epi != EPI_BNBWD || p.e_scale || !p.ex2)) return hipErrorInvalidValue;
    if ((p.pro == PRO_BNRELU || poolf || bnadd) && (!p.p_mean || !p.p_gamma || !p.p_rstd || !p.p_beta)) return hipErrorInvalidValue;
    if (poolf && (p.h % 2 || p.w % 2 || (int64_t)p.n * p.h * p.w != 4 * p.m || p.wtrans)) return hipErrorInvalidValue;
    if (!poolf && (int64_t)p.n * p.h * p.w != p.m) return hipErrorInvalidValue;
    if (p.pro == PRO_POOLUP && (p.h % 2 || p.w % 2)) return hipErrorInvalidValue;
    if (p.pro == PRO_BNGRAD && (!p.a2 || !p.p_mean || !p.p_rstd ||
                                (p.p_split ? (!p.p_alpha || !p.p_betap) : (!p.p_gamma || !p.p_dbeta || !p.p_dgamma))))
        return hipErrorInvalidValue;
    if ((p.epi == EPI_STATS || p.epi == EPI_BNBWD) && !p.part) return hipErrorInvalidValue;
    if (p.epi == EPI_BNBWD && (!p.ex || !p.e_mean || !p.e_rstd || !p.e_gamma || !p.e_beta)) return hipErrorInvalidValue;
    if (p.epi == EPI_RELUMASK && !p.ex) return hipErrorInvalidValue;
    if (p.taps == 9) {
        if (p.pro == PRO_BNGRAD) return p.N <= 32 ? run_f32_ek<9, 2, FP_BNGRAD>(p, s) : run_f32_ek<9, 4, FP_BNGRAD>(p, s);
        return p.N <= 32 ? run_f32_ek<9, 2, FP_ONE>(p, s) : run_f32_ek<9, 4, FP_ONE>(p, s);
    }
    if (bnadd) return p.N <= 32 ? run_f32_ek<1, 2, FP_BNADD>(p, s) : run_f32_ek<1, 4, FP_BNADD>(p, s);
    if (poolf) return p.N <= 32 ? run_f32_ek<1, 2, FP_POOL>(p, s) : run_f32_ek<1, 4, FP_POOL>(p, s);
    if (p.pro == PRO_BNGRAD) return p.N <= 32 ? run_f32_ek<1, 2, FP_BNGRAD>(p, s) : run_f32_ek<1, 4, FP_BNGRAD>(p, s);
    return p.N <= 32 ? run_f32_ek<1, 2, FP_ONE>(p, s) : run_f32_ek<1, 4, FP_ONE>(p, s);
}

}  // namespace bnr
