// conv_poolup.hip -- data gradient of a bf16 1x1 CONV that was followed by
// 2x2 average pooling (transition layers), with the BN-backward epilogue.
//
// The gradient of the pooling is constant over a window, and so is the data
// gradient of a 1x1 CONV of it: the product runs over window rows (a quarter
// of the pixel rows: a quarter of the matrix work, operand loads and staging)
// and the epilogue applies each row to its window's four pixels.  Every pixel
// gets the value the product over pixel rows gives.
//
// What bounds it: the epilogue reads the BN input and writes dy for every
// pixel, 2 N bf16 values a pixel against N / 4 products, so HBM.  A workgroup
// of 4 waves takes BM windows x 128 output channels; all its BN-input vectors
// (BM / 4 a thread) are requested after the last operand chunk and are in
// flight during the last products, so the epilogue does not wait row by row.
// Against the kernels over pixel rows: [128, 14, 14] 1024 <- 512 channels 124 -> 37 us
// (109 MB: 2.9 TB/s), [64, 56, 56] 256 <- 128 channels 72 -> 45 us (219 MB: 4.9 TB/s),
// [9, 30, 26] 144 <- 72 channels 12.7 -> 10.5 us.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "tiles.hpp"
#include "trace.hpp"

namespace bnr {

constexpr int kPuBN = 128, kPuBK = 64, kPuStr = kPuBK + 8, kPuCStr = kPuBN + 8;
constexpr int kPuRStep = kThreads / (kPuBN / 8);              // windows per pass of the epilogue

template <int BM> constexpr size_t pu_lds()
{
    const size_t stage = (size_t)(BM + kPuBN) * kPuStr * 2, red = 2ull * kPuRStep * kPuBN * sizeof(float);
    return stage > red ? stage : red;                         // (the output tile is smaller than the stage)
}

// BM: windows per tile.  EK: epilogue kind (EK_STORE, EK_STORE_ACC, EK_BNBWD*).
template <int BM, int EK>
__global__ __launch_bounds__(kThreads, BM == 64 && EK == EK_BNBWD_SCACC ? 2 : 3) void k_conv_poolup(RowsParams p, int ntiles)
{
    using T = bf16_t;
    using M = Mfma<T>;
    constexpr int VPR = kPuBK / 8;                            // vectors per staged row
    constexpr int NA = BM * VPR / kThreads, NB = kPuBN * VPR / kThreads;
    constexpr int TM = BM / 16, TN = 2;                       // a wave: every window, 32 channels
    constexpr int NW = BM / kPuRStep;                         // windows per thread in the epilogue
    constexpr bool BNB = EK == EK_BNBWD || EK == EK_BNBWD_SC || EK == EK_BNBWD_SCACC;
    constexpr bool ACC = EK == EK_STORE_ACC || EK == EK_BNBWD_SCACC;
    static_assert(NA >= 1 && NA * kThreads == BM * VPR && NW >= 1, "tile");
    static_assert((size_t)BM * kPuCStr * 2 <= pu_lds<BM>(), "output tile");
    __shared__ __align__(16) unsigned char smem[pu_lds<BM>()];
    __shared__ __align__(32) float epar[BNB ? 4 : 1][kPuBN];  // gamma, beta, mean, rstd
    T *As = reinterpret_cast<T *>(smem);                      // [BM][kPuStr] windows
    T *Bs = As + BM * kPuStr;                                 // [128][kPuStr] weights, rows of n

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // neighbouring ids share a window tile (its g rows stay in one XCD's L2)
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    const int mt = lid / ntiles, n0 = (lid - mt * ntiles) * kPuBN;
    const int K = p.K, N = p.N, W = p.w;
    const int64_t mw = p.m / 4, w0 = (int64_t)mt * BM;

    // operand addresses, clamped to real rows (their values are zeroed or
    // never stored); channel vector c0 + vk is the same in every slot
    const int vk = (tid % VPR) * 8;
    const T *gp[NA], *wp[NB];
    bool gok[NA];
    #pragma unroll
    for (int j = 0; j < NA; j++) {
        const int64_t r = w0 + tid / VPR + j * (kThreads / VPR);
        gok[j] = r < mw;
        gp[j] = reinterpret_cast<const T *>(p.a) + (gok[j] ? r : mw - 1) * p.a_ldc;
    }
    #pragma unroll
    for (int j = 0; j < NB; j++)
        wp[j] = reinterpret_cast<const T *>(p.wraw) + (int64_t)min(n0 + tid / VPR + j * (kThreads / VPR), N - 1) * K;

    vec16 ra[NA], rw[NB];
    auto load_chunk = [&](int c0) __attribute__((always_inline)) {
        const int c = min(c0 + vk, K - 8);
        #pragma unroll
        for (int j = 0; j < NA; j++) ra[j] = ldg16(gp[j] + c);
        #pragma unroll
        for (int j = 0; j < NB; j++) rw[j] = ldg16(wp[j] + c);
    };
    auto store_chunk = [&](int c0) __attribute__((always_inline)) {
        const bool cok = c0 + vk < K;
        #pragma unroll
        for (int j = 0; j < NA; j++) {
            float f[8];
            Elem<T>::unpack(ra[j], f);
            #pragma unroll
            for (int e = 0; e < 8; e++) f[e] *= 0.25f;
            vec16 o = Elem<T>::pack(f);
            #pragma unroll
            for (int i = 0; i < 4; i++) o.u[i] = (cok & gok[j]) ? o.u[i] : 0u;
            *reinterpret_cast<vec16 *>(As + (tid / VPR + j * (kThreads / VPR)) * kPuStr + vk) = o;
        }
        #pragma unroll
        for (int j = 0; j < NB; j++) {
            vec16 o = rw[j];
            #pragma unroll
            for (int i = 0; i < 4; i++) o.u[i] = cok ? o.u[i] : 0u;
            *reinterpret_cast<vec16 *>(Bs + (tid / VPR + j * (kThreads / VPR)) * kPuStr + vk) = o;
        }
    };

    // channels in the accumulator's rows: a lane holds 4 consecutive channels
    // of one window
    f32x4 acc[TM][TN];
    #pragma unroll
    for (int rb = 0; rb < TM; rb++)
        #pragma unroll
        for (int cb = 0; cb < TN; cb++) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const T *al = As + (lane & 15) * kPuStr + (lane >> 4) * 8;
    const T *bl = Bs + (wave * TN * 16 + (lane & 15)) * kPuStr + (lane >> 4) * 8;
    auto products = [&]() __attribute__((always_inline)) {
        #pragma unroll
        for (int ks = 0; ks < kPuBK; ks += M::KSTEP) {
            typename M::frag b[TN];
            #pragma unroll
            for (int cb = 0; cb < TN; cb++) b[cb] = M::load(bl + cb * 16 * kPuStr + ks);
            #pragma unroll
            for (int rb = 0; rb < TM; rb++) {
                const typename M::frag a = M::load(al + rb * 16 * kPuStr + ks);
                #pragma unroll
                for (int cb = 0; cb < TN; cb++) M::mma(acc[rb][cb], b[cb], a);
            }
        }
    };

    // ---- epilogue geometry: channel vector n, windows w0 + r0 + j kPuRStep ----
    const int v = tid % (kPuBN / 8), r0 = tid / (kPuBN / 8);
    const int n = n0 + v * 8, nc = min(n, N - 8);             // (nc: a channel vector that exists)
    const bool col_ok = n < N;
    bool zs = BNB && p.e_zsrc;                                // this thread's vector reads z (else x)
    if (BNB) {
        // (parameters of the tile's channels wait in LDS: the BN-input vectors
        // need the registers)
        if (tid < kPuBN) {
            const int c = min(n0 + tid, N - 1);
            const float ga = p.e_gamma[c], be = p.e_beta[c], mu = p.e_mean[c], rs = p.e_rstd[c];
            epar[0][tid] = ga; epar[1][tid] = be; epar[2][tid] = mu; epar[3][tid] = rs;
        }
        if (zs)
            for (int e = 0; e < 8; e++) zs = zs && p.e_gamma[nc + e] != 0.f;
    }
    const bool from2 = BNB && p.e_zsrc && !zs;
    const T *xs = reinterpret_cast<const T *>(from2 ? p.ex2 : p.ex);
    const int64_t xl = from2 ? p.ex2_ldc : p.ex_ldc;
    int64_t pix[NW];                                          // first pixel of each window
    #pragma unroll
    for (int j = 0; j < NW; j++) {
        const int64_t q = min(w0 + r0 + j * kPuRStep, mw - 1);
        const int64_t row = q / (W / 2);                      // window row: two image rows
        pix[j] = 2 * (row * W + (q - row * (W / 2)));
    }
    vec16 xv[BNB ? NW : 1][4];

    const int nch = (K + kPuBK - 1) / kPuBK;
    load_chunk(0);
    for (int ch = 0; ch + 1 < nch; ch++) {
        store_chunk(ch * kPuBK);
        __syncthreads();
        load_chunk((ch + 1) * kPuBK);
        __builtin_amdgcn_sched_barrier(0);
        products();
        __syncthreads();
    }
    if (BNB) {
        #pragma unroll
        for (int j = 0; j < NW; j++)
            #pragma unroll
            for (int q = 0; q < 4; q++) xv[j][q] = ldg16(xs + (pix[j] + (q >> 1) * W + (q & 1)) * xl + nc);
        __builtin_amdgcn_sched_barrier(0);
    }
    store_chunk((nch - 1) * kPuBK);
    __syncthreads();
    products();
    __syncthreads();

    T *Cs = reinterpret_cast<T *>(smem);                      // [BM][kPuCStr]
    #pragma unroll
    for (int rb = 0; rb < TM; rb++)
        #pragma unroll
        for (int cb = 0; cb < TN; cb++) {
            const uint2 o = make_uint2(pack2bf(acc[rb][cb][0], acc[rb][cb][1]), pack2bf(acc[rb][cb][2], acc[rb][cb][3]));
            *reinterpret_cast<uint2 *>(Cs + (rb * 16 + (lane & 15)) * kPuCStr + wave * TN * 16 + cb * 16 +
                                       (lane >> 4) * 4) = o;
        }
    __syncthreads();

    float emu[8], ers[8], eg[8], eb[8], es[8];
    if (BNB) {
        float ga[8], be[8];
        lds_f8(epar[0] + v * 8, ga);
        lds_f8(epar[1] + v * 8, be);
        lds_f8(epar[2] + v * 8, emu);
        lds_f8(epar[3] + v * 8, ers);
        #pragma unroll
        for (int e = 0; e < 8; e++) {
            bn_coef(ga[e], be[e], emu[e], ers[e], eg[e], eb[e]);
            es[e] = eg[e];                                    // summed-form scale
            if (zs) {                                         // mask [z > 0], xhat = (z - beta) / gamma
                emu[e] = be[e]; ers[e] = 1.0f / ga[e]; eg[e] = 1.f; eb[e] = 0.f;
            }
        }
    }
    float s1[8], s2[8];
    #pragma unroll
    for (int e = 0; e < 8; e++) { s1[e] = 0.f; s2[e] = 0.f; }
    #pragma unroll
    for (int j = 0; j < NW; j++) {
        const bool ok = col_ok && w0 + r0 + j * kPuRStep < mw;
        if (!ok) continue;
        const vec16 cv = *reinterpret_cast<const vec16 *>(Cs + (r0 + j * kPuRStep) * kPuCStr + v * 8);
        float f[8];
        Elem<T>::unpack(cv, f);
        T *dst[4];
        vec16 ov[4];
        #pragma unroll
        for (int q = 0; q < 4; q++) {
            dst[q] = reinterpret_cast<T *>(p.y) + (pix[j] + (q >> 1) * W + (q & 1)) * p.y_ldc + n;
            if (ACC) ov[q] = ldg16(dst[q]);
        }
        // (a window's four pixels are added first, then the windows, and the
        // threads' sums in pairs: chains rounded dgamma up to 20% further off)
        float t1[8], t2[8];
        #pragma unroll
        for (int q = 0; q < 4; q++) {
            float o[8], old[8];
            if (ACC) Elem<T>::unpack(ov[q], old);
            if (BNB) {
                float x[8];
                Elem<T>::unpack(xv[BNB ? j : 0][q], x);
                #pragma unroll
                for (int e = 0; e < 8; e++) {
                    const float xh = (x[e] - emu[e]) * ers[e];
                    const float d = bn_lin(x[e], eg[e], eb[e]) > 0.f ? f[e] : 0.f;
                    t1[e] = q ? t1[e] + d : d;
                    t2[e] = q ? __builtin_fmaf(d, xh, t2[e]) : d * xh;
                    o[e] = EK == EK_BNBWD ? d : (ACC ? __builtin_fmaf(d, es[e], old[e]) : d * es[e]);
                }
                stg16(dst[q], Elem<T>::pack(o));
            } else if (ACC) {
                #pragma unroll
                for (int e = 0; e < 8; e++) o[e] = f[e] + old[e];
                stg16(dst[q], Elem<T>::pack(o));
            } else {
                stg16(dst[q], cv);
            }
        }
        if (BNB)
            #pragma unroll
            for (int e = 0; e < 8; e++) { s1[e] += t1[e]; s2[e] += t2[e]; }
    }
    if (BNB) {
        __syncthreads();
        float *red = reinterpret_cast<float *>(smem);
        #pragma unroll
        for (int e = 0; e < 8; e++) {
            red[r0 * kPuBN + v * 8 + e] = s1[e];
            red[(kPuRStep + r0) * kPuBN + v * 8 + e] = s2[e];
        }
        __syncthreads();
        // one column a thread, its rows added in pairs
        static_assert(kThreads == 2 * kPuBN && kPuRStep == 16, "columns of both sums, rows");
        const int c = tid % kPuBN, k = tid / kPuBN;
        float t[kPuRStep];
        #pragma unroll
        for (int j = 0; j < kPuRStep; j++) t[j] = red[(k * kPuRStep + j) * kPuBN + c];
        #pragma unroll
        for (int st = 1; st < kPuRStep; st *= 2)
            #pragma unroll
            for (int j = 0; j < kPuRStep; j += 2 * st) t[j] += t[j + st];
        if (n0 + c < N) p.part[((int64_t)mt * 2 + k) * N + n0 + c] = t[0];
    }
}

// ------------------------------------------------------------- launchers ---
// Windows per tile: 64, or 32 while 64 would leave the chip's compute units
// without two workgroups each (a smaller tile stages the weights for half the rows).
static int pu_bm(int64_t m, int N)
{
    return ceil_div(m / 4, 64) * ceil_div(N, kPuBN) < 2 * device_cus() ? 32 : 64;
}

bool conv_poolup_supported(const RowsParams &p)
{
    return p.dtype == DT_BF16 && p.taps == 1 && p.pro == PRO_POOLUP && (p.epi == EPI_BNBWD || p.epi == EPI_STORE);
}

int64_t conv_poolup_partial_rows(int64_t m, int N) { return ceil_div(m / 4, pu_bm(m, N)); }

template <int BM>
static void run_poolup(const RowsParams &p, int ntiles, unsigned grid, hipStream_t s)
{
    switch (epilogue_kind(p.epi, p.accumulate, p.e_scale)) {
    case EK_STORE: hipLaunchKernelGGL((k_conv_poolup<BM, EK_STORE>), dim3(grid), dim3(kThreads), 0, s, p, ntiles); break;
    case EK_STORE_ACC:
        hipLaunchKernelGGL((k_conv_poolup<BM, EK_STORE_ACC>), dim3(grid), dim3(kThreads), 0, s, p, ntiles);
        break;
    case EK_BNBWD: hipLaunchKernelGGL((k_conv_poolup<BM, EK_BNBWD>), dim3(grid), dim3(kThreads), 0, s, p, ntiles); break;
    case EK_BNBWD_SC:
        hipLaunchKernelGGL((k_conv_poolup<BM, EK_BNBWD_SC>), dim3(grid), dim3(kThreads), 0, s, p, ntiles);
        break;
    default:
        hipLaunchKernelGGL((k_conv_poolup<BM, EK_BNBWD_SCACC>), dim3(grid), dim3(kThreads), 0, s, p, ntiles);
        break;
    }
}

hipError_t launch_conv_poolup(const RowsParams &p, hipStream_t s)
{
    if (!conv_poolup_supported(p) || !p.a || !p.wraw || !p.wtrans || !p.y || p.m < 4 || p.K < 8 || p.N < 8 || p.K % 8 ||
        p.N % 8 || p.h % 2 || p.w % 2 || (int64_t)p.n * p.h * p.w != p.m)
        return hipErrorInvalidValue;
    if (p.epi == EPI_BNBWD && (!p.part || !p.ex || !p.e_mean || !p.e_rstd || !p.e_gamma || !p.e_beta ||
                               (p.e_zsrc && !p.ex2)))
        return hipErrorInvalidValue;
    const int bm = pu_bm(p.m, p.N), ntiles = (int)ceil_div(p.N, kPuBN);
    const int64_t blocks = ceil_div(p.m / 4, bm) * ntiles;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    const double m = (double)p.m;
    double by = m / 4.0 * p.K + m * p.N + (double)p.K * p.N;
    if (p.epi == EPI_BNBWD) by += m * p.N;
    if (p.accumulate) by += m * p.N;
    TraceScope tr(KC_CONV, KID_CONV_1X1, s, 2.0 * by, 2.0 * (m / 4.0) * p.K * p.N);
    if (bm == 32) run_poolup<32>(p, ntiles, (unsigned)blocks, s);
    else run_poolup<64>(p, ntiles, (unsigned)blocks, s);
    return hipGetLastError();
}

}  // namespace bnr
