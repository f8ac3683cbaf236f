// conv3x3.hip -- persistent 3x3 CONV (stride 1, zero padding 1), forward and
// data gradient, on the gfx950 matrix cores with the BN fission/fusion
// prologues and epilogues.
//
// The GEMM rows are the positions of the zero-padded image grid,
// P = (img (H + 2) + hp) (W + 2) + wp: a 3x3 tap is then the constant row
// offset (dh (W + 2) + dw) for every output row, padding taps read zero rows,
// and an A fragment is one LDS read at a wave-uniform row plus a fixed lane
// offset (no per-lane masks or address arithmetic in the matrix-core loop).
// Outputs at padding positions are computed and discarded (2 (H + W + 2) of
// every (H + 2)(W + 2) positions).
// One 512-thread workgroup per CU owns a contiguous range of positions
// [P0, P1) and walks it in tiles of TR rows (64; 128 where one wave covers
// all channels of a row).
//   * Weights: each of the 8 waves owns a 32-channel slice of the GEMM K
//     (input channels) and a 32-column slice of the outputs, and keeps the
//     matrix-core fragments of that slice for all nine taps in registers
//     (72 VGPRs).  The data gradient's [n][k] rows are fragments as they lie in
//     memory; the forward's [k][n] rows are copied to LDS as they are and
//     read by transposing reads.  The remaining 8 / (K slices x N slices)
//     waves split the rows of a tile.
//   * Inputs: a ring buffer of position rows in LDS: the window of the current
//     tile, [p0 - (W+3), p0 + TR + W + 3), and the TR rows the next one adds,
//     so each input pixel is read from HBM and transformed by the prologue
//     once (no halo re-reads inside a workgroup); padding positions are
//     written as zeros.
// One barrier per tile.  Between two barriers the matrix cores work on tile t
// (partial tiles of the K slices to one of two float32 buffers in LDS), the
// epilogue runs on tile t - 1 (the other buffer) and the rows of tile t + 1
// are transformed into the ring; none of the three depends on another.  Half
// of the waves (one of the two of each SIMD) run the matrix-core part first,
// the other half last, so a SIMD's matrix cores and its vector units are busy
// at the same time.  Global loads (ring rows and epilogue operands) go to U
// register sets and stay in flight for U - 1 tiles.  Zero padding applies to
// the CONV input, i.e. after BN and ReLU.  The float32 partial tiles of the K
// slices are added in LDS in a fixed order.
//
// The epilogue reads whole 16-byte channel vectors of one pixel row, so every
// global access is coalesced, and keeps the per-channel statistics of the
// workgroup's rows in registers: one partial row per workgroup.  Prologue /
// epilogue modes are those of conv_rows.hip.
//
// What bounds it: instructions issued per wave, not HBM (loading the same
// rows over and over saved 3 of 46 us).  Two phases per 128-row tile with a
// position decode per row and a ring wrap per fragment took 840 instructions
// per wave and phase pair, half of them scalar; the walkers (p3_step) and one
// address per filter row leave about 350.  128 -> 32 channels forward on
// 64 images of 56 x 56: 40.2 -> 32 us; its data gradient with the BN-backward
// epilogue: 51 -> 44 us (HBM floor 23); 64 -> 64 channels, 128 images,
// forward: 73 -> 50 us (averages of a kernel trace).  Slower: 768 threads (three waves per SIMD), 8-byte
// vectors so that every wave holds rows of each part, all three parts in one
// basic block with the matrix-core work interleaved (34.6, 36, 36-39 us
// against 33.5, by HIP events).
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "tiles.hpp"
#include "trace.hpp"

namespace bnr {

constexpr int kP3Threads = 512;
constexpr int kP3MaxW = 61;         // widest image row (a tile and its 2 (W + 3) halo rows in p3_fill batches)
constexpr int kP3MaxH = 896;        // tallest image that has been run (nothing below depends on it)

// Rows of a tile with wk x wn channel slices (every wave has at least 16), the
// ring batches (of one tile's rows) that cover a tile's window, the ring rows
// (one batch more: the one being written while the window is read), and the
// ring rows copied past its end, so that the rows a wave reads for one filter
// row of a tile are contiguous wherever they start.
constexpr int p3_tile_rows(int wk, int wn) { return wk * wn >= 2 ? 64 : 128; }
constexpr int p3_fill(int tr) { return (tr + 2 * (kP3MaxW + 3) + tr - 1) / tr; }
constexpr int p3_ring(int tr) { return (p3_fill(tr) + 1) * tr; }
constexpr int p3_copies(int wk, int wn) { return p3_tile_rows(wk, wn) * wk * wn / 8 + 2; }

// LDS layout (bytes): [ring: ring rows, then the copies; lda bf16 per row]
// [stage: the forward's weights Ws[9][KP][NP] bf16 at the start; afterwards
// two float32 buffers red[WK][TR][ldr] of K-slice partial tiles, and finally
// the statistics scratch]
// [coefficients: 3 KP + 4 NP floats].
struct P3Adv { int da, db, dpix; };   // positions as rows and columns (mod the image) and pixels
struct P3Geom {
    int KP, NP;
    int PW, PH, MP;                 // padded row length W + 2, image height H + 2, positions n PH PW
    int grid, mp_q, mp_r;           // workgroups and MP = mp_q grid + mp_r (set by the launcher)
    P3Adv ring_adv, epi_adv;        // advance of the ring rows and of the epilogue rows from one batch / tile to the next
    size_t ring_bytes, stage_bytes, lds;
};

static P3Geom p3_geom(int K, int N, int W)
{
    P3Geom g;
    g.KP = K <= 32 ? 32 : (K <= 64 ? 64 : 128);
    g.NP = N <= 32 ? 32 : (N <= 64 ? 64 : 128);
    const int wk = g.KP / 32, wn = g.NP / 32, tr = p3_tile_rows(wk, wn);
    g.ring_bytes = (size_t)(p3_ring(tr) + p3_copies(wk, wn)) * (g.KP + 8) * 2;
    g.PW = W + 2;
    g.PH = 0; g.MP = 0; g.ring_adv = g.epi_adv = P3Adv{0, 0, 0};   // set by the launcher
    g.grid = 1; g.mp_q = 0; g.mp_r = 0;
    const size_t wst = (size_t)9 * g.KP * g.NP * 2;
    const size_t red = (size_t)2 * wk * tr * (g.NP + 4) * 4;
    const size_t stats = (size_t)2 * (kP3Threads / (g.NP / 8)) * g.NP * 4;
    g.stage_bytes = wst > red ? wst : red;
    if (stats > g.stage_bytes) g.stage_bytes = stats;
    g.lds = g.ring_bytes + g.stage_bytes + (size_t)(3 * g.KP + 4 * g.NP) * 4;
    return g;
}

// One position of the padded grid, kept as its column and row less one (wq in
// [-1, W], hq in [-1, H]: both in range means a pixel) with NO byte offsets of
// its pixel in operands of different pixel strides, and advanced by a tile's
// rows at a time: adds and selects only (a division or a multiply-shift decode
// per row and tile was most of the kernel's instructions).  Positions before
// the first image are padding; those after the last have offsets past the end
// of every view (raw-buffer loads return zeros), and their outputs are not
// stored.
template <int NO> struct P3Walk { int wq, hq; uint32_t off[NO]; };
template <int NO>
__device__ __forceinline__ void p3_start(P3Walk<NO> &w, int P, const P3Geom &g, int H, int W, const int *ld)
{
    const int q = P + g.PH * g.PW;                            // P >= -(PW + 1): one image earlier is >= 0
    const int t = q / g.PW, img = t / g.PH;
    w.wq = q - t * g.PW - 1;
    w.hq = t - img * g.PH - 1;
    const int pix = ((img - 1) * H + w.hq) * W + w.wq;
    #pragma unroll
    for (int i = 0; i < NO; i++) w.off[i] += (uint32_t)(pix * ld[i]) * 2u;   // (the caller put its channel there)
}
template <int NO>
__device__ __forceinline__ void p3_step(P3Walk<NO> &w, const P3Adv &a, const P3Geom &g, int W, const int *ld)
{
    w.wq += a.db;
    const bool cw = w.wq >= g.PW - 1;
    w.wq -= cw ? g.PW : 0;
    w.hq += a.da + (cw ? 1 : 0);
    const bool ch = w.hq >= g.PH - 1;
    w.hq -= ch ? g.PH : 0;
    #pragma unroll
    for (int i = 0; i < NO; i++)
        w.off[i] += (uint32_t)(a.dpix * ld[i]) * 2u + (cw ? (uint32_t)(-4 * ld[i]) : 0u) +
                    (ch ? (uint32_t)(-4 * W * ld[i]) : 0u);
}
template <int NO> __device__ __forceinline__ bool p3_is_pixel(const P3Walk<NO> &w, int H, int W)
{
    return ((unsigned)w.wq < (unsigned)W) & ((unsigned)w.hq < (unsigned)H);
}

// WK x WN: 32-channel K slices x 32-column N slices (one per wave); the
// other 8 / (WK WN) waves split the tile rows.  The epilogue kind EK and the
// prologue PC are compile-time, so each part is straight-line code and the
// compiler's memory counters stay exact across it (a runtime mode switch
// makes it wait for every outstanding load at each branch).
// PC: PC3_BNGRAD (the deferred BN input gradient, which reads a second
// operand), PC3_BNRELU (the forward BN+ReLU with the statistics epilogue),
// PC3_RUNTIME (PRO_NONE / PRO_BNRELU / PRO_RELU chosen at run time).
// PC3_BNRELU_SAVE: BN+ReLU whose result z is also stored (the materialised
// O2' sweep; each workgroup stores the positions of its own range once).
enum { PC3_RUNTIME = 0, PC3_BNGRAD = 1, PC3_BNRELU = 2, PC3_BNRELU_SAVE = 3 };
// The BN-backward epilogue reading the stored z (p.e_zsrc) is an epilogue kind
// of its own, so the plain BN-backward epilogue carries none of its code.
constexpr int EK3_BNBWD_Z = 7;

// BRIEF: ranges of at most two tiles (small images, or few): the ring holds all
// their rows at once and there is nothing to overlap, so the tiles' products
// come one after the other, then their epilogues, without the loop's barriers
// and the parts that have nothing to do.  Data gradient 32 -> 128 channels on 76
// images of 32 x 8: 18.6 us in the loop (three iterations), 16.0 this way, 16.7
// in 128-row tiles of two phases; forward 15.4, 14.1, 16.7.  A kernel of its
// own: both in one spilled registers (18.0 and 18.8 for that data gradient).
template <int WK, int WN, int EK, int PC, bool BRIEF>
__global__ __launch_bounds__(kP3Threads) void k_conv3x3(RowsParams p, P3Geom g)
{
    constexpr bool BNG = PC == PC3_BNGRAD;
    constexpr bool ZK = EK == EK3_BNBWD_Z;                        // BN backward from the stored z
    constexpr bool BNB = EK == EK_BNBWD || ZK;                    // BN-backward epilogue
    constexpr bool SAVE = PC == PC3_BNRELU_SAVE;
    const int pro = PC == PC3_BNRELU || SAVE ? PRO_BNRELU : (PC == PC3_BNGRAD ? PRO_BNGRAD : p.pro);
    using T = bf16_t;
    using M = Mfma<T>;
    constexpr int VEC = 8;
    constexpr int KPC = 32 * WK, NPC = 32 * WN;
    constexpr int TR = p3_tile_rows(WK, WN);                     // rows per tile
    constexpr int WR = 8 / (WK * WN);                            // row groups
    constexpr int RB = TR / (16 * WR);                           // 16-row blocks per wave
    constexpr int VPK = KPC / VEC, SROWS = kP3Threads / VPK;     // vectors per ring row; rows per staging pass
    constexpr int NVA = (TR + SROWS - 1) / SROWS;                // ring vectors per thread and tile
    constexpr int VPRO = NPC / VEC, RSTEP = kP3Threads / VPRO;
    constexpr int RPT = (TR + RSTEP - 1) / RSTEP;                // epilogue rows per thread
    constexpr bool READS = EK == EK_STORE_ACC || EK == EK_RELUMASK || BNB;
    constexpr int NVB = BNG ? NVA : 1, NVX = READS ? RPT : 1;
    constexpr int FB = p3_fill(TR), RING = p3_ring(TR);          // batches of the first window, ring rows
    constexpr int COPIES = 16 * RB + 2;
    static_assert(COPIES == p3_copies(WK, WN) && COPIES <= TR, "ring copies");
    constexpr int U = 3;                                          // register sets of loads in flight
    static_assert(WR * WK * WN == 8 && RB >= 1, "wave layout");
    extern __shared__ __align__(16) unsigned char smem[];
    T *ring = reinterpret_cast<T *>(smem);                       // [RING + COPIES][lda]
    unsigned char *stage = smem + g.ring_bytes;
    T *Ws = reinterpret_cast<T *>(stage);                        // [9][KPC][NPC] (start only)
    float *red = reinterpret_cast<float *>(stage);               // [2][WK][TR][ldr]
    float *coef = reinterpret_cast<float *>(stage + g.stage_bytes);
    float *epi = coef + 3 * KPC;
    constexpr int lda = KPC + 8, ldr = NPC + 4;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % WR, wk = (wave / WR) % WK, wn = wave / (WR * WK);
    const int K = p.K, N = p.N;
    const int m = (int)p.m;                                      // launcher: m < 2^30
    const int H = p.h, W = p.w, PW = g.PW;
    // range [floor(b MP / G), floor((b + 1) MP / G)) in 32-bit arithmetic
    // (b mp_q <= MP < 2^30, b mp_r < G^2): no 64-bit division, whose branches
    // would serialise the kernel-argument loads around it
    const int bid = blockIdx.x;
    const int P0 = bid * g.mp_q + (int)((uint32_t)(bid * g.mp_r) / (uint32_t)g.grid);
    const int P1 = (bid + 1) * g.mp_q + (int)((uint32_t)((bid + 1) * g.mp_r) / (uint32_t)g.grid);
    const int H1 = PW + 1;
    const T *wsrc = reinterpret_cast<const T *>(p.wraw);
    constexpr uint32_t ES = sizeof(T);
    // operand views as raw buffers (launcher guarantees each spans < 2^31 bytes)
    const int a_ldc = (int)p.a_ldc, a2_ldc = (int)p.a2_ldc, y_ldc = (int)p.y_ldc, ex_ldc = (int)p.ex_ldc;
    const uint32_t abytes = (uint32_t)(((int64_t)(m - 1) * a_ldc + K) * ES);
    const uint32_t a2bytes = BNG ? (uint32_t)(((int64_t)(m - 1) * a2_ldc + K) * ES) : 0u;
    const __amdgpu_buffer_rsrc_t ybuf = buf_view(p.y, (uint32_t)(((int64_t)(m - 1) * y_ldc + N) * ES));
    const int side_ldc = (int)p.side_ldc, ex2_ldc = (int)p.ex2_ldc;
    const __amdgpu_buffer_rsrc_t sbuf = buf_view(SAVE ? p.side : p.a,
                                                 SAVE ? (uint32_t)(((int64_t)(m - 1) * side_ldc + K) * ES) : 0u);
    const __amdgpu_buffer_rsrc_t xbuf = buf_view(p.ex ? p.ex : p.y,
                                                 p.ex ? (uint32_t)(((int64_t)(m - 1) * ex_ldc + N) * ES) : 0u);

    // ---- ring rows: this thread's channel vector av of rows ar0, ar0 + SROWS
    // of each batch of TR consecutive positions (batch b: from P0 - H1 + b TR);
    // keep: all ones for a pixel, 0 for padding ----
    constexpr bool STAGES_ALL = SROWS <= TR;                     // else the last waves hold no row of a batch
    const bool stages = STAGES_ALL || wave * 64 < TR * VPK;
    const int av = tid % VPK, ar0 = tid / VPK, ac = av * VEC;
    const bool ac_ok = ac < K && (STAGES_ALL || ar0 < TR);
    constexpr int NOR = BNG ? 2 : 1;
    const int rld[2] = {a_ldc, SAVE ? side_ldc : a2_ldc};
    struct Rows { vec16 a[NVA]; vec16 b[NVB]; uint32_t keep[NVA]; };
    P3Walk<NOR> rw[NVA];
    #pragma unroll
    for (int j = 0; j < NVA; j++) {
        #pragma unroll
        for (int i = 0; i < NOR; i++) rw[j].off[i] = (uint32_t)ac * ES;
        p3_start(rw[j], P0 - H1 + ar0 + j * SROWS, g, H, W, rld);
    }
    const int NB = (P1 - P0 + 2 * H1 + TR - 1) / TR;             // batches that an output of this range needs
    auto load_rows = [&](int b, Rows &bt) __attribute__((always_inline)) {
        // (a batch past the last needed one reads nothing: an empty view)
        const __amdgpu_buffer_rsrc_t av_ = buf_view(p.a, b < NB ? abytes : 0u);
        const __amdgpu_buffer_rsrc_t bv_ = buf_view(BNG ? p.a2 : p.a, b < NB ? a2bytes : 0u);
        #pragma unroll
        for (int j = 0; j < NVA; j++) {
            const bool px = p3_is_pixel(rw[j], H, W);
            bt.keep[j] = px ? 0xffffffffu : 0u;
            const bool ok = px & ac_ok;
            bt.a[j] = bld16(av_, ok ? rw[j].off[0] : kBufOff);
            if (BNG) bt.b[j < NVB ? j : 0] = bld16(bv_, ok ? rw[j].off[NOR - 1] : kBufOff);
            p3_step(rw[j], g.ring_adv, g, W, rld);
        }
    };
    // ---- prologue loads, in the order they are needed: the per-channel
    // parameters (thread c holds channel c; KPC, NPC <= 128), the weights,
    // then the first tile's window (positions [P0 - H1, P0 + TR + H1)).  Loads
    // complete in issue order for the wait counter, so the weights wait only
    // for the parameters, and the window stays in flight.
    //   BNRELU: z = max(x * c0 + c1, 0) with c0 = gamma*rstd, c1 = beta - mean*gamma*rstd
    //   BNGRAD: d = c0 * dy + c1 * x + c2  (the deferred BN input gradient: deferred_coef_of)
    float q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f, q4 = 0.f;
    if (tid < K && pro == PRO_BNRELU) {
        q0 = p.p_gamma[tid]; q1 = p.p_beta[tid]; q2 = p.p_mean[tid]; q3 = p.p_rstd[tid];
    } else if (tid < K && pro == PRO_BNGRAD) {
        q1 = p.p_mean[tid]; q2 = p.p_rstd[tid];
        if (p.p_split) { q0 = p.p_alpha[tid]; q3 = p.p_betap[tid]; }
        else { q0 = p.p_gamma[tid]; q3 = p.p_dgamma[tid]; q4 = p.p_dbeta[tid]; }
    }
    float ep0 = 0.f, ep1 = 1.f, epg = 0.f, epb = 0.f;
    if (tid < N && BNB) { ep0 = p.e_mean[tid]; ep1 = p.e_rstd[tid]; epg = p.e_gamma[tid]; epb = p.e_beta[tid]; }
    if (tid < N && EK == EK_STATS && p.e_shift) ep0 = p.e_shift[tid];     // statistics of y - shift

    // this wave's weight fragments: K slice wk, columns wn*32 + {0, 16}, nine taps
    typename M::frag bfr[9][2];
    const __amdgpu_buffer_rsrc_t wbuf = buf_view(wsrc, (uint32_t)(9 * K * N * ES));
    constexpr int NW = (9 * KPC * VPRO + kP3Threads - 1) / kP3Threads;   // forward: 16-byte vectors per thread
    vec16 wv[NW];
    if (!p.wtrans) {      // W[tap][k][n] rows of n (k = c_in, n = c_out), copied as they are
        #pragma unroll
        for (int u = 0; u < NW; u++) {
            const int i = tid + u * kP3Threads;
            const int row = i / VPRO, n0 = (i % VPRO) * VEC, tap = row / KPC, k = row % KPC;
            const bool ok = tap < 9 && k < K && n0 < N;
            wv[u] = bld16(wbuf, ok ? (uint32_t)((tap * K + k) * N + n0) * ES : kBufOff);
        }
    } else {              // W[8 - tap][n][k] (n = c_in, k = c_out): rows of k are fragments
        #pragma unroll
        for (int tap = 0; tap < 9; tap++)
            #pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                const int n = wn * 32 + cb * 16 + (lane & 15), k0 = wk * 32 + (lane >> 4) * M::KPL;
                const bool ok = n < N && k0 < K;
                const vec16 v = bld16(wbuf, ok ? (uint32_t)(((8 - tap) * N + n) * K + k0) * ES : kBufOff);
                bfr[tap][cb] = M::from_words(v.u);
            }
    }
    constexpr int NFILL = BRIEF ? FB + 1 : FB;       // BRIEF: the whole ring
    Rows fill[NFILL];
    #pragma unroll
    for (int f = 0; f < NFILL; f++) load_rows(f, fill[f]);
    if (!p.wtrans) {
        #pragma unroll
        for (int u = 0; u < NW; u++) {
            const int i = tid + u * kP3Threads;
            if (i < 9 * KPC * VPRO) *reinterpret_cast<vec16 *>(Ws + i * VEC) = wv[u];
        }
    }
    // ---- per-channel prologue / epilogue parameters -> LDS ----
    if (tid < KPC) {
        const int c = tid;
        float c0 = 0.f, c1 = 0.f, c2 = 0.f;
        if (c < K && pro == PRO_BNRELU) bn_coef(q0, q1, q2, q3, c0, c1);
        else if (c < K && pro == PRO_BNGRAD) deferred_coef_of(p.p_split, 1.0f / (float)m, q0, q1, q2, q3, q4, c0, c1, c2);
        coef[c] = c0; coef[KPC + c] = c1; coef[2 * KPC + c] = c2;
    }
    if (tid < NPC) {
        const int c = tid;
        float e0 = ep0, e1 = ep1, e2 = 0.f, e3 = 0.f;
        if (c < N && BNB) {      // mean, rstd and the forward's y = x c0 + c1
            bn_coef(epg, epb, e0, e1, e2, e3);
            // e_zsrc: the operand is the stored z = relu(y): mask [z > 0] as
            // fma(z, 1, 0) > 0, xhat = (z - beta) / gamma, unless the channel's
            // vector holds a gamma = 0 channel (its threads read x: ex2)
            bool zv = ZK;
            if (zv) {                              // (the eight loads together, then the test)
                float ga[VEC];
                #pragma unroll
                for (int i = 0; i < VEC; i++) ga[i] = p.e_gamma[(c & ~(VEC - 1)) + i];
                #pragma unroll
                for (int i = 0; i < VEC; i++) zv = zv && ga[i] != 0.f;
            }
            if (zv) { e0 = p.e_beta[c]; e1 = 1.0f / p.e_gamma[c]; e2 = 1.f; e3 = 0.f; }
        }
        epi[c] = e0; epi[NPC + c] = e1; epi[2 * NPC + c] = e2; epi[3 * NPC + c] = e3;
    }
    __syncthreads();
    if (!p.wtrans) {      // eight consecutive k of one column per lane: transposing reads
        const int g16 = lane >> 4, j16 = lane & 15;
        #pragma unroll
        for (int tap = 0; tap < 9; tap++)
            #pragma unroll
            for (int cb = 0; cb < 2; cb++)
                bfr[tap][cb] = tr_frag(Ws + (tap * KPC + wk * 32 + 8 * g16 + (j16 >> 2)) * NPC + wn * 32 + cb * 16 +
                                           4 * (j16 & 3), NPC);
    }
    // epilogue channels of this thread are fixed (their BN parameters are
    // read from LDS per tile: registers are the occupancy limit)
    const int v = tid % VPRO, r0 = tid / VPRO;
    const int n = v * VEC;
    const bool col_ok = n < N;
    constexpr bool zsrc = ZK;
    bool zs = zsrc && col_ok;                      // this thread's vector reads z (else x)
    if (zsrc) {                                    // (the eight loads together, then the test)
        float ga[VEC];
        #pragma unroll
        for (int e = 0; e < VEC; e++) ga[e] = p.e_gamma[col_ok ? n + e : 0];
        #pragma unroll
        for (int e = 0; e < VEC; e++) zs = zs && ga[e] != 0.f;
    }
    const char *zsrc_base = reinterpret_cast<const char *>(zs ? p.ex : (p.ex2 ? p.ex2 : p.ex));
    const int zsrc_ldc = zs ? ex_ldc : ex2_ldc;
    const uint32_t zsrc_off0 = col_ok ? (uint32_t)n * ES : 0u;

    // ---- prologue transform of batch b, then the ring writes (slot0: its ring
    // slot, a multiple of TR).  The mode switch is wave-uniform and outside the
    // vector loop; padding rows are zeroed by the ReLU's upper clamp (BNRELU)
    // or on the packed words; only the copies of the first ring rows are
    // written under a branch (around stores, no loads). ----
    float kc0[VEC], kc1[VEC];                        // BNRELU: this thread's channels' coefficients
    if (pro == PRO_BNRELU) { lds_f8(coef + ac, kc0); lds_f8(coef + KPC + ac, kc1); }
    else
        #pragma unroll
        for (int e = 0; e < VEC; e++) { kc0[e] = 0.f; kc1[e] = 0.f; }
    T *ring_w = ring + ar0 * lda + ac;
    P3Walk<1> sw[SAVE ? NVA : 1];                    // SAVE: the staged rows (behind the loads by FB + U batches)
    if (SAVE)
        #pragma unroll
        for (int j = 0; j < NVA; j++) {
            sw[j].off[0] = (uint32_t)ac * ES;
            p3_start(sw[j], P0 - H1 + ar0 + j * SROWS, g, H, W, rld + 1);
        }
    auto store_rows = [&](int b, int slot0, Rows &bt) __attribute__((always_inline)) {
        vec16 outv[NVA];
        if (BNG) {                                        // PRO_BNGRAD: d = c0 dy + c1 x + c2
            float c0[VEC], c1[VEC], c2[VEC];
            lds_f8(coef + ac, c0);
            lds_f8(coef + KPC + ac, c1);
            lds_f8(coef + 2 * KPC + ac, c2);
            #pragma unroll
            for (int j = 0; j < NVA; j++) {
                float f[VEC], x[VEC];
                Elem<T>::unpack(bt.a[j], f);
                Elem<T>::unpack(bt.b[j < NVB ? j : 0], x);
                #pragma unroll
                for (int e = 0; e < VEC; e++) f[e] = __builtin_fmaf(c0[e], f[e], __builtin_fmaf(c1[e], x[e], c2[e]));
                outv[j] = Elem<T>::pack(f);
                #pragma unroll
                for (int i = 0; i < 4; i++) outv[j].u[i] &= bt.keep[j];
            }
        } else if (pro == PRO_BNRELU) {                   // z = max(x c0 + c1, 0); padding: clamped to [0, 0]
            #pragma unroll
            for (int j = 0; j < NVA; j++) {
                float f[VEC];
                Elem<T>::unpack(bt.a[j], f);
                const float top = __uint_as_float(bt.keep[j] & 0x7f800000u);     // +inf or 0
                #pragma unroll
                for (int e = 0; e < VEC; e++) f[e] = __builtin_amdgcn_fmed3f(bn_lin(f[e], kc0[e], kc1[e]), 0.f, top);
                outv[j] = Elem<T>::pack(f);
            }
        } else if (pro == PRO_RELU) {                     // (padding rows load zeros)
            #pragma unroll
            for (int j = 0; j < NVA; j++) {
                float f[VEC];
                Elem<T>::unpack(bt.a[j], f);
                #pragma unroll
                for (int e = 0; e < VEC; e++) f[e] = __builtin_fmaxf(f[e], 0.f);
                outv[j] = Elem<T>::pack(f);
            }
        } else {
            #pragma unroll
            for (int j = 0; j < NVA; j++) outv[j] = bt.a[j];     // padding rows load zeros
        }
        T *dst = ring_w + slot0 * lda;
        #pragma unroll
        for (int j = 0; j < NVA; j++) *reinterpret_cast<vec16 *>(dst + j * SROWS * lda) = outv[j];
        if (slot0 == 0)
            #pragma unroll
            for (int j = 0; j < NVA; j++)
                if (j * SROWS < COPIES && ar0 + j * SROWS < COPIES)
                    *reinterpret_cast<vec16 *>(dst + (RING + j * SROWS) * lda) = outv[j];
        if (SAVE)
            #pragma unroll
            for (int j = 0; j < NVA; j++) {
                const int q = b * TR - H1 + ar0 + j * SROWS;     // stored by the workgroup that owns the position
                const bool ok = (q >= 0) & (q < P1 - P0) & (bt.keep[j] != 0u) & ac_ok;
                bst16(sbuf, ok ? sw[j].off[0] : kBufOff, outv[j]);
                p3_step(sw[j], g.ring_adv, g, W, rld + 1);
            }
    };

    // ---- epilogue operand: thread = one channel vector of rows r0, r0+RSTEP, ... ----
    struct Epi { vec16 x[NVX]; uint32_t yoff[RPT]; };   // yoff: kBufOff for padding / past the end
    // ALT: a tile's rows are half of the threads' vectors; the waves of the
    // first half take the even tiles, the others the odd ones (thread r0 holds
    // row r0 of a pair of tiles)
    constexpr bool ALT = RSTEP > TR;
    static_assert(!ALT || (RSTEP == 2 * TR && RPT == 1), "epilogue rows");
    const int half = ALT ? wave * 64 / (TR * VPRO) : 0;
    auto epi_mine = [&](int tile) __attribute__((always_inline)) -> bool { return !ALT || (tile & 1) == half; };
    constexpr bool XOP = EK == EK_RELUMASK || BNB;   // an operand of its own
    constexpr int NOE = XOP ? 2 : 1;
    const int eld[2] = {y_ldc, ZK ? zsrc_ldc : ex_ldc};
    P3Walk<NOE> ew[RPT];
    float s1[VEC], s2[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; e++) { s1[e] = 0.f; s2[e] = 0.f; }
    #pragma unroll
    for (int j = 0; j < RPT; j++) {
        #pragma unroll
        for (int i = 0; i < NOE; i++) ew[j].off[i] = (uint32_t)n * ES;
        p3_start(ew[j], P0 + r0 + j * RSTEP, g, H, W, eld);
    }
    auto load_epi = [&](int t, Epi &ep) __attribute__((always_inline)) {
        const int nrows = P1 - P0 - t * TR;                      // (may be past the end: no row)
        #pragma unroll
        for (int j = 0; j < RPT; j++) {
            const int r = (ALT ? r0 % TR : r0) + j * RSTEP;
            const bool ok = p3_is_pixel(ew[j], H, W) & col_ok & (r < nrows);
            ep.yoff[j] = ok ? ew[j].off[0] : kBufOff;
            if (EK == EK_STORE_ACC) ep.x[j < NVX ? j : 0] = bld16(ybuf, ep.yoff[j]);
            else if (ZK)       // z, or x (gamma = 0 in the vector): one load from this thread's
                // source; a row that is not stored reads the thread's own channels of
                // pixel 0, because 0 times what it reads is added to their sums
                ep.x[j < NVX ? j : 0] = ldg16(zsrc_base + (ok ? ew[j].off[NOE - 1] : zsrc_off0));
            else if (XOP) ep.x[j < NVX ? j : 0] = bld16(xbuf, ok ? ew[j].off[NOE - 1] : kBufOff);
            p3_step(ew[j], g.epi_adv, g, W, eld);
        }
    };

    // ---- the first window ----
    const int NT = (P1 - P0 + TR - 1) / TR;
    Epi brief_ep[BRIEF ? 2 : 1];     // BRIEF: the tiles' epilogue operands
    if (BRIEF)
        #pragma unroll
        for (int t = 0; t < 2; t++)
            if (epi_mine(t)) load_epi(t, brief_ep[BRIEF ? t : 0]);
    if (stages)
        #pragma unroll
        for (int f = 0; f < NFILL; f++) store_rows(f, f * TR, fill[f]);

    const int lane_off = (lane & 15) * lda + wk * 32 + (lane >> 4) * M::KPL;
    int sb = wr * 16 * RB;          // ring slot of tile row (wr 16 RB) less H1
    int ss = FB * TR;               // ring slot of the batch being written

    // ---- matrix cores on tile t: 16 RB rows x 32 columns x 32 K per wave, nine taps ----
    auto mma_tile = [&](int t) __attribute__((always_inline)) {
        f32x4 acc[RB][2];               // set by the first tap's products
        // one address per filter row (the ring rows from tap column -1 on; the
        // copies make them contiguous): the taps and 16-row blocks of a filter
        // row are immediate offsets.  The next tap's fragments are read while
        // this tap's are multiplied
        const T *abase[3];
        #pragma unroll
        for (int kh = 0; kh < 3; kh++) {
            int u = sb + kh * PW;                        // (H1 - 1 = PW)
            u = u >= RING ? u - RING : u;
            abase[kh] = ring + u * lda + lane_off;
        }
        typename M::frag af[2][RB];
        auto load_tap = [&](int tap, typename M::frag *dst) __attribute__((always_inline)) {
            #pragma unroll
            for (int ib = 0; ib < RB; ib++) dst[ib] = M::load(abase[tap / 3] + (tap % 3 + ib * 16) * lda);
        };
        load_tap(0, af[0]);
        #pragma unroll
        for (int tap = 0; tap < 9; tap++) {
            if (tap + 1 < 9) load_tap(tap + 1, af[(tap + 1) % 2]);
            __builtin_amdgcn_sched_barrier(0);
            #pragma unroll
            for (int ib = 0; ib < RB; ib++) {
                if (tap == 0) {
                    M::mma0(acc[ib][0], bfr[0][0], af[0][ib]);
                    M::mma0(acc[ib][1], bfr[0][1], af[0][ib]);
                } else {
                    M::mma(acc[ib][0], bfr[tap][0], af[tap % 2][ib]);
                    M::mma(acc[ib][1], bfr[tap][1], af[tap % 2][ib]);
                }
            }
        }
        // float32 partial tile of this K slice -> LDS (the weights are the
        // matrix cores' first operand, so a lane holds four consecutive
        // channels of one position: one 16-byte write)
        float *rd = red + (t & 1) * (WK * TR * ldr);
        #pragma unroll
        for (int ib = 0; ib < RB; ib++)
            #pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                const int row = wr * 16 * RB + ib * 16 + (lane & 15);
                const int col = wn * 32 + cb * 16 + (lane >> 4) * 4;
                *reinterpret_cast<f32x4 *>(rd + (wk * TR + row) * ldr + col) = acc[ib][cb];
            }
    };
    // ---- epilogue of tile t - 1: sum of the K slices (fixed order), rounded
    // to the storage type; all outputs of this thread first (no branch, invalid
    // rows contribute zeros), then the stores back to back ----
    auto epi_tile = [&](int t, Epi &ep) __attribute__((always_inline)) {
        const float *rd = red + ((t - 1) & 1) * (WK * TR * ldr) + (ALT ? r0 % TR : r0) * ldr + n;
        vec16 vo[RPT];
        float eM[VEC], eR[VEC], eC0[VEC], eC1[VEC];
        if (BNB) {
            lds_f8(epi + n, eM);
            lds_f8(epi + NPC + n, eR);
            lds_f8(epi + 2 * NPC + n, eC0);
            lds_f8(epi + 3 * NPC + n, eC1);
        }
        #pragma unroll
        for (int j = 0; j < RPT; j++) {
            const bool ok = (int)ep.yoff[j] >= 0;
            float f[VEC];
            #pragma unroll
            for (int q = 0; q < WK; q++) {
                const float4 *src = reinterpret_cast<const float4 *>(rd + (q * TR + j * RSTEP) * ldr);
                const float4 lo = src[0], hi = src[1];
                if (q == 0) {
                    f[0] = lo.x; f[1] = lo.y; f[2] = lo.z; f[3] = lo.w;
                    f[4] = hi.x; f[5] = hi.y; f[6] = hi.z; f[7] = hi.w;
                } else {
                    f[0] += lo.x; f[1] += lo.y; f[2] += lo.z; f[3] += lo.w;
                    f[4] += hi.x; f[5] += hi.y; f[6] += hi.z; f[7] += hi.w;
                }
            }
            const vec16 cv = Elem<T>::pack(f);
            vo[j] = cv;
            if (EK == EK_STORE_ACC) {
                float old[VEC];
                Elem<T>::unpack(cv, f);
                Elem<T>::unpack(ep.x[j < NVX ? j : 0], old);
                #pragma unroll
                for (int e = 0; e < VEC; e++) f[e] += old[e];
                vo[j] = Elem<T>::pack(f);
            } else if (EK == EK_STATS) {      // (rows that are not stored count as zeros)
                vec16 cm = cv;
                const uint32_t keep = ok ? 0xffffffffu : 0u;
                #pragma unroll
                for (int i = 0; i < 4; i++) cm.u[i] &= keep;
                Elem<T>::unpack(cm, f);
                if (p.e_shift) {
                    lds_f8(epi + n, eM);
                    #pragma unroll
                    for (int e = 0; e < VEC; e++) f[e] -= ok ? eM[e] : 0.f;
                }
                #pragma unroll
                for (int e = 0; e < VEC; e++) {
                    s1[e] += f[e];
                    s2[e] = __builtin_fmaf(f[e], f[e], s2[e]);
                }
            } else if (EK == EK_RELUMASK) {
                float yv[VEC];
                Elem<T>::unpack(cv, f);
                Elem<T>::unpack(ep.x[j < NVX ? j : 0], yv);
                #pragma unroll
                for (int e = 0; e < VEC; e++) f[e] = yv[e] > 0.f ? f[e] : 0.f;
                vo[j] = Elem<T>::pack(f);
            } else if (BNB) {
                // (xhat per element, as in the other CONV kernels: rstd times the
                // finished sum instead saved 0.3% and put dgamma up to 6%
                // further from float64)
                float x[VEC];
                vec16 cm = cv;
                const uint32_t keep = ok ? 0xffffffffu : 0u;
                #pragma unroll
                for (int i = 0; i < 4; i++) cm.u[i] &= keep;
                Elem<T>::unpack(cm, f);
                Elem<T>::unpack(ep.x[j < NVX ? j : 0], x);
                #pragma unroll
                for (int e = 0; e < VEC; e++) {
                    const float xh = (x[e] - eM[e]) * eR[e];
                    const float d = bn_lin(x[e], eC0[e], eC1[e]) > 0.f ? f[e] : 0.f;
                    f[e] = d;
                    s1[e] += d;
                    s2[e] += d * xh;
                }
                vo[j] = Elem<T>::pack(f);
            }
        }
        #pragma unroll
        for (int j = 0; j < RPT; j++) bst16(ybuf, ep.yoff[j], vo[j]);
    };

    if constexpr (BRIEF) {
        __syncthreads();
        #pragma unroll 1
        for (int t = 0; t < NT; t++) {
            mma_tile(t);
            sb += TR;
        }
        __syncthreads();
        #pragma unroll
        for (int t = 0; t < 2; t++)
            if (t < NT && epi_mine(t)) epi_tile(t + 1, brief_ep[t]);
        __syncthreads();
    } else {
        // set i holds, for the iterations t = i mod U, ring batch FB + t and the
        // epilogue operand of tile t - 1
        Rows rs[U];
        Epi es[U];
        #pragma unroll
        for (int i = 0; i < U; i++) {
            load_rows(FB + i, rs[i]);
            if (i > 0 && epi_mine(i - 1)) load_epi(i - 1, es[i]);
        }
        #pragma unroll
        for (int j = 0; j < RPT; j++) es[0].yoff[j] = kBufOff;       // (no tile before the first)
        #pragma unroll
        for (int j = 0; j < NVX; j++) es[0].x[j] = zero16();
        __syncthreads();
        // iteration t (0 .. NT): tile t on the matrix cores, epilogue of tile
        // t - 1, ring rows of tile t + 1; then the set's loads for iteration t + U
        // (unconditional: past the end they read nothing)
        const bool mma_first = wave < 4;
        auto iter = [&](int t, Rows &bt, Epi &ep) __attribute__((always_inline)) {
            if (mma_first && t < NT) mma_tile(t);
            if (epi_mine(t - 1)) epi_tile(t, ep);
            if (stages && FB + t < NB) store_rows(FB + t, ss, bt);
            load_rows(FB + t + U, bt);
            if (epi_mine(t + U - 1)) load_epi(t + U - 1, ep);
            if (!mma_first && t < NT) mma_tile(t);
            sb += TR;
            if (sb >= RING) sb -= RING;
            ss += TR;
            if (ss >= RING) ss -= RING;
            __syncthreads();
        };
        for (int t = 0; t <= NT; t += U) {
            iter(t, rs[0], es[0]);
            if (t + 1 > NT) break;
            iter(t + 1, rs[1], es[1]);
            if (t + 2 > NT) break;
            iter(t + 2, rs[2], es[2]);
        }
        static_assert(U == 3, "unrolled by the register sets");
    }

    // ---- per-workgroup statistics partial row ----
    if (EK == EK_STATS || BNB) {
        #pragma unroll
        for (int e = 0; e < VEC; e++) {
            red[r0 * NPC + n + e] = s1[e];
            red[(RSTEP + r0) * NPC + n + e] = s2[e];
        }
        lds_colsum2(red, RSTEP, NPC, NPC, kP3Threads, tid, p.part + (int64_t)blockIdx.x * 2 * N,
                    p.part + (int64_t)blockIdx.x * 2 * N + N, N);
    }
}

// ------------------------------------------------------------- launchers ---
// (operands past 32-bit offsets and the summed-gradient epilogue: conv_rows)
bool conv3x3_supported(const RowsParams &p)
{
    if (p.dtype != DT_BF16 || p.taps != 9 || p.pro == PRO_POOLUP || p.e_scale || p.K > 128 || p.N > 128 || p.w > kP3MaxW ||
        p.w < 1 || p.h > kP3MaxH || p.h < 1)
        return false;
    // 32-bit pixel indices and positions, raw-buffer operand views: every span below 2^31 bytes
    const int64_t lim = (int64_t)1 << 31;
    const bool save = p.pro == PRO_BNRELU && p.side;
    if (p.m >= (lim >> 1) || (int64_t)p.n * (p.h + 2) * (p.w + 2) >= (lim >> 1) || (p.m * p.a_ldc + p.K) * 2 >= lim ||
        (p.m * p.y_ldc + p.N) * 2 >= lim || (p.a2 && (p.m * p.a2_ldc + p.K) * 2 >= lim) ||
        (p.ex && (p.m * p.ex_ldc + p.N) * 2 >= lim) || (save && (p.m * p.side_ldc + p.K) * 2 >= lim) ||
        (p.ex2 && (p.m * p.ex2_ldc + p.N) * 2 >= lim))
        return false;
    const P3Geom g = p3_geom(p.K, p.N, p.w);
    const int wk = g.KP / 32, wn = g.NP / 32;
    if (wk * wn > 4) return false;                 // every wave one K and one N slice, at least two row groups
    return g.lds <= 160 * 1024;
}

// One workgroup per 32 pixels, at most one per CU: a small image (14 x 14,
// 7 x 7) would otherwise leave most CUs idle, and each workgroup's launch
// prologue (weights, parameters, ring fill) is a fixed cost that more
// workgroups share out; a range shorter than a tile is a masked tile.
int64_t conv3x3_partial_rows(int64_t m)
{
    const int64_t tiles = ceil_div(m, 32);
    const int64_t g = device_cus();
    return tiles < g ? tiles : g;
}

template <int WK, int WN, int EK, int PC, bool BRIEF>
static hipError_t run_p3_brief(const RowsParams &p, const P3Geom &g, hipStream_t s)
{
    constexpr bool BNG = PC == PC3_BNGRAD;
    auto kern = k_conv3x3<WK, WN, EK, PC, BRIEF>;
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const double e = 2.0, m = (double)p.m;
    double a = m * p.K;
    if (BNG || PC == PC3_BNRELU_SAVE) a *= 2.0;     // second operand read / z written
    double out = m * p.N;
    if (EK == EK_STORE_ACC || EK == EK_RELUMASK || EK == EK_BNBWD || EK == EK3_BNBWD_Z) out += m * p.N;
    TraceScope tr(KC_CONV, KID_CONV_3X3, s, e * (a + out + 9.0 * p.K * p.N), 2.0 * m * 9.0 * p.K * p.N);
    hipLaunchKernelGGL(kern, dim3(g.grid), dim3(kP3Threads), g.lds, s, p, g);
    return hipGetLastError();
}

template <int WK, int WN, int EK, int PC>
static hipError_t run_p3(const RowsParams &p, const P3Geom &g0, hipStream_t s)
{
    P3Geom g = g0;
    g.grid = (int)conv3x3_partial_rows(p.m);
    g.mp_q = g.MP / g.grid;
    g.mp_r = g.MP % g.grid;
    const bool brief = g.mp_q + (g.mp_r ? 1 : 0) <= 2 * p3_tile_rows(WK, WN);
    return brief ? run_p3_brief<WK, WN, EK, PC, true>(p, g, s) : run_p3_brief<WK, WN, EK, PC, false>(p, g, s);
}

// (K slices, N slices) with WK * WN <= 4, WK in {1, 2, 4}
template <int EK, int PC>
static hipError_t run_p3_shape(const RowsParams &p, const P3Geom &g, hipStream_t s)
{
    const int wk = g.KP / 32, wn = g.NP / 32;
    switch (wk * 8 + wn) {
    case 1 * 8 + 1: return run_p3<1, 1, EK, PC>(p, g, s);
    case 1 * 8 + 2: return run_p3<1, 2, EK, PC>(p, g, s);
    case 1 * 8 + 4: return run_p3<1, 4, EK, PC>(p, g, s);
    case 2 * 8 + 1: return run_p3<2, 1, EK, PC>(p, g, s);
    case 2 * 8 + 2: return run_p3<2, 2, EK, PC>(p, g, s);
    case 4 * 8 + 1: return run_p3<4, 1, EK, PC>(p, g, s);
    default: return hipErrorInvalidValue;
    }
}

template <int PC>
static hipError_t run_p3_ek(const RowsParams &p, const P3Geom &g, int ek, hipStream_t s)
{
    switch (ek) {
    case EK_STORE: return run_p3_shape<EK_STORE, PC>(p, g, s);
    case EK_STORE_ACC: return run_p3_shape<EK_STORE_ACC, PC>(p, g, s);
    case EK_STATS: return run_p3_shape<EK_STATS, PC>(p, g, s);
    case EK_RELUMASK: return run_p3_shape<EK_RELUMASK, PC>(p, g, s);
    default: return p.e_zsrc ? run_p3_shape<EK3_BNBWD_Z, PC>(p, g, s) : run_p3_shape<EK_BNBWD, PC>(p, g, s);
    }
}

hipError_t launch_conv3x3(const RowsParams &p, hipStream_t s)
{
    if (!p.a || !p.wraw || !p.y || !conv3x3_supported(p)) return hipErrorInvalidValue;
    if (p.pro == PRO_BNRELU && (!p.p_mean || !p.p_gamma || !p.p_rstd || !p.p_beta)) return hipErrorInvalidValue;
    if (p.pro == PRO_BNGRAD && (!p.a2 || !p.p_mean || !p.p_rstd ||
                                (p.p_split ? (!p.p_alpha || !p.p_betap) : (!p.p_gamma || !p.p_dbeta || !p.p_dgamma))))
        return hipErrorInvalidValue;
    if ((p.epi == EPI_STATS || p.epi == EPI_BNBWD) && !p.part) return hipErrorInvalidValue;
    if (p.epi == EPI_BNBWD && (!p.ex || !p.e_mean || !p.e_rstd || !p.e_gamma || !p.e_beta)) return hipErrorInvalidValue;
    if (p.epi == EPI_RELUMASK && !p.ex) return hipErrorInvalidValue;
    if ((int64_t)p.n * p.h * p.w != p.m || p.m < 1) return hipErrorInvalidValue;
    const bool save = p.pro == PRO_BNRELU && p.side;
    if (p.side && (!save || p.wtrans || (p.epi != EPI_STORE && p.epi != EPI_STATS) || p.accumulate))
        return hipErrorInvalidValue;
    if (p.e_zsrc && (p.epi != EPI_BNBWD || !p.ex2)) return hipErrorInvalidValue;
    P3Geom g = p3_geom(p.K, p.N, p.w);
    g.PH = p.h + 2;
    const auto advance = [&](int positions) {
        const int rows = positions / g.PW;
        P3Adv a;
        a.db = positions % g.PW;
        a.da = rows % g.PH;
        a.dpix = rows / g.PH * (p.h * p.w) + a.da * p.w + a.db;
        return a;
    };
    const int tr = p3_tile_rows(g.KP / 32, g.NP / 32);
    g.ring_adv = advance(tr);
    g.epi_adv = advance(kP3Threads / (g.NP / 8) > tr ? 2 * tr : tr);      // (k_conv3x3: ALT)
    g.MP = (int)((int64_t)p.n * g.PH * g.PW);                     // padded positions
    const int ek = epilogue_kind(p.epi, p.accumulate, 0);
    if (save) return ek == EK_STATS ? run_p3_shape<EK_STATS, PC3_BNRELU_SAVE>(p, g, s)
                                    : run_p3_shape<EK_STORE, PC3_BNRELU_SAVE>(p, g, s);
    if (p.pro == PRO_BNGRAD) return run_p3_ek<PC3_BNGRAD>(p, g, ek, s);
    if (p.pro == PRO_BNRELU && ek == EK_STATS) return run_p3_shape<EK_STATS, PC3_BNRELU>(p, g, s);
    return run_p3_ek<PC3_RUNTIME>(p, g, ek, s);
}

}  // namespace bnr
