// net_ends.hip -- the layers at the two ends of a DenseNet training step.
//
//  * First CONV (7x7, stride 2, pad 3) with the sub-BN1 statistics epilogue
//    of the BN after it, and its weight gradient with the BN input gradient
//    formed on load (Sec. 3.2 fission/fusion applied to the network's first
//    layer; Sec. 3.1 names the 7x7 first CONV of DenseNet-121).
//  * BN -> ReLU -> 3x3/2 max pooling: forward with sub-BN2 + ReLU applied
//    while the pooling reads its input and the statistics of the pooled
//    output (the block input) in the same pass; backward with the ReLU mask
//    and the BN reductions in the pooling-gradient pass.
//  * Classifier head: BN -> ReLU -> global average pooling -> FC -> softmax
//    cross-entropy, forward and backward.
//
// First CONV on the matrix cores (bf16).  The image is staged in LDS with
// four channels per pixel (8 bytes; channels >= c_in read as 0), so for a
// filter row kh the 7 taps x 4 channels of one output pixel are 28
// consecutive elements at pixel 2*ow of the staged input row: a K step of 32
// is one filter row (tap slot 7 has zero weights) and a 16x16x32 fragment is
// one 16-byte LDS read per lane.  The weight fragments of all 7 filter rows
// stay in registers for the whole persistent loop.
#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "tiles.hpp"
#include "trace.hpp"

namespace bnr {

namespace {

constexpr int kSK = kStemK;                  // 7 taps per filter row
constexpr int kSIR = 2 * kStemRows + kSK - 2;     // staged input rows per item (9)
constexpr int kSPitch = 72;                  // LDS pitch (elements) of 64-channel rows
constexpr int kSKB = 2 * kSK;                // 16-wide k blocks of the weight gradient (14)

__host__ __device__ __forceinline__ int stem_rpx(int wo) { return 2 * wo + 6; }

// Item = (image, kStemRows consecutive output rows).
struct StemItem { int n, oh0, rows, pv; };
__device__ __forceinline__ StemItem stem_item(const StemParams &p, int64_t it)
{
    const int per = (p.ho + kStemRows - 1) / kStemRows;
    StemItem s;
    s.n = (int)(it / per);
    s.oh0 = (int)(it - (int64_t)s.n * per) * kStemRows;
    s.rows = min(kStemRows, p.ho - s.oh0);
    s.pv = s.rows * p.wo;
    return s;
}

// Stage the input rows of an item: row r <-> image row 2*oh0 - 3 + r, pixel
// j <-> image column j - 3; zero outside the image; channels >= c_in zeroed.
__device__ __forceinline__ void stem_stage_image(const StemParams &p, const StemItem &t, uint2 *img_s, int tid)
{
    const int RPX = stem_rpx(p.wo);
    const uint2 *img = reinterpret_cast<const uint2 *>(p.img);
    const uint32_t keep_lo = p.c_in >= 2 ? 0xffffffffu : 0x0000ffffu;
    const uint32_t keep_hi = p.c_in >= 4 ? 0xffffffffu : (p.c_in == 3 ? 0x0000ffffu : 0u);
    const int ih0 = 2 * t.oh0 - kStemPad;
    for (int q = tid; q < kSIR * RPX; q += kThreads) {
        const int r = q / RPX, j = q - r * RPX;
        const int ih = ih0 + r, iw = j - kStemPad;
        uint2 v = make_uint2(0u, 0u);
        if (ih >= 0 && ih < p.h && iw >= 0 && iw < p.w) {
            v = img[((int64_t)t.n * p.h + ih) * p.w + iw];
            v.x &= keep_lo;
            v.y &= keep_hi;
        }
        img_s[q] = v;
    }
}

}  // namespace

static_assert(kStemRows == 2, "the weight gradient's row of a pixel is one comparison");

// --------------------------------------------------------------------------
// First CONV forward (bf16): out[n][oh][ow][co] = sum_{kh,kw,ci} img[n][2oh-3+kh]
// [2ow-3+kw][ci] w[kh][kw][ci][co], optional per-channel sum / sum of squares
// of the stored (bf16-rounded) outputs, one partial row per workgroup.
// Wave w computes the item's 16-pixel blocks w, w+4, ... for all 64 channels.
template <bool STATS>
__global__ __launch_bounds__(kThreads, 2) void k_stem_conv(StemParams p)
{
    using M = Mfma<bf16_t>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int RPX = stem_rpx(p.wo);
    uint2 *img_s = reinterpret_cast<uint2 *>(smem);
    bf16_t *stg = reinterpret_cast<bf16_t *>(smem + (size_t)kSIR * RPX * 8);   // [4 waves][4][16][kSPitch]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g16 = lane >> 4, l16 = lane & 15;
    const int wo = p.wo;
    const int MB = (kStemRows * wo + 15) / 16;
    const int64_t items = (int64_t)p.n * ((p.ho + kStemRows - 1) / kStemRows);

    // weight fragments: K step kh, lane k = 8*g16 + e <-> kw = 2*g16 + e/4, ci = e%4
    bf16x8 bw[kSK][4];
    const bf16_t *wt = reinterpret_cast<const bf16_t *>(p.wt);
    #pragma unroll
    for (int kh = 0; kh < kSK; kh++)
        #pragma unroll
        for (int nb = 0; nb < 4; nb++) {
            uint32_t wd[4];
            #pragma unroll
            for (int e2 = 0; e2 < 4; e2++) {
                uint32_t h2[2];
                #pragma unroll
                for (int u = 0; u < 2; u++) {
                    // (an unconditional load at a clamped index, then a select:
                    // a load under a branch costs one memory round trip each)
                    const int e = 2 * e2 + u, kw = 2 * g16 + e / 4, ci = e % 4;
                    const bool ok = kw < kSK && ci < p.c_in;
                    const uint32_t v =
                        wt[ok ? ((kh * kSK + kw) * p.c_in + ci) * kStemCout + nb * 16 + l16 : nb * 16 + l16];
                    h2[u] = ok ? v : 0u;
                }
                wd[e2] = h2[0] | (h2[1] << 16);
            }
            bw[kh][nb] = M::from_words(wd);
        }

    float s1[4] = {0.f, 0.f, 0.f, 0.f}, s2[4] = {0.f, 0.f, 0.f, 0.f}, sh[4] = {0.f, 0.f, 0.f, 0.f};
    if (STATS && p.shift)                         // statistics of s - shift
        for (int nb = 0; nb < 4; nb++) sh[nb] = p.shift[nb * 16 + (threadIdx.x & 15)];
    const int lid = xcd_remap(blockIdx.x, gridDim.x);
    for (int64_t it = lid; it < items; it += gridDim.x) {
        const StemItem t = stem_item(p, it);
        stem_stage_image(p, t, img_s, tid);
        __syncthreads();
        f32x4 acc[4][4];
        #pragma unroll
        for (int mi = 0; mi < 4; mi++)
            #pragma unroll
            for (int nb = 0; nb < 4; nb++) acc[mi][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int mi = 0; mi < 4; mi++) {
            const int mb = wave + 4 * mi;
            if (mb < MB) {                                        // wave-uniform
                int pp = mb * 16 + l16;
                if (pp >= t.pv) pp = 0;                           // padding rows read pixel 0 (finite)
                const int r = pp / wo, ow = pp - r * wo;
                const bf16_t *a0 = reinterpret_cast<const bf16_t *>(img_s + 2 * r * RPX + 2 * ow + 2 * g16);
                #pragma unroll
                for (int kh = 0; kh < kSK; kh++) {
                    const bf16x8 a = M::load(a0 + (size_t)kh * RPX * 4);
                    #pragma unroll
                    for (int nb = 0; nb < 4; nb++) M::mma(acc[mi][nb], a, bw[kh][nb]);
                }
            }
        }
        // epilogue: round, statistics of the stored values, stage for coalesced stores
        #pragma unroll
        for (int mi = 0; mi < 4; mi++) {
            const int mb = wave + 4 * mi;
            if (mb < MB) {
                #pragma unroll
                for (int nb = 0; nb < 4; nb++)
                    #pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const int pp = mb * 16 + 4 * g16 + i;
                        const bf16_t b = f2bf(acc[mi][nb][i]);
                        if (STATS && pp < t.pv) {
                            const float v = bf2f(b) - sh[nb];
                            s1[nb] += v;
                            s2[nb] += v * v;
                        }
                        stg[((wave * 4 + mi) * 16 + 4 * g16 + i) * kSPitch + nb * 16 + l16] = b;
                    }
            }
        }
        __syncthreads();
        bf16_t *dst = reinterpret_cast<bf16_t *>(p.s) + ((int64_t)t.n * p.ho + t.oh0) * wo * kStemCout;
        for (int v = tid; v < t.pv * 8; v += kThreads) {
            const int pp = v >> 3, c8 = v & 7, mb = pp >> 4;
            const bf16_t *src = stg + (((mb & 3) * 4 + (mb >> 2)) * 16 + (pp & 15)) * kSPitch + c8 * 8;
            stg16(dst + (int64_t)pp * kStemCout + c8 * 8, *reinterpret_cast<const vec16 *>(src));
        }
        __syncthreads();
    }
    if (STATS) {
        #pragma unroll
        for (int nb = 0; nb < 4; nb++) {
            s1[nb] += __shfl_xor(s1[nb], 16, 64);
            s1[nb] += __shfl_xor(s1[nb], 32, 64);
            s2[nb] += __shfl_xor(s2[nb], 16, 64);
            s2[nb] += __shfl_xor(s2[nb], 32, 64);
        }
        float *red = reinterpret_cast<float *>(stg);              // [4 waves][2][64]
        if (g16 == 0)
            #pragma unroll
            for (int nb = 0; nb < 4; nb++) {
                red[(wave * 2) * kStemCout + nb * 16 + l16] = s1[nb];
                red[(wave * 2 + 1) * kStemCout + nb * 16 + l16] = s2[nb];
            }
        __syncthreads();
        if (tid < 2 * kStemCout) {
            const int k = tid / kStemCout, c = tid - k * kStemCout;
            float a = 0.f;
            for (int wv = 0; wv < 4; wv++) a += red[(wv * 2 + k) * kStemCout + c];
            p.part[(int64_t)blockIdx.x * 2 * kStemCout + k * kStemCout + c] = a;
        }
    }
}

// float32 first CONV: one thread per output element (the float32
// configuration only runs at test sizes).
__global__ __launch_bounds__(kThreads) void k_stem_conv_f32(StemParams p)
{
    const float *img = reinterpret_cast<const float *>(p.img), *wt = reinterpret_cast<const float *>(p.wt);
    float *out = reinterpret_cast<float *>(p.s);
    const int64_t total = (int64_t)p.n * p.ho * p.wo * kStemCout;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total; i += (int64_t)gridDim.x * kThreads) {
        const int co = (int)(i % kStemCout);
        const int64_t pix = i / kStemCout;
        const int ow = (int)(pix % p.wo);
        const int64_t t = pix / p.wo;
        const int oh = (int)(t % p.ho);
        const int64_t n = t / p.ho;
        float acc = 0.f;
        for (int kh = 0; kh < kSK; kh++) {
            const int ih = 2 * oh - kStemPad + kh;
            if (ih < 0 || ih >= p.h) continue;
            for (int kw = 0; kw < kSK; kw++) {
                const int iw = 2 * ow - kStemPad + kw;
                if (iw < 0 || iw >= p.w) continue;
                const float *x = img + ((n * p.h + ih) * p.w + iw) * kStemPix;
                for (int ci = 0; ci < p.c_in; ci++)
                    acc = __builtin_fmaf(x[ci], wt[((kh * kSK + kw) * p.c_in + ci) * kStemCout + co], acc);
            }
        }
        out[i] = acc;
    }
}

// --------------------------------------------------------------------------
// First CONV weight gradient (bf16): dW[kh][kw][ci][co] = sum over output
// pixels of img(patch) * g, g the gradient of the CONV output (dense, or the
// deferred input gradient of the BN after it, formed on load and rounded to
// bf16 as a materialised gradient would be).  Split-K over items: each
// workgroup writes one float32 partial of dW.  Both operands are staged
// row-major and read transposed (ds_read_b64_tr_b16): the G rows are output
// pixels x 64 channels; the patch row of pixel p for filter row kh is the 32
// elements at pixel 2*ow of staged input row kh + 2r.  Wave w owns the
// 16-wide k blocks w, w+4, ... (k = kh*32 + kw*4 + ci) for all 64 channels.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

__device__ __forceinline__ bf16x8 tr_pair(const bf16_t *lo, const bf16_t *hi)
{
    const s16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(lo));
    const s16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(hi));
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    const s16x8_t v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(bf16x8, v);
}

template <int GS>
__global__ __launch_bounds__(kThreads, 2) void k_stem_wgrad(StemParams p)
{
    using M = Mfma<bf16_t>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int RPX = stem_rpx(p.wo);
    const int wo = p.wo;
    const int PP = (kStemRows * wo + 31) / 32 * 32;
    uint2 *img_s = reinterpret_cast<uint2 *>(smem);
    bf16_t *Gs = reinterpret_cast<bf16_t *>(smem + (size_t)kSIR * RPX * 8);   // [PP][kSPitch]
    float *gco = reinterpret_cast<float *>(Gs + (size_t)PP * kSPitch);         // [3][64]
    const bf16_t *img_e = reinterpret_cast<const bf16_t *>(img_s);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g16 = lane >> 4, l16 = lane & 15;
    const int64_t m_out = (int64_t)p.n * p.ho * wo;
    const int64_t items = (int64_t)p.n * ((p.ho + kStemRows - 1) / kStemRows);

    if (GS == GB_BNGRAD && tid < kStemCout) {
        float A, B, C;
        deferred_coef(0, tid, 1.0f / (float)m_out, p.g_gamma, p.g_mean, p.g_rstd, p.g_dgamma, p.g_dbeta, nullptr,
                      nullptr, A, B, C);
        gco[tid] = A;
        gco[kStemCout + tid] = B;
        gco[2 * kStemCout + tid] = C;
    }
    __syncthreads();

    f32x4 acc[4][4];
    #pragma unroll
    for (int ki = 0; ki < 4; ki++)
        #pragma unroll
        for (int cb = 0; cb < 4; cb++) acc[ki][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // (128 images of 224 x 224: 236 us with loads, transform, barrier and
    // products in sequence, a division per staged pixel and position; 110 us
    // with the next item's loads in flight during the products.)
    // Register stage of one item: image pixel slots q = tid + j 256 of the
    // kSIR x RPX staged pixels, gradient slots (pixel tid / 8 + 32 j, channel
    // vector tid % 8).  Their rows and columns are split once; an item is a
    // base pointer and range tests (loads at a clamped position, zeroed when
    // they are written to LDS).
    constexpr int NI = (kSIR * (kStemMaxW + 6) + kThreads - 1) / kThreads, NG = (kStemRows * (kStemMaxW / 2) + 31) / 32;
    constexpr int kNever = -(1 << 28);
    int ir[NI], io[NI];
    #pragma unroll
    for (int j = 0; j < NI; j++) {
        const int q = tid + j * kThreads, r = q / RPX, iw = q - r * RPX - kStemPad;
        ir[j] = q < kSIR * RPX && iw >= 0 && iw < p.w ? r : kNever;
        io[j] = r * p.w + iw;
    }
    const uint32_t keep_lo = p.c_in >= 2 ? 0xffffffffu : 0x0000ffffu;
    const uint32_t keep_hi = p.c_in >= 4 ? 0xffffffffu : (p.c_in == 3 ? 0x0000ffffu : 0u);
    const int c8 = (tid & 7) * 8, gp0 = tid >> 3;
    float gA[8], gB[8], gC[8];
    if (GS == GB_BNGRAD) { lds_f8(gco + c8, gA); lds_f8(gco + kStemCout + c8, gB); lds_f8(gco + 2 * kStemCout + c8, gC); }
    const uint2 *img = reinterpret_cast<const uint2 *>(p.img);
    const bf16_t *gsrc = reinterpret_cast<const bf16_t *>(p.g);
    const bf16_t *gx = reinterpret_cast<const bf16_t *>(p.gx);
    const int g_ld = GS == GB_BNGRAD ? kStemCout : (int)p.g_ldc, gx_ld = (int)p.gx_ldc;
    uint2 vi[NI];
    vec16 vg[NG], vx[GS == GB_BNGRAD ? NG : 1];
    auto load_item = [&](const StemItem &t) __attribute__((always_inline)) {
        const uint2 *base = img + (int64_t)t.n * p.h * p.w;
        const int ih0 = 2 * t.oh0 - kStemPad, o0 = ih0 * p.w;
        #pragma unroll
        for (int j = 0; j < NI; j++) vi[j] = base[(unsigned)(ih0 + ir[j]) < (unsigned)p.h ? o0 + io[j] : 0];
        const int64_t q0 = ((int64_t)t.n * p.ho + t.oh0) * wo;
        const bf16_t *gb = gsrc + q0 * g_ld + c8, *xb = gx + q0 * gx_ld + c8;
        #pragma unroll
        for (int j = 0; j < NG; j++) {
            const int pp = gp0 + 32 * j < t.pv ? gp0 + 32 * j : 0;
            vg[j] = ldg16(gb + pp * g_ld);
            if (GS == GB_BNGRAD) vx[GS == GB_BNGRAD ? j : 0] = ldg16(xb + pp * gx_ld);
        }
    };
    auto store_item = [&](const StemItem &t) __attribute__((always_inline)) {
        const int ih0 = 2 * t.oh0 - kStemPad;
        #pragma unroll
        for (int j = 0; j < NI; j++) {
            const bool in = (unsigned)(ih0 + ir[j]) < (unsigned)p.h;
            if (tid + j * kThreads < kSIR * RPX)
                img_s[tid + j * kThreads] = make_uint2(in ? vi[j].x & keep_lo : 0u, in ? vi[j].y & keep_hi : 0u);
        }
        #pragma unroll
        for (int j = 0; j < NG; j++) {
            const int pp = gp0 + 32 * j;
            vec16 o = vg[j];
            if (GS == GB_BNGRAD) {
                float d[8], x[8];
                Elem<bf16_t>::unpack(vg[j], d);
                Elem<bf16_t>::unpack(vx[GS == GB_BNGRAD ? j : 0], x);
                #pragma unroll
                for (int e = 0; e < 8; e++) d[e] = __builtin_fmaf(gA[e], d[e], __builtin_fmaf(gB[e], x[e], gC[e]));
                o = Elem<bf16_t>::pack(d);
            }
            const uint32_t keep = pp < t.pv ? 0xffffffffu : 0u;
            #pragma unroll
            for (int e = 0; e < 4; e++) o.u[e] &= keep;
            if (pp < PP) *reinterpret_cast<vec16 *>(Gs + pp * kSPitch + c8) = o;
        }
    };
    StemItem t = stem_item(p, blockIdx.x < items ? blockIdx.x : 0);
    if (blockIdx.x < items) load_item(t);
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        store_item(t);
        const int pv = t.pv;
        __syncthreads();
        if (it + gridDim.x < items) {                    // the next item arrives during the matrix-core work
            t = stem_item(p, it + gridDim.x);
            load_item(t);
        }
        for (int p0 = 0; p0 < PP; p0 += 32) {
            bf16x8 b[4];
            const bf16_t *gb = Gs + (p0 + 8 * g16 + (l16 >> 2)) * kSPitch + 4 * (l16 & 3);
            #pragma unroll
            for (int cb = 0; cb < 4; cb++) b[cb] = tr_pair(gb + cb * 16, gb + 4 * kSPitch + cb * 16);
            // patch rows of this lane's two pixels (padding pixels read pixel 0)
            int plo = p0 + 8 * g16 + (l16 >> 2), phi = plo + 4;
            if (plo >= pv) plo = 0;
            if (phi >= pv) phi = 0;
            const int rlo = plo >= wo ? 1 : 0, rhi = phi >= wo ? 1 : 0;     // (items of two output rows)
            const int blo = 2 * rlo * RPX + 2 * (plo - rlo * wo) + (l16 & 3);
            const int bhi = 2 * rhi * RPX + 2 * (phi - rhi * wo) + (l16 & 3);
            #pragma unroll
            for (int ki = 0; ki < 4; ki++) {
                const int kb = wave + 4 * ki;
                if (kb < kSKB) {                                   // wave-uniform
                    const int off = ((kb >> 1) * RPX + 4 * (kb & 1)) * 4;
                    const bf16x8 a = tr_pair(img_e + (size_t)blo * 4 + off, img_e + (size_t)bhi * 4 + off);
                    #pragma unroll
                    for (int cb = 0; cb < 4; cb++) M::mma(acc[ki][cb], a, b[cb]);
                }
            }
        }
        __syncthreads();
    }
    // partial dW: C row k = kb*16 + 4*g16 + i <-> kh = kb/2, kw = 4*(kb%2) + g16, ci = i
    float *dst = p.dwpart + (int64_t)blockIdx.x * kSK * kSK * p.c_in * kStemCout;
    #pragma unroll
    for (int ki = 0; ki < 4; ki++) {
        const int kb = wave + 4 * ki;
        if (kb >= kSKB) continue;
        const int kh = kb >> 1, kw = 4 * (kb & 1) + g16;
        if (kw >= kSK) continue;
        #pragma unroll
        for (int cb = 0; cb < 4; cb++)
            #pragma unroll
            for (int i = 0; i < 4; i++)
                if (i < p.c_in) dst[((kh * kSK + kw) * p.c_in + i) * kStemCout + cb * 16 + l16] = acc[ki][cb][i];
    }
}

// float32 first-CONV weight gradient: one thread per weight, summing over all
// output pixels (test sizes).
template <int GS>
__global__ __launch_bounds__(kThreads) void k_stem_wgrad_f32(StemParams p)
{
    const int nw = kSK * kSK * p.c_in * kStemCout;
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= nw) return;
    const int co = i % kStemCout, r = i / kStemCout;
    const int ci = r % p.c_in, kw = (r / p.c_in) % kSK, kh = r / (p.c_in * kSK);
    const int64_t m_out = (int64_t)p.n * p.ho * p.wo;
    float A = 1.f, B = 0.f, C = 0.f, K = 0.f;
    if (GS == GB_BNGRAD) {
        deferred_coef(0, co, 1.0f / (float)m_out, p.g_gamma, p.g_mean, p.g_rstd, p.g_dgamma, p.g_dbeta, nullptr,
                      nullptr, A, B, C);
        K = bn_centre<float>(p.g_ctr, co);      // d = A dy + B (x - K) + C
    }
    const float *img = reinterpret_cast<const float *>(p.img);
    const float *g = reinterpret_cast<const float *>(p.g), *gx = reinterpret_cast<const float *>(p.gx);
    float acc = 0.f;
    for (int64_t q = 0; q < m_out; q++) {
        const int ow = (int)(q % p.wo);
        const int64_t t = q / p.wo;
        const int oh = (int)(t % p.ho);
        const int64_t n = t / p.ho;
        const int ih = 2 * oh - kStemPad + kh, iw = 2 * ow - kStemPad + kw;
        if (ih < 0 || ih >= p.h || iw < 0 || iw >= p.w) continue;
        const float gv = GS == GB_BNGRAD ? __builtin_fmaf(A, g[q * kStemCout + co], __builtin_fmaf(B, gx[q * p.gx_ldc + co] - K, C))
                                         : g[q * p.g_ldc + co];
        acc = __builtin_fmaf(img[((n * p.h + ih) * p.w + iw) * kStemPix + ci], gv, acc);
    }
    p.dwpart[i] = acc;
}

// --------------------------------------------------------------------------
// 3x3 / stride 2 / pad 1 max pooling (taps outside the image never win), with
// BN: y = relu(gamma*(x-mean)*rstd + beta) pooled.  The transform is monotone
// per channel (increasing for gamma > 0, decreasing for gamma < 0, constant
// for gamma = 0), so the first maximum of the transformed window is the first
// maximum of sign(gamma)*x (for gamma = 0 the first tap), and the pooled value
// is the transform of the input there.  Without BN: plain max pooling of x.
// STATS: per-channel sum and sum of squares of the stored outputs.  Row
// blocks over output pixels as in the statistics sweeps.
template <typename T, bool BN, bool STATS>
__global__ __launch_bounds__(kThreads) void k_maxpool_fwd(MaxPoolParams p, int64_t rows_per_block)
{
    constexpr int VEC = Elem<T>::VEC;
    __shared__ float red[2][STATS ? kThreads * VEC : 1];
    const int C = p.c, ho = p.ho, wo = p.wo;
    const int64_t m_out = (int64_t)p.n * ho * wo;
    const int cvec = C / VEC;
    const int vb = min(kStatsMaxVec, cvec - (int)blockIdx.y * kStatsMaxVec);
    const int ry = kThreads / vb;
    const int tid = threadIdx.x, tx = tid % vb, ty = tid / vb;
    const int c0 = ((int)blockIdx.y * kStatsMaxVec + tx) * VEC;
    float sg[VEC], k[VEC], b[VEC], kc[VEC], s1[VEC], s2[VEC], sh[VEC];
    #pragma unroll
    for (int i = 0; i < VEC; i++) { s1[i] = s2[i] = 0.f; sh[i] = 0.f; sg[i] = 1.f; k[i] = 1.f; b[i] = 0.f; kc[i] = 0.f; }
    if (STATS && p.shift && ty < ry)                                      // statistics of y - shift
        #pragma unroll
        for (int i = 0; i < VEC; i++) sh[i] = p.shift[c0 + i];
    if (BN && ty < ry) {            // (all loads in one branch: one memory round trip)
        float g[VEC], be[VEC], mu[VEC], rs[VEC];
        #pragma unroll
        for (int i = 0; i < VEC; i++) {
            g[i] = p.gamma[c0 + i]; be[i] = p.beta[c0 + i]; mu[i] = p.mean[c0 + i]; rs[i] = p.rstd[c0 + i];
            kc[i] = bn_centre<T>(p.ctr, c0 + i);
        }
        #pragma unroll
        for (int i = 0; i < VEC; i++) {
            sg[i] = g[i] > 0.f ? 1.f : (g[i] < 0.f ? -1.f : 0.f);
            bn_coef(g[i], be[i], mu[i], rs[i], k[i], b[i]);
        }
    }
    const T *x = reinterpret_cast<const T *>(p.x);
    T *y = reinterpret_cast<T *>(p.y);
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = min(m_out, r0 + rows_per_block);
    if (ty < ry) {
        for (int64_t r = r0 + ty; r < r1; r += ry) {
            const int ow = (int)(r % wo);
            const int64_t t = r / wo;
            const int oh = (int)(t % ho);
            const int64_t n = t / ho;
            float best[VEC], bv[VEC];
            #pragma unroll
            for (int i = 0; i < VEC; i++) { best[i] = -INFINITY; bv[i] = 0.f; }
            // the nine taps' loads first, at clamped positions (a load under a
            // bounds branch costs one memory round trip each), then the
            // first-maximum scan in tap order over the taps inside the image
            vec16 tv[9];
            bool tin[9];
            #pragma unroll
            for (int t9 = 0; t9 < 9; t9++) {
                const int ih = 2 * oh - 1 + t9 / 3, iw = 2 * ow - 1 + t9 % 3;
                tin[t9] = ih >= 0 && ih < p.h && iw >= 0 && iw < p.w;
                const int ihc = ih < 0 ? 0 : (ih >= p.h ? p.h - 1 : ih), iwc = iw < 0 ? 0 : (iw >= p.w ? p.w - 1 : iw);
                tv[t9] = ldg16(x + ((n * p.h + ihc) * p.w + iwc) * p.x_ldc + c0);
            }
            #pragma unroll
            for (int t9 = 0; t9 < 9; t9++) {
                if (!tin[t9]) continue;
                float f[VEC];
                Elem<T>::unpack(tv[t9], f);
                #pragma unroll
                for (int i = 0; i < VEC; i++) {
                    const float key = BN ? sg[i] * f[i] : f[i];
                    if (key > best[i]) { best[i] = key; bv[i] = f[i]; }
                }
            }
            float o[VEC];
            #pragma unroll
            for (int i = 0; i < VEC; i++) {
                o[i] = bv[i];
                if (BN) {
                    const float v = bn_lin(bv[i] - kc[i], k[i], b[i]);
                    o[i] = v > 0.f ? v : 0.f;
                }
            }
            const vec16 ov = Elem<T>::pack(o);
            stg16(y + r * p.y_ldc + c0, ov);
            if (STATS) {
                Elem<T>::unpack(ov, o);
                #pragma unroll
                for (int i = 0; i < VEC; i++) { const float d = o[i] - sh[i]; s1[i] += d; s2[i] += d * d; }
            }
        }
    }
    if (STATS) {
        const int nch = vb * VEC;
        if (ty < ry)
            #pragma unroll
            for (int i = 0; i < VEC; i++) {
                red[0][ty * nch + tx * VEC + i] = s1[i];
                red[1][ty * nch + tx * VEC + i] = s2[i];
            }
        __syncthreads();
        if (tid < nch) {
            float a = 0.f, bb = 0.f;
            for (int j = 0; j < ry; j++) { a += red[0][j * nch + tid]; bb += red[1][j * nch + tid]; }
            const int c = (int)blockIdx.y * kStatsMaxVec * VEC + tid;
            float *pr = p.part + (int64_t)blockIdx.x * 2 * C;
            pr[c] = a;
            pr[C + c] = bb;
        }
    }
}

// Backward of k_maxpool_fwd: every input pixel of the image gets the sum of the
// gradients of the windows (in row-major window order) whose first maximum it
// is.  With BN that is the gradient of the ReLU output: dy = dz [y > 0] (y
// recomputed from x) is stored and the BN reductions sum(dy), sum(dy * xhat) of
// the stored dy are accumulated; without BN dz is stored.
// A workgroup takes chunks of consecutive row pairs of
// one image; thread (ow, v) owns channel vector v of window column ow and of
// the input columns 2 ow, 2 ow + 1.  Per window row it reads two input rows
// (the third is carried: every input row is reduced over its three columns
// once, "first maximum" kept as value and column), so the first-maximum tap of
// every window, the gradients routed to a pixel block and the block's BN input
// all come from registers, except what the right-hand neighbour's windows
// hold, which goes through LDS (three row buffers, one barrier per row).
// A value wins over an earlier one only if it is greater (NaN never wins).
// What bounds it: instructions (about 1000 vector ones per row pair and wave)
// and the load round trip of each row.  128 images of 112 x 112 x 64: 240 us
// with the windows of every row pair scanned twice from global memory and
// their codes in LDS bytes, 219 us this way (HBM floor 83); 1024 or 2048
// chunks instead of 512: 228 and 252 us.
constexpr int mp_threads(int vec) { return kMaxPoolMaxWo * kMaxPoolMaxC / vec; }
template <typename T, bool BN>
__global__ __launch_bounds__(mp_threads(Elem<T>::VEC), 4) void k_maxpool_bwd(MaxPoolParams p, int pairs_per_chunk,
                                                                            int chunks_per_image, int64_t chunks)
{
    constexpr int VEC = Elem<T>::VEC, NTHR = mp_threads(VEC), CW = VEC / 4;      // CW: code words of a vector
    // row buffers of the windows' gradients and codes (with a guard vector past
    // the last column), then the partial sums
    constexpr int LD = NTHR + 16;
    __shared__ __align__(16) unsigned char raw[3 * LD * (16 + 4 * CW)];
    __shared__ __align__(16) float par[4][kMaxPoolMaxC];           // sign(gamma), c0, c1, mean
    vec16 (*g_s)[LD] = reinterpret_cast<vec16 (*)[LD]>(raw);                               // [3][LD]
    uint32_t (*c_s)[CW][LD] = reinterpret_cast<uint32_t (*)[CW][LD]>(raw + 3 * LD * 16);   // [3][CW][LD]
    float (*red)[NTHR * VEC] = reinterpret_cast<float (*)[NTHR * VEC]>(raw);               // [2][NTHR VEC]
    static_assert(sizeof(raw) >= 2 * NTHR * VEC * sizeof(float), "partial sums");
    const int C = p.c, h = p.h, w = p.w, ho = p.ho, wo = p.wo, cvec = C / VEC;
    const int tid = threadIdx.x, v = tid % cvec, ow = tid / cvec;
    const bool act = ow < wo;
    if (tid < C) {
        const float g = BN ? p.gamma[tid] : 1.f;
        float c0 = 1.f, c1 = 0.f;
        if (BN) bn_coef(g, p.beta[tid], p.mean[tid], p.rstd[tid], c0, c1);
        par[0][tid] = g > 0.f ? 1.f : (g < 0.f ? -1.f : 0.f);
        par[1][tid] = c0;
        par[2][tid] = c1;
        par[3][tid] = BN ? p.mean[tid] : 0.f;
    }
    // no window past the last column, ever: code 15 matches no tap
    for (int i = tid; i < 3 * CW * 16; i += blockDim.x) c_s[i / (CW * 16)][i / 16 % CW][(int)(wo * cvec) + i % 16] = 0x0f0f0f0fu;
    for (int i = tid; i < 3 * 16; i += blockDim.x) g_s[i / 16][wo * cvec + i % 16] = zero16();
    __syncthreads();
    const float *sgn = par[0] + v * VEC;
    float s1[VEC], s2[VEC], kc[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; e++) { s1[e] = s2[e] = 0.f; kc[e] = BN ? bn_centre<T>(p.ctr, v * VEC + e) : 0.f; }
    const T *x = reinterpret_cast<const T *>(p.x) + v * VEC;
    const T *gy = reinterpret_cast<const T *>(p.g) + v * VEC;
    T *dy = reinterpret_cast<T *>(p.y) + v * VEC;
    const int cl = 2 * ow - 1 >= 0 ? 2 * ow - 1 : 0, cm = act ? 2 * ow : 0, cr = 2 * ow + 1 < w ? 2 * ow + 1 : w - 1;
    const bool in_l = ow > 0, in_r = 2 * ow + 1 < w;
    const int clc = act ? cl : 0, crc = act ? cr : 0;

    // first maximum of an input row's three columns (value, column 0..2 in
    // cols, four bits a channel); the vectors of columns 2 ow, 2 ow + 1 stay
    // with the caller
    auto row_max = [&](const vec16 &vl, const vec16 &vm, const vec16 &vr, bool in, float *best,
                       uint32_t &cols) __attribute__((always_inline)) {
        float l[VEC], m_[VEC], r[VEC];
        Elem<T>::unpack(vl, l);
        Elem<T>::unpack(vm, m_);
        Elem<T>::unpack(vr, r);
        cols = 0u;
        // (a tap outside the image: sign(gamma) x - inf, which never wins)
        const float ol = in && in_l ? 0.f : -INFINITY, om = in ? 0.f : -INFINITY, orr = in && in_r ? 0.f : -INFINITY;
        #pragma unroll
        for (int e = 0; e < VEC; e++) {
            const float sg = BN ? sgn[e] : 1.f;
            const float kl = __builtin_fmaf(sg, l[e], ol), km = __builtin_fmaf(sg, m_[e], om);
            const float kr = __builtin_fmaf(sg, r[e], orr);
            float b = __builtin_fmaxf(kl, -INFINITY);              // (NaN never wins)
            uint32_t c = km > b ? 1u : 0u;
            b = __builtin_fmaxf(b, km);
            c = kr > b ? 2u : c;
            best[e] = __builtin_fmaxf(b, kr);
            cols |= c << (4 * e);
        }
    };

    for (int64_t ck = blockIdx.x; ck < chunks; ck += gridDim.x) {
        const int n = (int)(ck / chunks_per_image);
        const int j0 = (int)(ck - (int64_t)n * chunks_per_image) * pairs_per_chunk;
        const int hp = (h + 1) / 2, j1 = min(hp, j0 + pairs_per_chunk);
        const T *xn = x + (int64_t)n * h * w * p.x_ldc;
        const T *gn = gy + (int64_t)n * ho * wo * p.g_ldc;
        T *dn = dy + (int64_t)n * h * w * C;
        auto ldx = [&](int row, int col) __attribute__((always_inline)) {
            const int rc = row < 0 ? 0 : (row < h ? row : h - 1);
            return ldg16(xn + (int64_t)(rc * w + col) * p.x_ldc);
        };
        // the row above the chunk
        float hb[VEC];
        uint32_t hc;
        {
            const int r = 2 * j0 - 1;
            const vec16 a = ldx(r, clc), b = ldx(r, cm), c = ldx(r, crc);
            row_max(a, b, c, r >= 0, hb, hc);
        }
        vec16 xp[4], gp = zero16();                 // pixel block and gradient of the window row before
        uint32_t cp[CW];
        #pragma unroll
        for (int i = 0; i < CW; i++) cp[i] = 0x0f0f0f0fu;
        #pragma unroll
        for (int i = 0; i < 4; i++) xp[i] = zero16();
        for (int oh = j0; oh <= j1; oh++) {
            // ---- window row oh: input rows 2 oh - 1 (carried), 2 oh, 2 oh + 1 ----
            const int r0 = 2 * oh, r1 = 2 * oh + 1;
            const bool wrow = oh < ho;
            vec16 xa[3], xb[3];
            xa[0] = ldx(r0, clc); xa[1] = ldx(r0, cm); xa[2] = ldx(r0, crc);
            xb[0] = ldx(r1, clc); xb[1] = ldx(r1, cm); xb[2] = ldx(r1, crc);
            const vec16 gw = ldg16(gn + (int64_t)((wrow ? oh : ho - 1) * wo + (act ? ow : 0)) * p.g_ldc);
            float ba[VEC], bb[VEC];
            uint32_t ca, cb, code[CW];
            row_max(xa[0], xa[1], xa[2], r0 < h, ba, ca);
            row_max(xb[0], xb[1], xb[2], r1 < h, bb, cb);
            #pragma unroll
            for (int i = 0; i < CW; i++) code[i] = 0u;
            #pragma unroll
            for (int e = 0; e < VEC; e++) {
                // (a row without a value above -inf holds column 0: tap 0, as a scan that nothing wins)
                uint32_t t = (hc >> (4 * e)) & 3u;
                if (ba[e] > hb[e]) t = 3u + ((ca >> (4 * e)) & 3u);
                if (bb[e] > __builtin_fmaxf(hb[e], ba[e])) t = 6u + ((cb >> (4 * e)) & 3u);
                code[e / 4] |= t << (8 * (e % 4));
                hb[e] = bb[e];
            }
            hc = cb;
            #pragma unroll
            for (int i = 0; i < CW; i++) code[i] = wrow && act ? code[i] : 0x0f0f0f0fu;
            const int buf = oh % 3, pbuf = (oh + 2) % 3;
            if (act) {
                g_s[buf][tid] = gw;
                #pragma unroll
                for (int i = 0; i < CW; i++) c_s[buf][i][tid] = code[i];
            }
            __syncthreads();
            // ---- pixels of rows 2 j, 2 j + 1, columns 2 ow, 2 ow + 1 (j = oh - 1) ----
            if (oh > j0 && act) {
                const int j = oh - 1;
                const vec16 gpr = g_s[pbuf][tid + cvec], gwr = g_s[buf][tid + cvec];
                uint32_t cpr[CW], cwr[CW];
                #pragma unroll
                for (int i = 0; i < CW; i++) { cpr[i] = c_s[pbuf][i][tid + cvec]; cwr[i] = c_s[buf][i][tid + cvec]; }
                float a00[VEC], a01[VEC], a10[VEC], a11[VEC];      // gradients of windows (j, ow), (j, ow + 1), (j + 1, ..)
                Elem<T>::unpack(gp, a00);
                Elem<T>::unpack(gpr, a01);
                Elem<T>::unpack(gw, a10);
                Elem<T>::unpack(gwr, a11);
                float dz[4][VEC];
                #pragma unroll
                for (int e = 0; e < VEC; e++) {
                    const int sh = 8 * (e % 4), q = e / 4;
                    const uint32_t t00 = (cp[q] >> sh) & 15u, t01 = (cpr[q] >> sh) & 15u;
                    const uint32_t t10 = (code[q] >> sh) & 15u, t11 = (cwr[q] >> sh) & 15u;
                    // (row-major window order; an unmatched window adds zero)
                    dz[0][e] = t00 == 4u ? a00[e] : 0.f;
                    dz[1][e] = (t00 == 5u ? a00[e] : 0.f) + (t01 == 3u ? a01[e] : 0.f);
                    dz[2][e] = (t00 == 7u ? a00[e] : 0.f) + (t10 == 1u ? a10[e] : 0.f);
                    dz[3][e] = (t00 == 8u ? a00[e] : 0.f) + (t01 == 6u ? a01[e] : 0.f);
                    dz[3][e] += t10 == 2u ? a10[e] : 0.f;
                    dz[3][e] += t11 == 0u ? a11[e] : 0.f;
                    dz[0][e] += 0.f;                               // (0 + -0 = 0, as a sum from zero)
                }
                #pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int row = 2 * j + (i >> 1), col = 2 * ow + (i & 1);
                    if (row < h && col < w) {
                        float o[VEC];
                        T *dst = dn + (int64_t)(row * w + col) * C;
                        if (BN) {
                            float f[VEC];
                            Elem<T>::unpack(xp[i], f);
                            #pragma unroll
                            for (int e = 0; e < VEC; e++)
                                o[e] = bn_lin(f[e] - kc[e], par[1][v * VEC + e], par[2][v * VEC + e]) > 0.f ? dz[i][e] : 0.f;
                            const vec16 ov = Elem<T>::pack(o);
                            stg16(dst, ov);
                            Elem<T>::unpack(ov, o);
                            #pragma unroll
                            for (int e = 0; e < VEC; e++) {        // (xhat's rstd multiplies the finished sum)
                                s1[e] += o[e];
                                s2[e] = __builtin_fmaf(o[e], (f[e] - kc[e]) - par[3][v * VEC + e], s2[e]);
                            }
                        } else {
                            stg16(dst, Elem<T>::pack(dz[i]));
                        }
                    }
                }
            }
            xp[0] = xa[1]; xp[1] = xa[2]; xp[2] = xb[1]; xp[3] = xb[2];
            gp = gw;
            #pragma unroll
            for (int i = 0; i < CW; i++) cp[i] = code[i];
        }
        __syncthreads();                            // (the buffers' next writer is another chunk's first row)
    }
    if (BN) {
        // threads tid = v + cvec ow hold channel vector v
        #pragma unroll
        for (int e = 0; e < VEC; e++) {
            const float rs = p.rstd[v * VEC + e];
            red[0][tid * VEC + e] = act ? s1[e] : 0.f;
            red[1][tid * VEC + e] = act ? s2[e] * rs : 0.f;
        }
        __syncthreads();
        if (tid < C) {
            const int cv = tid / VEC, e = tid - cv * VEC;
            float a = 0.f, b = 0.f;
            for (int u = cv; u < wo * cvec; u += cvec) { a += red[0][u * VEC + e]; b += red[1][u * VEC + e]; }
            float *pr = p.part + (int64_t)blockIdx.x * 2 * C;
            pr[tid] = a;
            pr[C + tid] = b;
        }
    }
}

// --------------------------------------------------------------------------
// Classifier head.
// Global average pooling of relu(bn(x)): f[n][c] = (1/hw) sum_p relu(...),
// one thread per (image, channel vector), pixels summed in order.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_head_pool(HeadParams p)
{
    constexpr int VEC = Elem<T>::VEC;
    const int cvec = p.c / VEC, hw = p.h * p.w;
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= p.n * cvec) return;
    const int n = i / cvec, c0 = (i - n * cvec) * VEC;
    float k[VEC], b[VEC], kc[VEC], acc[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; e++) {
        bn_coef(p.gamma[c0 + e], p.beta[c0 + e], p.mean[c0 + e], p.rstd[c0 + e], k[e], b[e]);
        kc[e] = bn_centre<T>(p.ctr, c0 + e);
        acc[e] = 0.f;
    }
    const T *x = reinterpret_cast<const T *>(p.x);
    for (int q = 0; q < hw; q++) {
        float f[VEC];
        Elem<T>::unpack(ldg16(x + ((int64_t)n * hw + q) * p.x_ldc + c0), f);
        #pragma unroll
        for (int e = 0; e < VEC; e++) {
            const float v = bn_lin(f[e] - kc[e], k[e], b[e]);
            acc[e] += v > 0.f ? v : 0.f;
        }
    }
    const float inv = 1.0f / (float)hw;
    #pragma unroll
    for (int e = 0; e < VEC; e++) p.f[(int64_t)n * p.c + c0 + e] = acc[e] * inv;
}

// Small float32 GEMM for the FC layer: out[i][j] = sum_k A(i,k) B(k,j) (+ bias[j]),
// A(i,k) = a[i*sai + k*sak] (float32), B(k,j) = b[k*sbk + j*sbj] (TB).  16 x
// kFcBN output tiles (for the 128-image batch: 8 x 63 workgroups, two per CU
// and more), K in chunks of 64 staged in LDS with the operand's contiguous
// index running across the threads (coalesced for either orientation),
// kFcBN / 16 consecutive outputs of one row per thread (A staged [i][k]: four
// k of its row in one 16-byte LDS read), k summed in order (deterministic).
constexpr int kFcBN = 16;                 // output columns per workgroup tile
template <typename TB>
__global__ __launch_bounds__(kThreads) void k_fc_gemm(int M, int N, int K, const float *__restrict__ a, int64_t sai,
                                                      int64_t sak, const TB *__restrict__ b, int64_t sbk,
                                                      int64_t sbj, const float *__restrict__ bias,
                                                      float *__restrict__ out)
{
    constexpr int BM = 16, BN = kFcBN, BK = 64;
    __shared__ __align__(16) float As[BM][BK + 4];
    __shared__ __align__(16) float Bs[BK][BN + 4];
    const int tid = threadIdx.x, tr = tid / 16, tc = tid % 16;
    const int i0 = blockIdx.y * BM, j0 = blockIdx.x * BN;
    constexpr int OPT = BN / 16;                     // consecutive outputs per thread
    float acc[OPT];
    #pragma unroll
    for (int v = 0; v < OPT; v++) acc[v] = 0.f;
    constexpr int NA = BK * BM / kThreads, NB = BK * BN / kThreads;
    for (int k0 = 0; k0 < K; k0 += BK) {
        // every load of the chunk at a clamped index first, then the LDS
        // writes with the out-of-range elements selected to zero (a load
        // under a bounds branch costs one memory round trip each)
        float av[NA];
        TB bv[NB];                                   // raw: converted after every load is issued
        bool aok[NA], bok[NB];
        #pragma unroll
        for (int u = 0; u < NA; u++) {
            const int e = tid + u * kThreads;
            const int kk = sak == 1 ? e % BK : e / BM, ii = sak == 1 ? e / BK : e % BM;
            const int gi = i0 + ii, gk = k0 + kk;
            aok[u] = gi < M && gk < K;
            av[u] = a[(aok[u] ? gi : 0) * sai + (aok[u] ? gk : 0) * sak];
        }
        #pragma unroll
        for (int u = 0; u < NB; u++) {
            const int e = tid + u * kThreads;
            const int kk = sbk == 1 ? e % BK : e / BN, jj = sbk == 1 ? e / BK : e % BN;
            const int gj = j0 + jj, gk = k0 + kk;
            bok[u] = gj < N && gk < K;
            const int64_t off = (int64_t)(bok[u] ? gk : 0) * sbk + (int64_t)(bok[u] ? gj : 0) * sbj;
            bv[u] = b[off];
        }
        __builtin_amdgcn_sched_barrier(0);   // keep every load above the writes (the scheduler sinks them)
        #pragma unroll
        for (int u = 0; u < NA; u++) {
            const int e = tid + u * kThreads;
            const int kk = sak == 1 ? e % BK : e / BM, ii = sak == 1 ? e / BK : e % BM;
            As[ii][kk] = aok[u] ? av[u] : 0.f;
        }
        #pragma unroll
        for (int u = 0; u < NB; u++) {
            const int e = tid + u * kThreads;
            const int kk = sbk == 1 ? e % BK : e / BN, jj = sbk == 1 ? e / BK : e % BN;
            float f;
            if constexpr (sizeof(TB) == 2) f = bf2f(bv[u]);
            else f = bv[u];
            Bs[kk][jj] = bok[u] ? f : 0.f;
        }
        __syncthreads();
        #pragma unroll 4
        for (int k4 = 0; k4 < BK; k4 += 4) {
            const float4 a4 = *reinterpret_cast<const float4 *>(&As[tr][k4]);
            const float ak[4] = {a4.x, a4.y, a4.z, a4.w};
            #pragma unroll
            for (int q = 0; q < 4; q++) {
                #pragma unroll
                for (int v = 0; v < OPT; v++) acc[v] = __builtin_fmaf(ak[q], Bs[k4 + q][OPT * tc + v], acc[v]);
            }
        }
        __syncthreads();
    }
    #pragma unroll
    for (int v = 0; v < OPT; v++) {
        const int gi = i0 + tr, gj = j0 + OPT * tc + v;
        if (gi < M && gj < N) out[(int64_t)gi * N + gj] = acc[v] + (bias ? bias[gj] : 0.f);
    }
}

// Softmax cross-entropy of logits [n][K] against labels and its gradient
// dlogits = (softmax - onehot) / n: one workgroup per row, which writes the
// row's loss to loss[1 + r]; k_loss_mean then adds the rows in order
// (deterministic) into loss[0].  A label outside [0, K) gives a NaN loss.
__global__ __launch_bounds__(kThreads) void k_softmax_ce(int n, int K, const float *__restrict__ logits,
                                                         const int32_t *__restrict__ labels,
                                                         float *__restrict__ dlogits, float *__restrict__ loss)
{
    __shared__ float red[kThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = blockIdx.x;
    const float *z = logits + (int64_t)r * K;
    float mx = -INFINITY;
    for (int j = tid; j < K; j += kThreads) mx = fmaxf(mx, z[j]);
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = red[0];
    for (int w = 1; w < kThreads / 64; w++) mx = fmaxf(mx, red[w]);
    __syncthreads();
    float se = 0.f;
    for (int j = tid; j < K; j += kThreads) se += expf(z[j] - mx);
    se = wave_sum(se);
    if (lane == 0) red[wave] = se;
    __syncthreads();
    se = red[0];
    for (int w = 1; w < kThreads / 64; w++) se += red[w];
    const int lab = labels[r];
    const bool ok = lab >= 0 && lab < K;
    const float inv = 1.0f / se, invn = 1.0f / (float)n;
    for (int j = tid; j < K; j += kThreads)
        dlogits[(int64_t)r * K + j] = (expf(z[j] - mx) * inv - (j == lab ? 1.f : 0.f)) * invn;
    if (tid == 0) loss[1 + r] = ok ? logf(se) + mx - z[lab] : NAN;
}

__global__ __launch_bounds__(64) void k_loss_mean(int n, float *__restrict__ loss)
{
    if (threadIdx.x != 0) return;
    double t = 0.0;
    for (int r = 0; r < n; r++) t += (double)loss[1 + r];
    loss[0] = (float)(t / (double)n);
}

// db[j] = sum_n dlogits[n][j] (rows in order).
__global__ __launch_bounds__(kThreads) void k_colsum(int n, int K, const float *__restrict__ g, float *__restrict__ out)
{
    const int j = blockIdx.x * kThreads + threadIdx.x;
    if (j >= K) return;
    float s = 0.f;
    for (int r = 0; r < n; r++) s += g[(int64_t)r * K + j];
    out[j] = s;
}

// Head BN backward over x [m][c] (m = n*h*w): dz = df[n][c] / hw, y recomputed,
// dy = dz [y > 0] (float32, not stored);
//   HB_SPLIT: out = gamma*rstd*dy (the summed-gradient term of the BN) and the
//             partial sums of dy and dy*xhat;
//   HB_SUMS : the partial sums only;
//   HB_DX   : out = gamma*rstd*(dy - dbeta/m - xhat*dgamma/m) (dbeta, dgamma
//             from a previous HB_SUMS pass and its combine).
template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_head_bn_bwd(HeadParams p, int64_t rows_per_block)
{
    constexpr int VEC = Elem<T>::VEC;
    __shared__ float red[2][MODE == HB_DX ? 1 : kThreads * VEC];
    const int C = p.c, hw = p.h * p.w;
    const int64_t m = (int64_t)p.n * hw;
    const int cvec = C / VEC;
    const int vb = min(kStatsMaxVec, cvec - (int)blockIdx.y * kStatsMaxVec);
    const int ry = kThreads / vb;
    const int tid = threadIdx.x, tx = tid % vb, ty = tid / vb;
    const int c0 = ((int)blockIdx.y * kStatsMaxVec + tx) * VEC;
    float k[VEC], b[VEC], mu[VEC], rs[VEC], kc[VEC], gk[VEC], s1[VEC], s2[VEC], da[VEC], db[VEC];
    const float inv_hw = 1.0f / (float)hw, inv_m = 1.0f / (float)m;
    #pragma unroll
    for (int i = 0; i < VEC; i++) {
        s1[i] = s2[i] = 0.f;
        k[i] = b[i] = mu[i] = gk[i] = da[i] = db[i] = kc[i] = 0.f;
        rs[i] = 1.f;
    }
    if (ty < ry) {                  // (all loads in one branch: one memory round trip)
        float g[VEC], be[VEC];
        #pragma unroll
        for (int i = 0; i < VEC; i++) {
            const int c = c0 + i;
            mu[i] = p.mean[c]; rs[i] = p.rstd[c]; g[i] = p.gamma[c]; be[i] = p.beta[c];
            kc[i] = bn_centre<T>(p.ctr, c);
            if (MODE == HB_DX) { da[i] = p.dbeta[c]; db[i] = p.dgamma[c]; }
        }
        #pragma unroll
        for (int i = 0; i < VEC; i++) {
            bn_coef(g[i], be[i], mu[i], rs[i], k[i], b[i]);
            gk[i] = k[i];
            if (MODE == HB_DX) { da[i] *= inv_m; db[i] *= inv_m; }
        }
    }
    const T *x = reinterpret_cast<const T *>(p.x);
    T *out = reinterpret_cast<T *>(p.gx);
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = min(m, r0 + rows_per_block);
    if (ty < ry) {
        for (int64_t r = r0 + ty; r < r1; r += ry) {
            const int64_t n = r / hw;
            float f[VEC], o[VEC];
            Elem<T>::unpack(ldg16(x + r * p.x_ldc + c0), f);
            #pragma unroll
            for (int i = 0; i < VEC; i++) {
                const float dz = p.df[n * C + c0 + i] * inv_hw;
                const float xc = f[i] - kc[i];
                const float dyv = bn_lin(xc, k[i], b[i]) > 0.f ? dz : 0.f;
                const float xh = (xc - mu[i]) * rs[i];
                if (MODE == HB_DX) {
                    o[i] = gk[i] * (dyv - da[i] - xh * db[i]);
                } else {
                    o[i] = gk[i] * dyv;
                    s1[i] += dyv;
                    s2[i] += dyv * xh;
                }
            }
            if (MODE != HB_SUMS) stg16(out + r * p.gx_ldc + c0, Elem<T>::pack(o));
        }
    }
    if (MODE != HB_DX) {
        const int nch = vb * VEC;
        if (ty < ry)
            #pragma unroll
            for (int i = 0; i < VEC; i++) {
                red[0][ty * nch + tx * VEC + i] = s1[i];
                red[1][ty * nch + tx * VEC + i] = s2[i];
            }
        __syncthreads();
        if (tid < nch) {
            float a = 0.f, bb = 0.f;
            for (int j = 0; j < ry; j++) { a += red[0][j * nch + tid]; bb += red[1][j * nch + tid]; }
            const int c = (int)blockIdx.y * kStatsMaxVec * VEC + tid;
            float *pr = p.part + (int64_t)blockIdx.x * 2 * C;
            pr[c] = a;
            pr[C + c] = bb;
        }
    }
}

// --------------------------------------------------------------- launchers --
int64_t stem_groups(int64_t items) { return items < kStemMaxGroups ? (items < 1 ? 1 : items) : kStemMaxGroups; }

static size_t stem_lds(int wo, bool wgrad)
{
    const size_t img = (size_t)kSIR * stem_rpx(wo) * 8;
    if (!wgrad) return img + (size_t)4 * 4 * 16 * kSPitch * 2;
    const size_t PP = (size_t)(kStemRows * wo + 31) / 32 * 32;
    return img + PP * kSPitch * 2 + 3 * kStemCout * sizeof(float);
}

hipError_t launch_stem_conv(int dtype, const StemParams &p, bool stats, hipStream_t s)
{
    if (!p.img || !p.wt || !p.s || (stats && !p.part) || p.c_in < 1 || p.c_in > kStemPix || p.w > kStemMaxW ||
        p.ho != stem_out(p.h) || p.wo != stem_out(p.w))
        return hipErrorInvalidValue;
    const int64_t m = (int64_t)p.n * p.ho * p.wo;
    const double e = dtype == DT_BF16 ? 2.0 : 4.0;
    TraceScope tr(KC_CONV, KID_STEM_CONV, s, e * ((double)p.n * p.h * p.w * kStemPix + (double)m * kStemCout),
                  2.0 * m * kStemCout * kSK * kSK * p.c_in);
    if (dtype == DT_BF16) {
        const int64_t items = (int64_t)p.n * ((p.ho + kStemRows - 1) / kStemRows);
        const unsigned g = (unsigned)stem_groups(items);
        const size_t lds = stem_lds(p.wo, false);
        if (stats) hipLaunchKernelGGL(k_stem_conv<true>, dim3(g), dim3(kThreads), lds, s, p);
        else hipLaunchKernelGGL(k_stem_conv<false>, dim3(g), dim3(kThreads), lds, s, p);
    } else {
        const int64_t total = m * kStemCout;
        const unsigned g = (unsigned)(ceil_div(total, kThreads) < 8192 ? ceil_div(total, kThreads) : 8192);
        hipLaunchKernelGGL(k_stem_conv_f32, dim3(g), dim3(kThreads), 0, s, p);
    }
    return hipGetLastError();
}

int64_t stem_wgrad_splits(int dtype, int64_t items) { return dtype == DT_BF16 ? stem_groups(items) : 1; }

hipError_t launch_stem_wgrad(int dtype, const StemParams &p, int gsrc, hipStream_t s)
{
    if (!p.img || !p.g || !p.dwpart || p.c_in < 1 || p.c_in > kStemPix || p.w > kStemMaxW ||
        p.ho != stem_out(p.h) || p.wo != stem_out(p.w) ||
        (gsrc == GB_BNGRAD && (!p.gx || !p.g_gamma || !p.g_mean || !p.g_rstd || !p.g_dgamma || !p.g_dbeta)) ||
        (gsrc != GB_BNGRAD && gsrc != GB_DENSE))
        return hipErrorInvalidValue;
    const int64_t m = (int64_t)p.n * p.ho * p.wo;
    const double e = dtype == DT_BF16 ? 2.0 : 4.0;
    const double nw = (double)kSK * kSK * p.c_in * kStemCout;
    const double gbytes = e * (double)m * kStemCout * (gsrc == GB_BNGRAD ? 2.0 : 1.0);
    TraceScope tr(KC_WGRAD, KID_STEM_WGRAD, s, e * (double)p.n * p.h * p.w * kStemPix + gbytes + 4.0 * nw,
                  2.0 * m * nw);
    if (dtype == DT_BF16) {
        const int64_t items = (int64_t)p.n * ((p.ho + kStemRows - 1) / kStemRows);
        const unsigned g = (unsigned)stem_groups(items);
        const size_t lds = stem_lds(p.wo, true);
        if (gsrc == GB_BNGRAD) hipLaunchKernelGGL(k_stem_wgrad<GB_BNGRAD>, dim3(g), dim3(kThreads), lds, s, p);
        else hipLaunchKernelGGL(k_stem_wgrad<GB_DENSE>, dim3(g), dim3(kThreads), lds, s, p);
    } else {
        const unsigned g = (unsigned)ceil_div((int64_t)nw, kThreads);
        if (gsrc == GB_BNGRAD) hipLaunchKernelGGL(k_stem_wgrad_f32<GB_BNGRAD>, dim3(g), dim3(kThreads), 0, s, p);
        else hipLaunchKernelGGL(k_stem_wgrad_f32<GB_DENSE>, dim3(g), dim3(kThreads), 0, s, p);
    }
    return hipGetLastError();
}

int64_t maxpool_fwd_rows(int dtype, int64_t m_out, int c) { return stats_row_blocks(m_out, c, dtype); }

hipError_t launch_maxpool_fwd(int dtype, const MaxPoolParams &p, bool bn, bool stats, hipStream_t s)
{
    if (!p.x || !p.y || (bn && (!p.gamma || !p.beta || !p.mean || !p.rstd)) || (stats && !p.part) ||
        p.ho != (p.h - 1) / 2 + 1 || p.wo != (p.w - 1) / 2 + 1)
        return hipErrorInvalidValue;
    const int64_t m_out = (int64_t)p.n * p.ho * p.wo;
    const int64_t R = maxpool_fwd_rows(dtype, m_out, p.c);
    const int64_t rpb = ceil_div(m_out, R);
    const int cb = (int)ceil_div(p.c, stats_ch_per_block(dtype));
    dim3 grid((unsigned)ceil_div(m_out, rpb), (unsigned)cb);
    const double e = dtype == DT_BF16 ? 2.0 : 4.0;
    TraceScope tr(KC_SWEEP, KID_MAXPOOL, s, e * p.c * ((double)p.n * p.h * p.w + (double)m_out), 0.0);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(kThreads), 0, s, p, rpb); };
    if (dtype == DT_BF16) {
        if (bn) { if (stats) go(k_maxpool_fwd<bf16_t, true, true>); else go(k_maxpool_fwd<bf16_t, true, false>); }
        else { if (stats) go(k_maxpool_fwd<bf16_t, false, true>); else go(k_maxpool_fwd<bf16_t, false, false>); }
    } else {
        if (bn) { if (stats) go(k_maxpool_fwd<float, true, true>); else go(k_maxpool_fwd<float, true, false>); }
        else { if (stats) go(k_maxpool_fwd<float, false, true>); else go(k_maxpool_fwd<float, false, false>); }
    }
    return hipGetLastError();
}

// Threads of a workgroup: its window columns' vectors, in whole waves.
static int mp_block(int wo, int cvec)
{
    const int t = (int)ceil_div((int64_t)wo * cvec, 64) * 64;
    return t < 64 ? 64 : t;
}

// Row pairs per chunk: the fewest of which all chunks fit the chip at once (a
// chunk reduces one window row more than it owns, so fewer and longer chunks
// do less, but a few chunks past the last free place cost a whole round: 40
// images of 112 x 112 took 86 us in 560 chunks for 512 places, 64 in 480; 60
// of 50 x 50, 46 us with 512 threads, 32 with 256 and twice the chunks).  Places:
// 1024 threads (128 registers each) and four workgroups' LDS per CU; counted
// for 8 channels a thread (float32 data takes two rounds).
static int maxpool_bwd_pairs(int n, int h, int w, int c)
{
    const int64_t hp = (h + 1) / 2;
    int per_cu = 1024 / mp_block((w - 1) / 2 + 1, c / 8);
    per_cu = per_cu < 1 ? 1 : (per_cu > 4 ? 4 : per_cu);
    const int64_t cpi = 256 * per_cu / n;                   // chunks per image
    return (int)(cpi < 1 ? hp : ceil_div(hp, cpi < hp ? cpi : hp));
}
// workgroups, one partial row each
int64_t maxpool_bwd_groups(int n, int h, int w, int c)
{
    const int64_t chunks = (int64_t)n * ceil_div((h + 1) / 2, maxpool_bwd_pairs(n, h, w, c));
    return chunks < kMaxPoolBwdGroups ? (chunks < 1 ? 1 : chunks) : kMaxPoolBwdGroups;
}

hipError_t launch_maxpool_bwd(int dtype, const MaxPoolParams &p, bool bn, hipStream_t s)
{
    const int vec = dtype == DT_BF16 ? 8 : 4, cvec = p.c / vec;
    if (!p.x || !p.g || !p.y || (bn && (!p.gamma || !p.beta || !p.mean || !p.rstd || !p.part)) ||
        p.c > kMaxPoolMaxC || p.wo > kMaxPoolMaxWo || cvec < 1 || (kThreads % cvec) ||
        p.ho != (p.h - 1) / 2 + 1 || p.wo != (p.w - 1) / 2 + 1)
        return hipErrorInvalidValue;
    const unsigned g = (unsigned)maxpool_bwd_groups(p.n, p.h, p.w, p.c);
    const double e = dtype == DT_BF16 ? 2.0 : 4.0, m = (double)p.n * p.h * p.w;
    TraceScope tr(KC_SWEEP, KID_MAXPOOL, s, e * p.c * ((bn ? 2.0 : 1.0) * m + (double)p.n * p.ho * p.wo), 0.0);
    const int pairs = maxpool_bwd_pairs(p.n, p.h, p.w, p.c), cpi = (int)ceil_div((p.h + 1) / 2, pairs);
    const int64_t chunks = (int64_t)p.n * cpi;
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(g), dim3((unsigned)mp_block(p.wo, cvec)), 0, s, p, pairs, cpi, chunks); };
    if (dtype == DT_BF16) {
        if (bn) go(k_maxpool_bwd<bf16_t, true>); else go(k_maxpool_bwd<bf16_t, false>);
    } else {
        if (bn) go(k_maxpool_bwd<float, true>); else go(k_maxpool_bwd<float, false>);
    }
    return hipGetLastError();
}

hipError_t launch_head_fwd(int dtype, const HeadParams &p, hipStream_t s)
{
    if (!p.x || !p.gamma || !p.beta || !p.mean || !p.rstd || !p.f || !p.wfc || !p.bfc || !p.labels || !p.logits ||
        !p.dlogits || !p.loss)
        return hipErrorInvalidValue;
    const int vec = dtype == DT_BF16 ? 8 : 4;
    const double e = dtype == DT_BF16 ? 2.0 : 4.0;
    TraceScope tr(KC_SMALL, KID_HEAD, s,
                  e * ((double)p.n * p.h * p.w * p.c + (double)p.c * p.classes) + 8.0 * p.n * p.classes,
                  2.0 * p.n * p.c * p.classes);
    const int nt = p.n * (p.c / vec);
    if (dtype == DT_BF16) hipLaunchKernelGGL(k_head_pool<bf16_t>, dim3((unsigned)ceil_div(nt, kThreads)), dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL(k_head_pool<float>, dim3((unsigned)ceil_div(nt, kThreads)), dim3(kThreads), 0, s, p);
    dim3 grid((unsigned)ceil_div(p.classes, kFcBN), (unsigned)ceil_div(p.n, 16));
    if (dtype == DT_BF16)
        hipLaunchKernelGGL(k_fc_gemm<bf16_t>, grid, dim3(kThreads), 0, s, p.n, p.classes, p.c, p.f, (int64_t)p.c,
                           (int64_t)1, (const bf16_t *)p.wfc, (int64_t)p.classes, (int64_t)1, p.bfc, p.logits);
    else
        hipLaunchKernelGGL(k_fc_gemm<float>, grid, dim3(kThreads), 0, s, p.n, p.classes, p.c, p.f, (int64_t)p.c,
                           (int64_t)1, (const float *)p.wfc, (int64_t)p.classes, (int64_t)1, p.bfc, p.logits);
    hipLaunchKernelGGL(k_softmax_ce, dim3((unsigned)p.n), dim3(kThreads), 0, s, p.n, p.classes, p.logits, p.labels,
                       p.dlogits, p.loss);
    hipLaunchKernelGGL(k_loss_mean, dim3(1), dim3(64), 0, s, p.n, p.loss);
    return hipGetLastError();
}

int64_t head_rows(int dtype, int64_t m, int c) { return stats_row_blocks(m, c, dtype); }

hipError_t launch_head_bwd_fc(int dtype, const HeadParams &p, hipStream_t s)
{
    if (!p.f || !p.wfc || !p.dlogits || !p.df || !p.dwfc || !p.dbfc) return hipErrorInvalidValue;
    TraceScope tr(KC_SMALL, KID_HEAD, s, 4.0 * ((double)p.n * p.classes + 2.0 * p.n * p.c + (double)p.c * p.classes),
                  4.0 * p.n * p.c * p.classes);
    // df = dlogits W^T: A = dlogits [n][K], B(k=j, col=c) = W[c][j]
    dim3 g1((unsigned)ceil_div(p.c, kFcBN), (unsigned)ceil_div(p.n, 16));
    if (dtype == DT_BF16)
        hipLaunchKernelGGL(k_fc_gemm<bf16_t>, g1, dim3(kThreads), 0, s, p.n, p.c, p.classes, p.dlogits,
                           (int64_t)p.classes, (int64_t)1, (const bf16_t *)p.wfc, (int64_t)1, (int64_t)p.classes,
                           (const float *)nullptr, p.df);
    else
        hipLaunchKernelGGL(k_fc_gemm<float>, g1, dim3(kThreads), 0, s, p.n, p.c, p.classes, p.dlogits,
                           (int64_t)p.classes, (int64_t)1, (const float *)p.wfc, (int64_t)1, (int64_t)p.classes,
                           (const float *)nullptr, p.df);
    // dW = f^T dlogits: A(i=c, k=n) = f[n][c], B(k=n, j) = dlogits[n][j]
    dim3 g2((unsigned)ceil_div(p.classes, kFcBN), (unsigned)ceil_div(p.c, 16));
    hipLaunchKernelGGL(k_fc_gemm<float>, g2, dim3(kThreads), 0, s, p.c, p.classes, p.n, p.f, (int64_t)1,
                       (int64_t)p.c, p.dlogits, (int64_t)p.classes, (int64_t)1, (const float *)nullptr, p.dwfc);
    hipLaunchKernelGGL(k_colsum, dim3((unsigned)ceil_div(p.classes, kThreads)), dim3(kThreads), 0, s, p.n, p.classes,
                       p.dlogits, p.dbfc);
    return hipGetLastError();
}

hipError_t launch_head_bn_bwd(int dtype, const HeadParams &p, int mode, hipStream_t s)
{
    if (!p.x || !p.gamma || !p.beta || !p.mean || !p.rstd || !p.df || (mode != HB_SUMS && !p.gx) ||
        (mode != HB_DX && !p.part) || (mode == HB_DX && (!p.dgamma || !p.dbeta)))
        return hipErrorInvalidValue;
    const int64_t m = (int64_t)p.n * p.h * p.w;
    const int64_t R = head_rows(dtype, m, p.c);
    const int64_t rpb = ceil_div(m, R);
    const int cb = (int)ceil_div(p.c, stats_ch_per_block(dtype));
    dim3 grid((unsigned)ceil_div(m, rpb), (unsigned)cb);
    const double e = dtype == DT_BF16 ? 2.0 : 4.0;
    TraceScope tr(KC_SMALL, KID_HEAD, s, e * (double)m * p.c * (mode == HB_SUMS ? 1.0 : 2.0) + 4.0 * p.n * p.c, 0.0);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(kThreads), 0, s, p, rpb); };
    if (dtype == DT_BF16) {
        if (mode == HB_SPLIT) go(k_head_bn_bwd<bf16_t, HB_SPLIT>);
        else if (mode == HB_SUMS) go(k_head_bn_bwd<bf16_t, HB_SUMS>);
        else go(k_head_bn_bwd<bf16_t, HB_DX>);
    } else {
        if (mode == HB_SPLIT) go(k_head_bn_bwd<float, HB_SPLIT>);
        else if (mode == HB_SUMS) go(k_head_bn_bwd<float, HB_SUMS>);
        else go(k_head_bn_bwd<float, HB_DX>);
    }
    return hipGetLastError();
}

}  // namespace bnr
