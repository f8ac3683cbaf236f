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

template <int GS, int MAXW>
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
    // they are written to LDS).  MAXW: the widest image the slots are for (images
    // of up to 64 in slots for 256 took up to 5% more than the sequence).
    constexpr int NI = (kSIR * (MAXW + 6) + kThreads - 1) / kThreads, NG = (kStemRows * (MAXW / 2) + 31) / 32;
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
// A workgroup takes chunks of consecutive row pairs of one image; thread
// (ow, v) owns four channels v of window column ow and of the input columns
// 2 ow, 2 ow + 1.  Per window row it reads two input rows (the third is
// carried: every input row is reduced over its three columns once, "first
// maximum" kept as value and column), so the first-maximum tap of every window,
// the gradients routed to a pixel and the pixel's BN input all come from
// registers, except what the right-hand neighbour's windows hold, which goes
// through LDS (three row buffers, one barrier per row).  Window row oh finishes
// input row 2 oh - 1 (which it shares with window row oh - 1) and input row
// 2 oh (its own).  The sums add the two pixels of an input row first and the
// workgroup's columns in float64.
// A value wins over an earlier one only if it is greater (NaN never wins).
// What bounds it: instruction issue and the load round trip of each row; rows
// are addressed by a scalar base and a 32-bit offset a column.  128 images of
// 112 x 112 x 64 in bf16: 249 us with the windows of every row pair scanned
// twice from global memory, 137 us this way (HBM floor 83); 5 of 17 x 17: 11.9
// and 10.1.  Eight bf16 channels a thread spilled registers (215 us; 13.1);
// without spilling they are no faster on large inputs and slower on small ones,
// which are one chain of steps (16 of 65 x 65: 27.8 us against 18.9).
constexpr int kMpVec = 4;                            // channels of a thread
constexpr int kMpThreads = kMaxPoolMaxWo * kMaxPoolMaxC / kMpVec;
// the channels of one 32-bit word
template <typename T> struct MpWord;
template <> struct MpWord<float> {
    static constexpr int N = 1;
    __device__ static __forceinline__ void unpack(uint32_t w, float *f) { f[0] = __uint_as_float(w); }
    __device__ static __forceinline__ uint32_t pack(const float *f) { return __float_as_uint(f[0]); }
};
template <> struct MpWord<bf16_t> {
    static constexpr int N = 2;
    __device__ static __forceinline__ void unpack(uint32_t w, float *f) {
        f[0] = __uint_as_float(w << 16);
        f[1] = __uint_as_float(w & 0xffff0000u);
    }
    __device__ static __forceinline__ uint32_t pack(const float *f) { return pack2bf(f[0], f[1]); }
};
// a thread's vector of NW words
template <int NW> struct alignas(4 * NW) MpVec {
    uint32_t u[NW];
    __device__ static __forceinline__ MpVec load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
        if constexpr (NW == 4) return __builtin_bit_cast(MpVec, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
        else return __builtin_bit_cast(MpVec, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t off) const {
        if constexpr (NW == 4) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, *this), r, off, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, *this), r, off, 0, 0);
    }
};
// LDS of a workgroup of nthr threads: three row buffers of the windows'
// gradients and codes (a byte a channel) with 16 guard vectors past the last
// column, then, in the same place, two arrays of partial sums
template <typename T> constexpr size_t mp_lds(int nthr)
{
    const size_t rows = (size_t)3 * (nthr + 16) * kMpVec * (sizeof(T) + 1), red = (size_t)2 * nthr * kMpVec * sizeof(float);
    return rows > red ? rows : red;
}
// waves per SIMD that the registers are held to
template <typename T> constexpr int mp_waves() { return sizeof(T) == 2 ? 5 : 4; }
// WIDE: an image row of x or g spans 2^31 bytes or more (64-bit offsets)
template <typename T, bool BN, bool WIDE>
__global__ __launch_bounds__(kMpThreads, mp_waves<T>()) void k_maxpool_bwd(MaxPoolParams p, int pairs_per_chunk,
                                                               unsigned chunks_per_image, unsigned chunks)
{
    using WD = MpWord<T>;
    constexpr int VEC = kMpVec, NW = VEC / WD::N;                  // words of a vector
    using V = MpVec<NW>;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) float par[4][kMaxPoolMaxC];           // sign(gamma), c0, c1, mean
    const int LD = blockDim.x + 16;
    V *g_s = reinterpret_cast<V *>(smem);                          // [3][LD]
    uint32_t *c_s = reinterpret_cast<uint32_t *>(smem + 3 * LD * sizeof(V));      // [3][LD]
    float *red = reinterpret_cast<float *>(smem);                  // [2][threads][VEC]
    const int C = p.c, h = p.h, w = p.w, ho = p.ho, wo = p.wo, cvec = C / VEC;
    const int tid = threadIdx.x, v = tid % cvec, ow = tid / cvec;
    const bool act = ow < wo;
    const T *x = reinterpret_cast<const T *>(p.x);
    const T *gy = reinterpret_cast<const T *>(p.g);
    T *dy = reinterpret_cast<T *>(p.y);
    const bool in_l = ow > 0, in_r = 2 * ow + 1 < w;
    const int cm = act ? 2 * ow : 0, cl = act && in_l ? cm - 1 : 0, cr = act ? (in_r ? cm + 1 : w - 1) : 0;
    const int gcol = act ? ow : 0, hp = (h + 1) / 2;

    // one window row: input rows 2 oh, 2 oh + 1 (columns 2 ow - 1 .. 2 ow + 1)
    // and the window's gradient
    struct Row { V a[3], b[3], g; };
    using Off = std::conditional_t<WIDE, uint64_t, uint32_t>;      // byte offset in an image row
    constexpr Off es = sizeof(T);
    const Off x_ld = (Off)p.x_ldc * es, g_ld = (Off)p.g_ldc * es, vo = (Off)(v * VEC) * es;
    const Off ol = (Off)cl * x_ld + vo, om = (Off)cm * x_ld + vo, orr = (Off)cr * x_ld + vo, og = (Off)gcol * g_ld + vo;
    const uint32_t od = (uint32_t)((cm * C + v * VEC) * sizeof(T)), drow = (uint32_t)(w * C * sizeof(T));
    auto ld = [&](const T *row, Off span, Off o) __attribute__((always_inline)) -> V {
        if constexpr (WIDE) return *reinterpret_cast<const V *>(reinterpret_cast<const char *>(row) + o);
        else return V::load(buf_view(row, span), o);
    };
    const Off xspan = (Off)(w - 1) * x_ld + (Off)C * es, gspan = (Off)(wo - 1) * g_ld + (Off)C * es;
    // of the chunk at hand: row pairs [j0, j1) of an image
    const T *xn, *gn;
    T *dn;
    int j0, j1;
    V top[3];                                    // the input row above it
    Row cur;
    auto xrow = [&](int row) __attribute__((always_inline)) {
        return xn + (int64_t)(row < 0 ? 0 : (row < h ? row : h - 1)) * w * p.x_ldc;
    };
    auto load_row = [&](int oh) __attribute__((always_inline)) {
        const T *ra = xrow(2 * oh), *rb = xrow(2 * oh + 1);
        cur.a[0] = ld(ra, xspan, ol); cur.a[1] = ld(ra, xspan, om); cur.a[2] = ld(ra, xspan, orr);
        cur.b[0] = ld(rb, xspan, ol); cur.b[1] = ld(rb, xspan, om); cur.b[2] = ld(rb, xspan, orr);
        cur.g = ld(gn + (int64_t)(oh < ho ? oh : ho - 1) * wo * p.g_ldc, gspan, og);
    };
    // (the image index is uniform: kept in a scalar, so are the row addresses)
    auto begin = [&](unsigned ck) __attribute__((always_inline)) {
        const int n = __builtin_amdgcn_readfirstlane((int)(ck / chunks_per_image));
        j0 = (int)(ck - (unsigned)n * chunks_per_image) * pairs_per_chunk;
        j1 = min(hp, j0 + pairs_per_chunk);
        xn = x + (int64_t)n * h * w * p.x_ldc;
        gn = gy + (int64_t)n * ho * wo * p.g_ldc;
        dn = dy + (int64_t)n * h * w * C;
        const T *ra = xrow(2 * j0 - 1);
        top[0] = ld(ra, xspan, ol); top[1] = ld(ra, xspan, om); top[2] = ld(ra, xspan, orr);
        load_row(j0);
    };

    // BN parameters, by way of LDS
    float pg = 1.f, pb = 0.f, pm = 0.f, pr = 1.f;
    if (BN && tid < C) { pg = p.gamma[tid]; pb = p.beta[tid]; pm = p.mean[tid]; pr = p.rstd[tid]; }
    float s1[VEC], s2[VEC], kc[VEC];
    #pragma unroll
    for (int e = 0; e < VEC; e++) { s1[e] = s2[e] = 0.f; kc[e] = BN ? bn_centre<T>(p.ctr, v * VEC + e) : 0.f; }
    const float *sgn = par[0] + v * VEC, *pc0 = par[1] + v * VEC, *pc1 = par[2] + v * VEC, *pmu = par[3] + v * VEC;

    // (a tap outside the image: sign(gamma) x - inf, which never wins)
    const float off_l = in_l ? 0.f : -INFINITY, off_r = in_r ? 0.f : -INFINITY;
    // first maximum of one channel's three columns of an input row
    auto max3 = [&](float sg, float l, float m, float r, bool in, float &best) __attribute__((always_inline)) -> uint32_t {
        const float omid = in ? 0.f : -INFINITY;
        const float kl = __builtin_fmaf(sg, l, in ? off_l : -INFINITY), km = __builtin_fmaf(sg, m, omid);
        const float kr = __builtin_fmaf(sg, r, in ? off_r : -INFINITY);
        float b = __builtin_fmaxf(kl, -INFINITY);                  // (NaN never wins)
        uint32_t c = km > b ? 1u : 0u;
        b = __builtin_fmaxf(b, km);
        c = kr > b ? 2u : c;
        best = __builtin_fmaxf(b, kr);
        return c;
    };

    for (unsigned ck = blockIdx.x; ck < chunks; ck += gridDim.x) {
        begin(ck);
        if (ck == blockIdx.x) {                      // (with the first chunk's loads in flight)
            if (tid < C) {
                float c0 = 1.f, c1 = 0.f;
                if (BN) bn_coef(pg, pb, pm, pr, c0, c1);
                par[0][tid] = pg > 0.f ? 1.f : (pg < 0.f ? -1.f : 0.f);
                par[1][tid] = c0;
                par[2][tid] = c1;
                par[3][tid] = pm;
            }
            // no window past the last column, ever: code 15 matches no tap
            if (tid < 3 * 16) {
                const int i = tid / 16 * LD + wo * cvec + tid % 16;
                c_s[i] = 0x0f0f0f0fu;
                g_s[i] = V{};
            }
        }
        __syncthreads();                             // (also: the row buffers' readers of the chunk before are done)
        // first maxima of the row above: value and column (four bits a channel)
        float hb[VEC];
        uint32_t hc = 0u;
        #pragma unroll
        for (int i = 0; i < NW; i++) {
            float fl[WD::N], fm[WD::N], fr[WD::N];
            WD::unpack(top[0].u[i], fl); WD::unpack(top[1].u[i], fm); WD::unpack(top[2].u[i], fr);
            #pragma unroll
            for (int t = 0; t < WD::N; t++) {
                const int e = i * WD::N + t;
                hc |= max3(BN ? sgn[e] : 1.f, fl[t], fm[t], fr[t], j0 > 0, hb[e]) << (4 * e);
            }
        }
        uint32_t cp = 0x0f0f0f0fu;                      // codes of the window row before
        V pb1 = V{}, pb2 = V{}, pgv = V{};      // its second input row's pixels, its gradient
        // finishes one input row's pixels, columns 2 ow and 2 ow + 1 (inputs x0,
        // x1): dz(i, t, e, z0, z1) gives channel e's gradients (word i, its channel t)
        auto finish_row = [&](int row, const V &x0, const V &x1, auto &&dz) __attribute__((always_inline)) {
            V o0, o1;
            #pragma unroll
            for (int i = 0; i < NW; i++) {
                float z0[WD::N], z1[WD::N];
                #pragma unroll
                for (int t = 0; t < WD::N; t++) dz(i, t, i * WD::N + t, z0[t], z1[t]);
                if (BN) {
                    float f0[WD::N], f1[WD::N];
                    WD::unpack(x0.u[i], f0);
                    WD::unpack(x1.u[i], f1);
                    #pragma unroll
                    for (int t = 0; t < WD::N; t++) {
                        const int e = i * WD::N + t;
                        f0[t] -= kc[e];
                        f1[t] -= kc[e];
                        z0[t] = bn_lin(f0[t], pc0[e], pc1[e]) > 0.f ? z0[t] : 0.f;
                        z1[t] = in_r && bn_lin(f1[t], pc0[e], pc1[e]) > 0.f ? z1[t] : 0.f;
                    }
                    o0.u[i] = WD::pack(z0);
                    o1.u[i] = WD::pack(z1);
                    WD::unpack(o0.u[i], z0);
                    WD::unpack(o1.u[i], z1);
                    #pragma unroll
                    for (int t = 0; t < WD::N; t++) {
                        const int e = i * WD::N + t;
                        const float m1 = in_r ? f1[t] - pmu[e] : 0.f;
                        s1[e] += z0[t] + z1[t];
                        s2[e] += __builtin_fmaf(z0[t], f0[t] - pmu[e], z1[t] * m1);
                    }
                } else {
                    o0.u[i] = WD::pack(z0);
                    o1.u[i] = WD::pack(z1);
                }
            }
            const __amdgpu_buffer_rsrc_t dst = buf_view(dn + (int64_t)row * w * C, drow);
            o0.store(dst, od);
            o1.store(dst, in_r ? od + (uint32_t)(C * sizeof(T)) : kBufOff);
        };

        auto step = [&](int oh) __attribute__((always_inline)) {
            // ---- window row oh: input rows 2 oh - 1 (carried), 2 oh, 2 oh + 1 ----
            const bool wrow = oh < ho;
            uint32_t code = 0u, nhc = 0u;
            #pragma unroll
            for (int i = 0; i < NW; i++) {
                float al[WD::N], am[WD::N], ar[WD::N], bl[WD::N], bm[WD::N], br[WD::N];
                WD::unpack(cur.a[0].u[i], al); WD::unpack(cur.a[1].u[i], am); WD::unpack(cur.a[2].u[i], ar);
                WD::unpack(cur.b[0].u[i], bl); WD::unpack(cur.b[1].u[i], bm); WD::unpack(cur.b[2].u[i], br);
                #pragma unroll
                for (int t = 0; t < WD::N; t++) {
                    const int e = i * WD::N + t;
                    const float sg = BN ? sgn[e] : 1.f;
                    float ba, bb;
                    const uint32_t ca = max3(sg, al[t], am[t], ar[t], true, ba);
                    const uint32_t cb = max3(sg, bl[t], bm[t], br[t], 2 * oh + 1 < h, bb);
                    // (a row without a value above -inf holds column 0: tap 0, as a scan that nothing wins)
                    uint32_t tap = (hc >> (4 * e)) & 3u;
                    tap = ba > hb[e] ? 3u + ca : tap;
                    tap = bb > __builtin_fmaxf(hb[e], ba) ? 6u + cb : tap;
                    code |= tap << (8 * e);
                    nhc |= cb << (4 * e);
                    hb[e] = bb;
                }
            }
            hc = nhc;
            code = wrow && act ? code : 0x0f0f0f0fu;
            V *gw_s = g_s + oh % 3 * LD + tid, *gp_s = g_s + (oh + 2) % 3 * LD + tid;
            uint32_t *cw_s = c_s + oh % 3 * LD + tid, *cp_s = c_s + (oh + 2) % 3 * LD + tid;
            if (act) {
                *gw_s = cur.g;
                *cw_s = code;
            }
            __syncthreads();
            if (act) {
                const V gwr = gw_s[cvec];
                const uint32_t cwr = cw_s[cvec];
                // (an unmatched window adds zero; sums start from +0)
                auto tap_of = [](uint32_t word, int e) __attribute__((always_inline)) { return (word >> (8 * e)) & 15u; };
                const bool odd = oh > j0 && 2 * oh - 1 < h, even = oh < j1;
                if (odd) {                              // windows (oh - 1, ow), (oh - 1, ow + 1), (oh, ow), (oh, ow + 1)
                    const V gpr = gp_s[cvec];
                    const uint32_t cpr = cp_s[cvec];
                    finish_row(2 * oh - 1, pb1, pb2,
                               [&](int i, int t, int e, float &z0, float &z1) __attribute__((always_inline)) {
                        float a00[WD::N], a01[WD::N], a10[WD::N], a11[WD::N];
                        WD::unpack(pgv.u[i], a00); WD::unpack(gpr.u[i], a01);
                        WD::unpack(cur.g.u[i], a10); WD::unpack(gwr.u[i], a11);
                        const uint32_t c00 = tap_of(cp, e), c01 = tap_of(cpr, e);
                        const uint32_t c10 = tap_of(code, e), c11 = tap_of(cwr, e);
                        z0 = (c00 == 7u ? a00[t] : 0.f) + (c10 == 1u ? a10[t] : 0.f);
                        z1 = (c00 == 8u ? a00[t] : 0.f) + (c01 == 6u ? a01[t] : 0.f);
                        z1 += c10 == 2u ? a10[t] : 0.f;
                        z1 += c11 == 0u ? a11[t] : 0.f;
                    });
                }
                if (even) {
                    finish_row(2 * oh, cur.a[1], cur.a[2],
                               [&](int i, int t, int e, float &z0, float &z1) __attribute__((always_inline)) {
                        float a00[WD::N], a01[WD::N];
                        WD::unpack(cur.g.u[i], a00); WD::unpack(gwr.u[i], a01);
                        const uint32_t c00 = tap_of(code, e), c01 = tap_of(cwr, e);
                        z0 = (c00 == 4u ? a00[t] : 0.f) + 0.f;              // (0 + -0 = 0, as a sum from zero)
                        z1 = (c00 == 5u ? a00[t] : 0.f) + (c01 == 3u ? a01[t] : 0.f);
                    });
                }
            }
            pb1 = cur.b[1]; pb2 = cur.b[2]; pgv = cur.g;
            if (oh < j1) load_row(oh + 1);
            cp = code;
        };
        for (int oh = j0; oh <= j1; oh++) step(oh);
    }
    __syncthreads();
    if (BN) {
        // threads tid = v + cvec ow hold channel vector v
        #pragma unroll
        for (int e = 0; e < VEC; e++) {
            const float rs = p.rstd[v * VEC + e];
            red[tid * VEC + e] = act ? s1[e] : 0.f;
            red[(blockDim.x + tid) * VEC + e] = act ? s2[e] * rs : 0.f;
        }
        __syncthreads();
        for (int k = tid; k < 2 * C; k += blockDim.x) {           // column k % C of sum k / C
            const int c = k < C ? k : k - C, n_ = wo * cvec;
            const float *col = red + ((k < C ? 0 : blockDim.x) + c / VEC) * VEC + c % VEC;
            double a[4] = {0.0, 0.0, 0.0, 0.0};                  // (four reads in flight)
            int u = 0;
            for (; u + 3 * cvec < n_; u += 4 * cvec)
                #pragma unroll
                for (int q = 0; q < 4; q++) a[q] += col[(u + q * cvec) * VEC];
            for (; u < n_; u += cvec) a[0] += col[u * VEC];
            p.part[(int64_t)blockIdx.x * 2 * C + k] = (float)((a[0] + a[1]) + (a[2] + a[3]));
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
        auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(g), dim3(kThreads), lds, s, p); };
        if (gsrc == GB_BNGRAD) { if (p.w <= 64) go(k_stem_wgrad<GB_BNGRAD, 64>); else go(k_stem_wgrad<GB_BNGRAD, kStemMaxW>); }
        else { if (p.w <= 64) go(k_stem_wgrad<GB_DENSE, 64>); else go(k_stem_wgrad<GB_DENSE, kStemMaxW>); }
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

// Threads of a workgroup: its window columns' vectors, in whole waves (at most
// 1024: wider images are refused before the launch).
static int mp_block(int wo, int cvec)
{
    const int64_t t = ceil_div((int64_t)wo * cvec, 64) * 64;
    return t < 64 ? 64 : (t > 1024 ? 1024 : (int)t);
}

// Chunks of the pooling backward.  A chunk of P row pairs costs P + 1 window
// rows and about one more to start, and the places on the chip are filled in
// whole rounds, so P is the best of four round counts by rounds x (P + 2).  Taken
// as whole images wherever there are more images than places, with a nearly
// empty last round, 520 images of 112 x 112 took 1099 us against 684 and 1103 of
// 16 x 16 (16 channels) 84 against 31.  Places: what the waves a SIMD holds and
// the LDS leave room for.
struct MpPlan { int nthr, pairs, cpi; int64_t chunks, groups; };
static MpPlan mp_plan(int dtype, int n, int h, int w, int c)
{
    const int hp = (h + 1) / 2;
    MpPlan best{};
    best.nthr = mp_block((w - 1) / 2 + 1, c / kMpVec);
    const size_t lds = (dtype == DT_BF16 ? mp_lds<bf16_t>(best.nthr) : mp_lds<float>(best.nthr)) +
                       4 * kMaxPoolMaxC * sizeof(float);
    const int64_t by_lds = 160 * 1024 / (int64_t)lds, by_regs = 256 * (dtype == DT_BF16 ? mp_waves<bf16_t>() : mp_waves<float>()) / best.nthr;
    int64_t places = device_cus() * (by_lds < by_regs ? by_lds : by_regs), cost = 0;
    if (places > kMaxPoolBwdGroups) places = kMaxPoolBwdGroups;
    for (int r = 1; r <= 4; r++) {
        const int64_t want = r * places / n, cut = want < 1 ? 1 : (want > hp ? hp : want);
        const int64_t pairs = ceil_div(hp, cut), cpi = ceil_div(hp, pairs), chunks = n * cpi;
        const int64_t t = ceil_div(chunks, places) * (pairs + 2);
        if (r == 1 || t < cost) {
            cost = t;
            best.pairs = (int)pairs; best.cpi = (int)cpi; best.chunks = chunks;
        }
    }
    best.groups = best.chunks < places ? best.chunks : places;
    return best;
}
// workgroups, one partial row each
int64_t maxpool_bwd_groups(int dtype, int n, int h, int w, int c)
{
    const int64_t g = mp_plan(dtype, n, h, w, c).groups;
    return g < 1 ? 1 : g;
}

hipError_t launch_maxpool_bwd(int dtype, const MaxPoolParams &p, bool bn, hipStream_t s)
{
    const int vec = dtype == DT_BF16 ? 8 : 4, cvec = p.c / vec;
    if (!p.x || !p.g || !p.y || (bn && (!p.gamma || !p.beta || !p.mean || !p.rstd || !p.part)) ||
        p.c > kMaxPoolMaxC || p.wo > kMaxPoolMaxWo || cvec < 1 || (kThreads % cvec) ||
        p.ho != (p.h - 1) / 2 + 1 || p.wo != (p.w - 1) / 2 + 1)
        return hipErrorInvalidValue;
    const double e = dtype == DT_BF16 ? 2.0 : 4.0, m = (double)p.n * p.h * p.w;
    TraceScope tr(KC_SWEEP, KID_MAXPOOL, s, e * p.c * ((bn ? 2.0 : 1.0) * m + (double)p.n * p.ho * p.wo), 0.0);
    const MpPlan pl = mp_plan(dtype, p.n, p.h, p.w, p.c);
    const int64_t lim = (int64_t)1 << 31, es = dtype == DT_BF16 ? 2 : 4;
    const bool wide = ((p.w - 1) * p.x_ldc + p.c) * es >= lim || ((p.wo - 1) * p.g_ldc + p.c) * es >= lim;
    if (pl.chunks >= lim) return hipErrorInvalidValue;           // (n < 2^31 and n h w <= 2^31: never)
    auto go = [&](auto kern, size_t lds) {
        hipLaunchKernelGGL(kern, dim3((unsigned)pl.groups), dim3((unsigned)pl.nthr), lds, s, p, pl.pairs, (unsigned)pl.cpi,
                           (unsigned)pl.chunks);
    };
    auto go_t = [&](auto t) {
        using T = decltype(t);
        const size_t lds = mp_lds<T>(pl.nthr);
        if (wide) { if (bn) go(k_maxpool_bwd<T, true, true>, lds); else go(k_maxpool_bwd<T, false, true>, lds); }
        else { if (bn) go(k_maxpool_bwd<T, true, false>, lds); else go(k_maxpool_bwd<T, false, false>, lds); }
    };
    if (dtype == DT_BF16) go_t(bf16_t()); else go_t(float());
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
