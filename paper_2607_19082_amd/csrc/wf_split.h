// Products of fp32 values on f16 MFMA (pairs of f16 values), and of bf16-pair
// activations on bf16 MFMA: the layers of the synthesis transform, and the
// plain product that hoists the hyperprior half of layer 1.
#pragma once

#include "wf_conv.h"
#include "wf_device.h"
#include "wf_pack.h"

namespace wf {

// ---- the synthesis transform's layers ----------------------------------------
//
// Bound by the matrix cores (1554 GFLOP at 4K).  fp32 MFMA peaks at 157
// TFLOP/s, f16 MFMA at sixteen times that, so the fp32 transform runs on f16
// pairs: x = x0 + x1 with x0 = f16(x), x1 = f16(x - x0) holds 22-23 of fp32's
// 24 bits, and three products x0 w0 + x0 w1 + x1 w0 accumulate in fp32.  The
// chain has one rounding per 32 values of k and product where the fp32 MFMA
// chain has eight, and the sum ends up closer to the 64-bit result than with
// fp32 operands (4K image: 2.3e-6 relative before).  f16's range is met by
// scaling with powers of two (exact): each weight column by its largest
// weight at plan time, the activations by the largest of the workgroup's own
// patch, found while it is staged (a later chunk with a larger value rescales
// the accumulators), both to [2^13, 2^14).  A scaled pair is exact to 2^-38 of
// the patch's largest value, so a workgroup goes to fp32 MFMA on the unscaled
// inputs (conv_tile_f32) when some pixel's own largest value is below 2^-15 of
// that (an outlier beside small values; inverse GDN: unless beta covers the
// difference), and when a value is infinite or NaN, which then propagates as
// in a product of fp32 values.
// The bf16 variant (bf16 weights, bf16-pair activations) has two products per
// operand pair and needs no scaling.
//
// A workgroup owns TW x TH output pixels of one parity class and 16 CT WC
// output channels.  Per chunk of 32 input channels it stages the pixels'
// patch (halo of one) once, split, in LDS ([half][k-group][pixel] of 16-byte
// operands: the 16 lanes of a k-group read 256 contiguous bytes), and every
// tap of the class then reads it shifted.  Weights come straight from L2 in
// operand order, one tap ahead of their use; a wave holds RT x CT tiles, so
// each weight operand feeds RT MFMA chains and each activation operand CT.
// Weights are the first MFMA operand: a lane then holds four consecutive
// channels of one pixel and stores 16 bytes.  4K (N = 192, M = 320): 20.36 ms
// with per-wave operand loads and fp32 MFMA, 4.95 ms now (the third layer
// with its inverse GDN 3.2 ms, 345 TFLOP/s of fp32 products, the matrix cores
// busy 57% at the 1.7 GHz that they then draw); bf16 at 120x68 latents
// (N = 128): 1.98 -> 0.44 ms.
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

struct SynthArgs {
    const float* in;
    float* out;
    const void* wp[4];        // packed panel per output class: [Cop/16][chunk][tap][NW][64] operands
    const int* ce;            // f16: [Cop] exponent each weight column was scaled by
    const float* bias;        // [Cop] bias (GDN: beta), zero-padded
    int B, Hi, Wi, Ci;        // input [B][Hi][Wi][Ci] (GDN: one row of all pixels)
    int Co, Cop, nch;         // output channels, padded; chunks of 32 input channels
    int Ho, Wo;               // output pixels
    int twl, ntx, nty;        // log2 of the tile's width; tiles along x, y
    int ncb, ncls;            // column blocks, classes
    int force_f32;            // a weight is not finite
    float covered;            // GDN: largest x^2 whose scaled error beta covers in every channel
    // inverse GDN in the epilogue of a transposed conv (k_synth with FUSE):
    const void* gwp;          // packed gamma^T [Cop/16][chunk][NW][64]
    const int* gce;           // f16: [Cop] scale exponents
    const float* beta;        // [Cop]
    int gforce;               // a gamma is not finite
};

// Workgroups of 128 pixels from which they are the faster ones (fp32, whole
// transform of a 16x16 latent, whose third layer has 128 of them: 119 us, with
// 64 x 64 tiles there 107; 50x75, second layer 469: 329 and 340).
constexpr int kSynthMinBlocks = 256;
constexpr int kSynthGroup = 32;   // tiles of a group (see k_synth)

struct SF16 {                 // fp32 transform on f16 pairs
    using V = h8;
    static constexpr int kNw = 2;
    static constexpr bool kScaled = true;
};
struct SBF16 {                // bf16 transform: bf16 weights, bf16-pair activations
    using V = b8;
    static constexpr int kNw = 1;
    static constexpr bool kScaled = false;
};

__device__ __forceinline__ f4 mfma_k32(h8 a, h8 b, f4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma_k32(b8 a, b8 b, f4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

// Largest |x| of a workgroup's threads as fp32 bits (an infinity or NaN then
// exceeds every finite value).  Holds a barrier.
__device__ __forceinline__ unsigned block_max_bits(unsigned m, unsigned* red) {
#pragma unroll
    for (int o = 32; o; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(max(max(red[0], red[1]), max(red[2], red[3])));
}
__device__ __forceinline__ unsigned abs_bits(float v) { return __builtin_bit_cast(unsigned, v) & 0x7fffffffu; }
constexpr unsigned kInfBits = 0x7f800000u;
constexpr int kSynthRange = 15;   // binary orders a pixel's largest value may lie below its patch's
// Exponent that scales a largest value with these bits to [2^13, 2^14).
__device__ __forceinline__ int scale_exp(unsigned bits) { return 127 + 13 - (int)(bits >> 23); }

// f16 pair of eight values scaled by 2^s.
__device__ __forceinline__ void split_f16(const float (&x)[8], int s, h8& hi, h8& lo) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float v = ldexpf(x[q], s);
        hi[q] = (_Float16)v;
        lo[q] = (_Float16)(v - (float)hi[q]);
    }
}

template <int MODE, int RT, int CT, int WC>
struct SynthShape {
    static constexpr int kWr = 4 / WC;                         // waves along the pixels
    static constexpr int kPx = 16 * RT * kWr;                  // pixels of a workgroup
    static constexpr int kCols = 16 * CT * WC;                 // output channels of a workgroup
    static constexpr int kHalo = MODE == XM_GDN || MODE == XM_GEMM ? 0 : 1;
    // patch pixels: 128 as 16 x 8 or 8 x 16 (180 with the halo), 64 as 16 x 4
    // or 8 x 8 (108), rounded up to 16: the k-groups' planes then start 256
    // bytes apart, and the lanes that one LDS cycle serves hit distinct banks
    static constexpr int kPatch = !kHalo ? kPx : (kPx == 128 ? 192 : 112);
    static constexpr int kItems = (kPatch * 4 + kThreads - 1) / kThreads;
};

// The tile in fp32 arithmetic, from the unscaled inputs and the weights put
// back together: the path of inputs that are not finite.
template <int MODE, int RT, int CT, class QY, class QX>
__device__ __forceinline__ void conv_tile_f32(const SynthArgs& a, const void* wp, int nk, int ntap, int nkx, int b, QY qy,
                                              QX qx, int ct0, f4 (&acc)[RT][CT]) {
    const int lane = threadIdx.x & 63, kq = lane >> 4;
    const h8* w = static_cast<const h8*>(wp) + lane;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = zero4();
    for (int k = 0; k < nk; ++k) {
        const int ch = k / ntap, t = k - ch * ntap, ty = t / nkx, tx = t - ty * nkx;
        const int dy = MODE == XM_DECONV ? 1 - ty : (MODE == XM_GDN || MODE == XM_GEMM ? 0 : ty - 1);
        const int dx = MODE == XM_DECONV ? 1 - tx : (MODE == XM_GDN || MODE == XM_GEMM ? 0 : tx - 1);
        const int c = ch * 32 + kq * 8;
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int n = (ct0 + j) * kTile + (lane & 15);
            const bool cv = (ct0 + j) * kTile < a.Cop;
            const h8* p = w + ((size_t)(cv ? ct0 + j : 0) * nk + k) * 2 * 64;
            const h8 w0 = p[0], w1 = p[64];
            const int e = cv ? -a.ce[n] : 0;
            float wf[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) wf[q] = ldexpf((float)w0[q] + (float)w1[q], e);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const int iy = qy(i) + dy, ix = qx(i) + dx;
                const bool ok = iy >= 0 && iy < a.Hi && ix >= 0 && ix < a.Wi && c < a.Ci;
                const size_t q0 = (((size_t)b * a.Hi + iy) * a.Wi + ix) * a.Ci + c;
                const f4 u = ld4<false>(a.in, q0, ok), v = ld4<false>(a.in, q0 + 4, ok);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    float x = q < 4 ? u[q & 3] : v[q & 3];
                    if (MODE == XM_GDN) x = x * x;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[q], x, acc[i][j], 0, 0, 0);
                }
            }
        }
    }
}

// Inverse GDN of a workgroup that holds all channels of its pixels, x in acc
// (lane: channels 4 (lane / 16) + q of each column tile, pixel lane % 16 of
// each row tile): z = gamma x^2 + beta with the squares exchanged through LDS
// as split operands, half of the row tiles at a time, then x sqrt(z) is
// stored.  One pass over memory instead of three (the separate kernel wrote,
// read and wrote the activations: third layer at 4K 2.45 + 1.31 ms, now 3.2).
template <class P, int RT, int CT, class Store>
__device__ __forceinline__ void gdn_epilogue(const SynthArgs& a, f4 (&acc)[RT][CT], int ct0, typename P::V* lds, unsigned* red,
                                             unsigned* pmax, Store store) {
    using V = typename P::V;
    constexpr int NW = P::kNw, HR = RT / 2, HP = HR * kTile;   // row tiles and pixels of a half
    const int lane = threadIdx.x & 63, kq = lane >> 4, nct = a.Cop / kTile, nch = (a.Co + 31) / 32;
    int s = 0;
    bool bad = false;
    if constexpr (P::kScaled) {
        unsigned pm[RT], m = 0;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            pm[i] = 0;
#pragma unroll
            for (int j = 0; j < CT; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) pm[i] = max(pm[i], abs_bits(acc[i][j][q] * acc[i][j][q]));
            m = max(m, pm[i]);
        }
        m = block_max_bits(m, red);                      // (its barrier: the last patch has been read)
        s = scale_exp(m);
        bad = a.gforce || m >= kInfBits;
        if (!bad && m > kSynthRange << 23 && m > __builtin_bit_cast(unsigned, a.covered)) {
            // each pixel's largest square over all waves' channels
            if (threadIdx.x < RT * kTile) pmax[threadIdx.x] = 0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < RT; ++i) atomicMax(&pmax[i * kTile + (lane & 15)], pm[i]);
            __syncthreads();
            int low = 0;
            if (threadIdx.x < RT * kTile) {
                const unsigned v = pmax[threadIdx.x];
                low = v != 0 && v < m - (kSynthRange << 23);
            }
            bad = __syncthreads_or(low);
        }
    } else {
        __syncthreads();
    }
    const V* w = static_cast<const V*>(a.gwp) + lane;
    size_t wo[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) wo[j] = (size_t)(ct0 + j < nct ? ct0 + j : 0) * nch * NW * 64;
    auto load_w = [&](int c, V (&wv)[CT][NW]) {
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int n = 0; n < NW; ++n) wv[j][n] = w[wo[j] + (size_t)(c * NW + n) * 64];
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        V wv[CT][NW];
        load_w(0, wv);
        // operands [hi, lo][chunk][k-group][pixel] (bad: the squares in fp32, channels 0-3 and 4-7 of a group)
#pragma unroll
        for (int i = 0; i < HR; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                const f4 x = acc[h * HR + i][j], x2 = x * x;
                const int n = (ct0 + j) * kTile + kq * 4;
                if (n >= nch * 32) continue;             // (wave-uniform: a column tile past the last chunk)
                const int at = (n >> 3) * HP + i * kTile + (lane & 15), lo = nch * 4 * HP;
                if (bad) {
                    *reinterpret_cast<f4*>(&lds[at + ((n & 4) ? lo : 0)]) = x2;
                } else {
                    typedef __attribute__((ext_vector_type(4))) unsigned short u4;
                    u4 hi, lw;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if constexpr (P::kScaled) {
                            const float v = ldexpf(x2[q], s);
                            const _Float16 t = (_Float16)v;
                            hi[q] = __builtin_bit_cast(unsigned short, t);
                            lw[q] = __builtin_bit_cast(unsigned short, (_Float16)(v - (float)t));
                        } else {
                            hi[q] = bf16_bits(x2[q]);
                            lw[q] = bf16_bits(x2[q] - bf16_value(hi[q]));
                        }
                    }
                    *reinterpret_cast<u4*>(reinterpret_cast<unsigned short*>(&lds[at]) + (n & 4)) = hi;
                    *reinterpret_cast<u4*>(reinterpret_cast<unsigned short*>(&lds[at + lo]) + (n & 4)) = lw;
                }
            }
        __syncthreads();
        f4 z[HR][CT];
#pragma unroll
        for (int i = 0; i < HR; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) z[i][j] = zero4();
        const int lo = nch * 4 * HP;
        if (P::kScaled && bad) {
            if constexpr (P::kScaled)
                for (int c = 0; c < nch; ++c)
#pragma unroll
                    for (int j = 0; j < CT; ++j) {
                        const V w0 = w[wo[j] + (size_t)(c * NW) * 64], w1 = w[wo[j] + (size_t)(c * NW + 1) * 64];
                        const int e = ct0 + j < nct ? -a.gce[(ct0 + j) * kTile + (lane & 15)] : 0;
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const float wf = ldexpf((float)w0[q] + (float)w1[q], e);
#pragma unroll
                            for (int i = 0; i < HR; ++i) {
                                const f4 x2 = *reinterpret_cast<const f4*>(&lds[(c * 4 + kq) * HP + i * kTile + (lane & 15) + (q < 4 ? 0 : lo)]);
                                z[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf, x2[q & 3], z[i][j], 0, 0, 0);
                            }
                        }
                    }
        } else {
            for (int c = 0; c < nch; ++c) {
                if (c) load_w(c, wv);
#pragma unroll
                for (int i = 0; i < HR; ++i) {
                    const int at = (c * 4 + kq) * HP + i * kTile + (lane & 15);
                    const V hi = lds[at], lw = lds[at + lo];
#pragma unroll
                    for (int j = 0; j < CT; ++j) z[i][j] = mfma_k32(wv[j][0], hi, z[i][j]);
                    if constexpr (NW == 2) {
#pragma unroll
                        for (int j = 0; j < CT; ++j) z[i][j] = mfma_k32(wv[j][1], hi, z[i][j]);
                    }
#pragma unroll
                    for (int j = 0; j < CT; ++j) z[i][j] = mfma_k32(wv[j][0], lw, z[i][j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int n = (ct0 + j) * kTile + kq * 4;
            if (ct0 + j >= nct) continue;
            const f4 beta = *reinterpret_cast<const f4*>(a.beta + n);
            int4 e{0, 0, 0, 0};
            if (P::kScaled && !bad) e = *reinterpret_cast<const int4*>(a.gce + n);
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const f4 x = acc[h * HR + i][j];
                f4 v = z[i][j];
                if constexpr (P::kScaled)
                    if (!bad) v = f4{ldexpf(v.x, -s - e.x), ldexpf(v.y, -s - e.y), ldexpf(v.z, -s - e.z), ldexpf(v.w, -s - e.w)};
                v = v + beta;
                store(h * HR + i, n, f4{x.x * sqrtf(v.x), x.y * sqrtf(v.y), x.z * sqrtf(v.z), x.w * sqrtf(v.w)});
            }
        }
        if (h == 0) __syncthreads();                     // the first half's operands have been read
    }
}

// Workgroup `bid` of a launch.
template <class P, int MODE, int RT, int CT, int WC, bool FUSE>
__device__ __forceinline__ void synth_tile(const SynthArgs& a, int bid) {
    using V = typename P::V;
    using S = SynthShape<MODE, RT, CT, WC>;
    constexpr int NW = P::kNw, NI = S::kItems, NP = S::kPatch, HALO = S::kHalo;
    static_assert(!FUSE || (MODE == XM_DECONV && WC == 4), "a wave needs all pixels of the workgroup");
    // the patch [hi, lo][k-group][pixel]; FUSE: also the squares of half of the pixels, all channels
    constexpr int kGdn = FUSE ? 2 * (S::kCols / 8) * (S::kPx / 2) : 0;
    __shared__ V patch[8 * NP > kGdn ? 8 * NP : kGdn];
    __shared__ unsigned red[4], pmax[FUSE && P::kScaled ? S::kPx : 1];

    // An XCD takes a run of neighbouring tiles, kSynthGroup of them at a time:
    // their patches then stay in its L2 for all classes and column blocks.
    // Within a group the class is the slowest index, the nine-tap class first:
    // workgroups go to an XCD's four shader engines in turn, so with the class
    // fastest one engine would get all of the nine-tap ones (measured: 2.90 ms
    // for the third layer of a 4K image), and the last workgroups of a launch
    // are then the short ones.
    const int ntiles = a.B * a.nty * a.ntx, per = (ntiles + kXcds - 1) / kXcds;
    int l = bid / kXcds;
    const int g0 = l / (kSynthGroup * a.ncls * a.ncb) * kSynthGroup, gn = min(kSynthGroup, per - g0);
    l -= g0 * a.ncls * a.ncb;
    const int cls = l / (gn * a.ncb), py = cls >> 1, px = cls & 1;
    l -= cls * gn * a.ncb;
    const int cb = l % a.ncb;
    int id = (bid % kXcds) * per + g0 + l / a.ncb;
    if (id >= ntiles) return;
    const int tx = id % a.ntx;
    id /= a.ntx;
    const int ty = id % a.nty, b = id / a.nty;
    const int TW = 1 << a.twl, TH = S::kPx >> a.twl, PW = TW + 2 * HALO, np = PW * (TH + 2 * HALO);
    const int y0 = ty * TH, x0 = tx * TW;

    const int nkx = MODE == XM_DECONV ? (px ? 2 : 3) : (HALO ? 3 : 1);
    const int nky = MODE == XM_DECONV ? (py ? 2 : 3) : (HALO ? 3 : 1);
    const int ntap = nkx * nky, nk = a.nch * ntap;

    const int wave = wave_id(), lane = threadIdx.x & 63, kq = lane >> 4;
    const int wr = wave / WC, wc = wave % WC;
    const int ct0 = (cb * WC + wc) * CT, nct = a.Cop / kTile;

    // patch items of this thread: pixel e / 4, channels 8 (e % 4) .. + 8
    int src[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int e = threadIdx.x + n * kThreads, p = e >> 2;
        const int ry = p / PW, iy = y0 - HALO + ry, ix = x0 - HALO + (p - ry * PW);
        const bool ok = p < np && iy >= 0 && iy < a.Hi && ix >= 0 && ix < a.Wi;
        src[n] = ok ? (int)((((size_t)b * a.Hi + iy) * a.Wi + ix) * a.Ci + (e & 3) * 8) : -1;
    }
    float st[NI][8];
    auto load_chunk = [&](int ch) {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const bool ok = src[n] >= 0 && ch * 32 + (threadIdx.x & 3) * 8 < a.Ci;
            const f4 u = ld4<false>(a.in, (size_t)(src[n] + ch * 32), ok), v = ld4<false>(a.in, (size_t)(src[n] + ch * 32 + 4), ok);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                st[n][q] = MODE == XM_GDN ? u[q] * u[q] : u[q];
                st[n][4 + q] = MODE == XM_GDN ? v[q] * v[q] : v[q];
            }
        }
    };

    // weights of k-step k: column tile ct at w + (ct nk + k) NW 64
    const V* w = static_cast<const V*>(a.wp[cls]) + lane;
    size_t wo[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) wo[j] = (size_t)(ct0 + j < nct ? ct0 + j : 0) * nk * NW * 64;
    auto load_w = [&](int k, V (&wv)[CT][NW]) {
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int n = 0; n < NW; ++n) wv[j][n] = w[wo[j] + (size_t)(k * NW + n) * 64];
    };

    // this lane's pixel of row tile i: patch index of its tap (0, 0), and the
    // step from one row tile to the next
    const int r0 = wr * RT * kTile + (lane & 15);
    const int at0 = kq * NP + (r0 >> a.twl) * PW + (r0 & (TW - 1));
    const int step = !HALO ? kTile : (kTile >> a.twl) * PW;

    f4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = zero4();

    int s = 1000;                                        // the activations' scale exponent (1000: none yet)
    unsigned big = 0, pm[NI];                            // largest |x| (bits) of the patch and of this thread's items
#pragma unroll
    for (int n = 0; n < NI; ++n) pm[n] = 0;
    bool bad = P::kScaled && a.force_f32;
    V wv[CT][NW], wn[CT][NW];
    load_chunk(0);
    load_w(0, wv);
    for (int ch = 0; ch < a.nch && !bad; ++ch) {
        if constexpr (P::kScaled) {
            unsigned m = 0;
#pragma unroll
            for (int n = 0; n < NI; ++n) {
#pragma unroll
                for (int q = 0; q < 8; ++q) pm[n] = max(pm[n], abs_bits(st[n][q]));
                m = max(m, pm[n]);
            }
            m = block_max_bits(m, red);                  // (its barrier: the chunk before has been read)
            big = m;
            if (m >= kInfBits) {
                bad = true;
                break;
            }
            const int need = scale_exp(m);
            if (need < s) {
                if (s < 1000)
#pragma unroll
                    for (int i = 0; i < RT; ++i)
#pragma unroll
                        for (int j = 0; j < CT; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q) acc[i][j][q] = ldexpf(acc[i][j][q], need - s);
                s = need;
            }
        } else {
            __syncthreads();
        }
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int e = threadIdx.x + n * kThreads;
            if (NP * 4 % kThreads == 0 || e < NP * 4) {
                V hi, lo;
                if constexpr (P::kScaled) {
                    split_f16(st[n], s, hi, lo);
                } else {
                    const b8x2 p = split8(f4{st[n][0], st[n][1], st[n][2], st[n][3]}, f4{st[n][4], st[n][5], st[n][6], st[n][7]});
                    hi = p.hi;
                    lo = p.lo;
                }
                patch[(e & 3) * NP + (e >> 2)] = hi;
                patch[(4 + (e & 3)) * NP + (e >> 2)] = lo;
            }
        }
        __syncthreads();
        int tap = 0;
        for (int t0 = 0; t0 < nky; ++t0)
            for (int t1 = 0; t1 < nkx; ++t1, ++tap) {
                const int k = ch * ntap + tap;
                // (pinned: the compiler would sink these loads to just before their use)
                load_w(min(k + 1, nk - 1), wn);
                if (tap == 0 && ch + 1 < a.nch) load_chunk(ch + 1);
                __builtin_amdgcn_sched_barrier(0);
                // patch row and column of this tap's pixel: dy + 1 and dx + 1
                const int oy = MODE == XM_DECONV ? 2 - t0 : t0, ox = MODE == XM_DECONV ? 2 - t1 : t1;
                const int at = at0 + (HALO ? oy * PW + ox : 0);
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    const V hi = patch[at + i * step], lo = patch[4 * NP + at + i * step];
#pragma unroll
                    for (int j = 0; j < CT; ++j) acc[i][j] = mfma_k32(wv[j][0], hi, acc[i][j]);
                    if constexpr (NW == 2) {
#pragma unroll
                        for (int j = 0; j < CT; ++j) acc[i][j] = mfma_k32(wv[j][1], hi, acc[i][j]);
                    }
#pragma unroll
                    for (int j = 0; j < CT; ++j) acc[i][j] = mfma_k32(wv[j][0], lo, acc[i][j]);
                }
#pragma unroll
                for (int j = 0; j < CT; ++j)
#pragma unroll
                    for (int n = 0; n < NW; ++n) wv[j][n] = wn[j][n];
            }
    }

    auto qy = [&](int i) { return y0 + ((r0 + i * kTile) >> a.twl); };   // row tile i's pixel of this lane
    auto qx = [&](int i) { return x0 + ((r0 + i * kTile) & (TW - 1)); };
    if constexpr (P::kScaled) {
        if (!bad && big > kSynthRange << 23 && (MODE != XM_GDN || big > __builtin_bit_cast(unsigned, a.covered))) {
            int low = 0;
#pragma unroll
            for (int n = 0; n < NI; ++n) {               // the four lanes of a pixel hold its k-groups
                unsigned m = max(pm[n], (unsigned)__shfl_xor((int)pm[n], 1));
                m = max(m, (unsigned)__shfl_xor((int)m, 2));
                low |= m != 0 && m < big - (kSynthRange << 23);
            }
            bad = __syncthreads_or(low);
        }
        if (bad) {
            // (uniform.  A chunk with a value that is not finite was left just
            // after block_max_bits' `red` was read; the epilogue writes it again)
            __syncthreads();
            s = 0;
            conv_tile_f32<MODE, RT, CT>(a, a.wp[cls], nk, ntap, nkx, b, qy, qx, ct0, acc);
        }
    }
    // a lane holds channels 4 (lane / 16) + q of each column tile, pixel lane % 16
    auto inside = [&](int i) { return qy(i) < a.Hi && qx(i) < a.Wi; };
    auto store = [&](int i, int n, f4 v) {
        const int oy = MODE == XM_DECONV ? 2 * qy(i) + py : qy(i), ox = MODE == XM_DECONV ? 2 * qx(i) + px : qx(i);
        if (inside(i)) *reinterpret_cast<f4*>(a.out + (((size_t)b * a.Ho + oy) * a.Wo + ox) * a.Co + n) = v;
    };
#pragma unroll
    for (int j = 0; j < CT; ++j) {
        const bool cv = ct0 + j < nct;                   // (wave-uniform)
        const int n = (cv ? ct0 + j : 0) * kTile + kq * 4;
        const f4 add = *reinterpret_cast<const f4*>(a.bias + n);
        if constexpr (P::kScaled) {
            const int4 ce = *reinterpret_cast<const int4*>(a.ce + n);
            const int4 e = bad ? int4{0, 0, 0, 0} : int4{-s - ce.x, -s - ce.y, -s - ce.z, -s - ce.w};
#pragma unroll
            for (int i = 0; i < RT; ++i)
                acc[i][j] = f4{ldexpf(acc[i][j].x, e.x), ldexpf(acc[i][j].y, e.y), ldexpf(acc[i][j].z, e.z), ldexpf(acc[i][j].w, e.w)};
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            acc[i][j] = acc[i][j] + add;
            // inverse GDN of the workgroup: zeros off the grid and past the last channel
            if (FUSE) acc[i][j] = cv && inside(i) ? acc[i][j] : zero4();
        }
    }
    if constexpr (FUSE) {
        gdn_epilogue<P, RT, CT>(a, acc, ct0, patch, red, pmax, store);
        return;
    }
#pragma unroll
    for (int j = 0; j < CT; ++j) {
        const int n = (ct0 + j) * kTile + kq * 4;
        if (ct0 + j >= nct) continue;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            f4 v = acc[i][j];
            if (MODE == XM_DECONV4) {                    // columns (class, channel)
                if (!inside(i)) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c4 = (n + q) / a.Co, c = n + q - c4 * a.Co;
                    if (c4 < 4)
                        a.out[(((size_t)b * a.Ho + 2 * qy(i) + (c4 >> 1)) * a.Wo + 2 * qx(i) + (c4 & 1)) * a.Co + c] = v[q];
                }
            } else {
                if (MODE == XM_GDN && inside(i)) {
                    const f4 x = *reinterpret_cast<const f4*>(a.in + (size_t)qx(i) * a.Co + n);
                    v = f4{x.x * sqrtf(v.x), x.y * sqrtf(v.y), x.z * sqrtf(v.z), x.w * sqrtf(v.w)};
                }
                store(i, n, v);
            }
        }
    }
}

// Pack a panel for synth_tile: wt(c, t, nkx, ci, n) is the weight of class c's
// tap t (nkx taps a row; ntap(c, nkx) of them) from input channel ci to column
// n < ncol, in (chunk of 32 channels, tap, channel) order.  f16: as pairs, the
// column scaled to [2^13, 2^14) (exponents in ce, of Cop entries); returns
// whether a weight is not finite.
template <class T, class F>
inline bool pack_split(bool bf, int nclass, int Ci, int ncol, int Cop, T ntap, F wt, std::vector<int>& ce,
                       std::vector<uint16_t> (&out)[4]) {
    const int nch = (Ci + 31) / 32, nw = bf ? 1 : 2;
    bool odd = false;
    ce.assign(Cop, 0);
    if (!bf)
        for (int n = 0; n < ncol; ++n) {
            float big = 0.0f;
            for (int c = 0; c < nclass; ++c) {
                int nkx;
                const int nt = ntap(c, nkx);
                for (int t = 0; t < nt; ++t)
                    for (int ci = 0; ci < Ci; ++ci) {
                        const float v = std::fabs(wt(c, t, nkx, ci, n));
                        if (!std::isfinite(v)) odd = true;
                        else if (v > big) big = v;
                    }
            }
            if (big > 0.0f) ce[n] = 13 - std::ilogb(big);
        }
    for (int c = 0; c < nclass; ++c) {
        int nkx;
        const int nt = ntap(c, nkx), nk = nch * nt;
        std::vector<uint16_t>& v = out[c];
        v.assign((size_t)Cop / kTile * nk * nw * 64 * 8, 0);
        for (int n = 0; n < ncol; ++n)
            for (int k = 0; k < nk; ++k)
                for (int q = 0; q < 32; ++q) {
                    const int ci = k / nt * 32 + q;
                    if (ci >= Ci) continue;
                    const float f = wt(c, k % nt, nkx, ci, n);
                    const size_t at = (((size_t)(n / kTile) * nk + k) * nw * 64 + (q / 8) * 16 + n % kTile) * 8 + q % 8;
                    if (bf) {
                        v[at] = bf16_round(f);
                    } else {
                        const float g = std::ldexp(f, ce[n]);
                        const uint16_t h = f16_round(g);
                        v[at] = h;
                        v[at + 64 * 8] = std::isfinite(g) ? f16_round(g - f16_value_of(h)) : 0;
                    }
                }
    }
    return odd;
}

}  // namespace wf
