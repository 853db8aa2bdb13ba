// The layers of the synthesis transform: products of fp32 values on bf16 MFMA
// (each value the sum of three bf16 values), and of bf16-pair activations with
// bf16 weights.
#pragma once

#include "wf_conv.h"
#include "wf_device.h"
#include "wf_pack.h"

namespace wf {

// Bound by the matrix cores (1554 GFLOP at 4K).  fp32 MFMA peaks at 157
// TFLOP/s, bf16 MFMA at sixteen times that.  An fp32 value is the exact sum of
// three bf16 values of the same exponent range, x = x0 + x1 + x2 with the
// 24 bits of its significand eight to a part, so no value is scaled and none
// loses bits beside a larger one.  Six products, x0 w0, x0 w1, x1 w0, x0 w2,
// x1 w1 and x2 w0, accumulate in fp32; the three left out are about 2^-22 of
// |x w| together at most, whatever the values (but for parts below fp32's
// normal range, in products under 2^-102), and the chain has one rounding per
// 32 values of k where the fp32 MFMA chain has eight: the sum ends up closer to
// the 64-bit result (4K image: 2.3e-6 relative with fp32 MFMA, 5e-7 so; 2.0e-6
// with the six products added to the running sum one by one, 6% faster).
// (Pairs of f16 values need three products only, 4.5 ms at 4K, but hold 22 bits
// and 2^-38 of the largest value beside them: with channels or weights 1e8
// apart the result was off by more than 1e-4.)
// An infinity or NaN, or a partial sum that overflows, leaves a result that is
// not finite; a wave that sees one computes its tile again on fp32 MFMA, from
// the inputs and the weights put back together (conv_tile_f32), so such values
// propagate as in a product of fp32 values.
// The bf16 variant (bf16 weights, bf16-pair activations) has two products per
// operand pair.
//
// A workgroup owns TW x TH output pixels of one parity class and 16 CT WC
// output channels.  Per chunk of 32 input channels it stages the pixels'
// patch (halo of one) once, split, in LDS ([part][k-group][pixel] of 16-byte
// operands: the 16 lanes of a k-group read 256 contiguous bytes), and every
// tap of the class then reads it shifted.  Weights come straight from L2 in
// operand order, one tap ahead of their use; a wave holds RT x CT tiles, so
// each weight operand feeds RT MFMA chains and each activation operand CT.
// Weights are the first MFMA operand: a lane then holds four consecutive
// channels of one pixel and stores 16 bytes.  4K (N = 192, M = 320): 20.36 ms
// with per-wave operand loads and fp32 MFMA, 7.2 ms now (the third layer
// with its inverse GDN 4.9 ms, 225 TFLOP/s of fp32 products, 1350 of bf16 ones,
// the matrix cores busy 68%); bf16 at 120x68 latents (N = 128): 1.98 -> 0.45 ms.
struct SynthArgs {
    const float* in;
    float* out;
    const void* wp[4];        // packed panel per output class: [Cop/16][chunk][tap][NW][64] operands
    const float* bias;        // [Cop] bias (GDN: beta), zero-padded
    int B, Hi, Wi, Ci;        // input [B][Hi][Wi][Ci] (GDN: one row of all pixels)
    int Co, Cop, nch;         // output channels, padded; chunks of 32 input channels
    int Ho, Wo;               // output pixels
    int twl, ntx, nty;        // log2 of the tile's width; tiles along x, y
    int ncb, ncls;            // column blocks, classes
    // inverse GDN in the epilogue of a transposed conv (k_synth with FUSE):
    const void* gwp;          // packed gamma^T [Cop/16][chunk][NW][64]
    const float* beta;        // [Cop]
};

constexpr int kSynthGroup = 32;   // tiles of a group (see k_synth)

struct SF32 {                 // fp32 transform: three parts of each operand
    static constexpr int kNx = 3, kNw = 3;
};
struct SBF16 {                // bf16 transform: bf16 weights, bf16-pair activations
    static constexpr int kNx = 2, kNw = 1;
};
template <class P>
constexpr bool kSplit3 = P::kNw == 3;

// Workgroups of 128 pixels in a layer from which they are the faster ones (two
// fit a compute unit).  us of a whole transform with that layer in 128 x 192
// tiles, inverse GDN in them, and in 64 x 64, for layers of this many of them.
// fp32 (N = 128 unless said): 192 250 / 232, 300 365 / 355, 320 154 / 151, 325
// 1228 / 1215 (N = 192 2488 / 2418), 432 169 / 171 (N = 192 293 / 301), 468
// 488 / 486 (938 / 942), 675 653 / 671.  bf16: 192 138 / 128, 255 482 / 458
// (898 / 866), 300 183 / 183, 320 104 / 102, 325 610 / 589 (1118 / 1137), 432
// 107 / 116, 468 244 / 251.
template <class P>
constexpr int kSynthMinBlocks = kSplit3<P> ? 432 : 320;

// Parts of eight values.  Three: x0 cut off after eight bits (rounded it could
// overflow), x1 rounded, x2 what is left; two: rounded, and the rest rounded.
template <int N>
__device__ __forceinline__ void split_parts(const float (&x)[8], b8 (&p)[N]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        __bf16 h;
        if constexpr (N == 3) h = __builtin_bit_cast(__bf16, (uint16_t)(__builtin_bit_cast(unsigned, x[q]) >> 16));
        else h = (__bf16)x[q];
        float r = x[q] - (float)h;
        p[0][q] = h;
#pragma unroll
        for (int n = 1; n < N; ++n) {
            p[n][q] = (__bf16)r;
            r -= (float)p[n][q];
        }
    }
}
// acc[j] += the product of the parts w[j] and x.  The six products of three
// parts are summed by themselves, the small ones first, so that acc is rounded
// once per 32 values of k.
template <class P, int CT>
__device__ __forceinline__ void mma_parts(const b8 (&w)[CT][P::kNw], const b8 (&x)[P::kNx], f4 (&acc)[CT]) {
    if constexpr (kSplit3<P>) {
        f4 t[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) t[j] = zero4();
        auto one = [&](int iw, int ix) {
#pragma unroll
            for (int j = 0; j < CT; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][iw], x[ix], t[j], 0, 0, 0);
        };
        one(2, 0);
        one(1, 1);
        one(0, 2);
        one(1, 0);
        one(0, 1);
        one(0, 0);
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[j] = acc[j] + t[j];
    } else {
#pragma unroll
        for (int ix = 0; ix < P::kNx; ++ix)
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][0], x[ix], acc[j], 0, 0, 0);
    }
}

__device__ __forceinline__ bool not_finite(const f4& v) {
    unsigned m = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) m = max(m, __builtin_bit_cast(unsigned, v[q]) & 0x7fffffffu);
    return m >= 0x7f800000u;
}

template <int MODE, int RT, int CT, int WC>
struct SynthShape {
    static constexpr int kWr = 4 / WC;                         // waves along the pixels
    static constexpr int kPx = 16 * RT * kWr;                  // pixels of a workgroup
    static constexpr int kCols = 16 * CT * WC;                 // output channels of a workgroup
    static constexpr int kHalo = MODE == XM_GDN ? 0 : 1;
    // patch pixels: 128 as 16 x 8 or 8 x 16 (180 with the halo), 64 as 16 x 4
    // or 8 x 8 (108), rounded up to 16: the k-groups' planes then start 256
    // bytes apart, and the lanes that one LDS cycle serves hit distinct banks
    static constexpr int kPatch = !kHalo ? kPx : (kPx == 128 ? 192 : 112);
    static constexpr int kItems = (kPatch * 4 + kThreads - 1) / kThreads;
};

// The wave's tile on fp32 MFMA, from the inputs and the weights put back
// together.
template <int MODE, int RT, int CT, class QY, class QX>
__device__ __forceinline__ void conv_tile_f32(const SynthArgs& a, const void* wp, int nk, int ntap, int nkx, int b, QY qy,
                                              QX qx, int ct0, f4 (&acc)[RT][CT]) {
    const int lane = threadIdx.x & 63, kq = lane >> 4;
    const b8* w = static_cast<const b8*>(wp) + lane;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = zero4();
    for (int k = 0; k < nk; ++k) {
        const int ch = k / ntap, t = k - ch * ntap, ty = t / nkx, tx = t - ty * nkx;
        const int dy = MODE == XM_DECONV ? 1 - ty : (MODE == XM_GDN ? 0 : ty - 1);
        const int dx = MODE == XM_DECONV ? 1 - tx : (MODE == XM_GDN ? 0 : tx - 1);
        const int c = ch * 32 + kq * 8;
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const bool cv = (ct0 + j) * kTile < a.Cop;
            const b8* p = w + ((size_t)(cv ? ct0 + j : 0) * nk + k) * 3 * 64;
            const b8 w0 = p[0], w1 = p[64], w2 = p[128];
            float wf[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) wf[q] = ((float)w0[q] + (float)w1[q]) + (float)w2[q];
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
// read and wrote the activations: third layer at 4K, f16 pairs, 2.45 + 1.31 ms
// against 3.2).
template <class P, int RT, int CT, class Store>
__device__ __forceinline__ void gdn_epilogue(const SynthArgs& a, f4 (&acc)[RT][CT], int ct0, b8* lds, Store store) {
    constexpr int NX = P::kNx, NW = P::kNw, HR = RT / 2, HP = HR * kTile;   // row tiles and pixels of a half
    const int lane = threadIdx.x & 63, kq = lane >> 4, nct = a.Cop / kTile, nch = (a.Co + 31) / 32;
    const int part = nch * 4 * HP;                       // 16-byte operands of one part
    const b8* w = static_cast<const b8*>(a.gwp) + lane;
    size_t wo[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) wo[j] = (size_t)(ct0 + j < nct ? ct0 + j : 0) * nch * NW * 64;
    auto load_w = [&](int c, b8 (&wv)[CT][NW]) {
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int n = 0; n < NW; ++n) wv[j][n] = w[wo[j] + (size_t)(c * NW + n) * 64];
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        b8 wv[CT][NW];
        load_w(0, wv);
        __syncthreads();                                 // the last patch, or the first half's operands, have been read
        // operands [part][chunk][k-group][pixel]
#pragma unroll
        for (int i = 0; i < HR; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                const f4 x = acc[h * HR + i][j], x2 = x * x;
                const int n = (ct0 + j) * kTile + kq * 4;
                if (n >= nch * 32) continue;             // (wave-uniform: a column tile past the last chunk)
                const int at = (n >> 3) * HP + i * kTile + (lane & 15);
                const float v[8] = {x2.x, x2.y, x2.z, x2.w};
                b8 p[NX];
                split_parts<NX>(v, p);
#pragma unroll
                for (int m = 0; m < NX; ++m) {
                    typedef __bf16 b4 __attribute__((ext_vector_type(4)));
                    *reinterpret_cast<b4*>(reinterpret_cast<uint16_t*>(&lds[at + m * part]) + (n & 4)) = p[m].lo;
                }
            }
        __syncthreads();
        f4 z[HR][CT];
#pragma unroll
        for (int i = 0; i < HR; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) z[i][j] = zero4();
        for (int c = 0; c < nch; ++c) {
            if (c) load_w(c, wv);
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const int at = (c * 4 + kq) * HP + i * kTile + (lane & 15);
                b8 x[NX];
#pragma unroll
                for (int m = 0; m < NX; ++m) x[m] = lds[at + m * part];
                mma_parts<P, CT>(wv, x, z[i]);
            }
        }
        if constexpr (kSplit3<P>) {
            bool nf = false;
#pragma unroll
            for (int i = 0; i < HR; ++i)
#pragma unroll
                for (int j = 0; j < CT; ++j) nf |= not_finite(z[i][j]);
            if (__any(nf)) {                             // (as in synth_tile; the operands are still in LDS)
#pragma unroll
                for (int i = 0; i < HR; ++i)
#pragma unroll
                    for (int j = 0; j < CT; ++j) z[i][j] = zero4();
                for (int c = 0; c < nch; ++c) {
                    load_w(c, wv);
#pragma unroll
                    for (int i = 0; i < HR; ++i) {
                        const int at = (c * 4 + kq) * HP + i * kTile + (lane & 15);
                        const b8 x0 = lds[at], x1 = lds[at + part], x2 = lds[at + 2 * part];
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            // (an infinite square left NaN in its other parts)
                            float x = (float)x0[q];
                            if (__builtin_isfinite(x)) x = (x + (float)x1[q]) + (float)x2[q];
#pragma unroll
                            for (int j = 0; j < CT; ++j)
                                z[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    ((float)wv[j][0][q] + (float)wv[j][1][q]) + (float)wv[j][2][q], x, z[i][j], 0, 0, 0);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int n = (ct0 + j) * kTile + kq * 4;
            if (ct0 + j >= nct) continue;
            const f4 beta = *reinterpret_cast<const f4*>(a.beta + n);
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const f4 x = acc[h * HR + i][j], v = z[i][j] + beta;
                store(h * HR + i, n, f4{x.x * sqrtf(v.x), x.y * sqrtf(v.y), x.z * sqrtf(v.z), x.w * sqrtf(v.w)});
            }
        }
    }
}

// Workgroup `bid` of a launch.
template <class P, int MODE, int RT, int CT, int WC, bool FUSE>
__device__ __forceinline__ void synth_tile(const SynthArgs& a, int bid) {
    using S = SynthShape<MODE, RT, CT, WC>;
    constexpr int NX = P::kNx, NW = P::kNw, NI = S::kItems, NP = S::kPatch, HALO = S::kHalo;
    static_assert(!FUSE || (MODE == XM_DECONV && WC == 4), "a wave needs all pixels of the workgroup");
    // the patch [part][k-group][pixel]; FUSE: also the squares of half of the pixels, all channels
    constexpr int kGdn = FUSE ? NX * (S::kCols / 8) * (S::kPx / 2) : 0;
    __shared__ b8 patch[4 * NX * NP > kGdn ? 4 * NX * NP : kGdn];

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
    const b8* w = static_cast<const b8*>(a.wp[cls]) + lane;
    size_t wo[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) wo[j] = (size_t)(ct0 + j < nct ? ct0 + j : 0) * nk * NW * 64;
    auto load_w = [&](int k, b8 (&wv)[CT][NW]) {
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

    b8 wv[CT][NW], wn[CT][NW];
    load_chunk(0);
    load_w(0, wv);
    for (int ch = 0; ch < a.nch; ++ch) {
        __syncthreads();                                 // the chunk before has been read
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int e = threadIdx.x + n * kThreads;
            if (NP * 4 % kThreads == 0 || e < NP * 4) {
                b8 p[NX];
                split_parts<NX>(st[n], p);
#pragma unroll
                for (int m = 0; m < NX; ++m) patch[(4 * m + (e & 3)) * NP + (e >> 2)] = p[m];
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
                    b8 x[NX];
#pragma unroll
                    for (int m = 0; m < NX; ++m) x[m] = patch[4 * m * NP + at + i * step];
                    mma_parts<P, CT>(wv, x, acc[i]);
                }
#pragma unroll
                for (int j = 0; j < CT; ++j)
#pragma unroll
                    for (int n = 0; n < NW; ++n) wv[j][n] = wn[j][n];
            }
    }

    auto qy = [&](int i) { return y0 + ((r0 + i * kTile) >> a.twl); };   // row tile i's pixel of this lane
    auto qx = [&](int i) { return x0 + ((r0 + i * kTile) & (TW - 1)); };
    if constexpr (kSplit3<P>) {
        bool nf = false;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) nf |= not_finite(acc[i][j]);
        if (__any(nf)) conv_tile_f32<MODE, RT, CT>(a, a.wp[cls], nk, ntap, nkx, b, qy, qx, ct0, acc);
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
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            acc[i][j] = acc[i][j] + add;
            // inverse GDN of the workgroup: zeros off the grid and past the last channel
            if (FUSE) acc[i][j] = cv && inside(i) ? acc[i][j] : zero4();
        }
    }
    if constexpr (FUSE) {
        gdn_epilogue<P, RT, CT>(a, acc, ct0, patch, store);
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
// n < ncol, in (chunk of 32 channels, tap, channel) order, rounded to bf16 or
// in three parts.
template <class T, class F>
inline void pack_split(bool bf, int nclass, int Ci, int ncol, int Cop, T ntap, F wt, std::vector<uint16_t> (&out)[4]) {
    const int nch = (Ci + 31) / 32, nw = bf ? 1 : 3;
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
                        uint16_t p[3];
                        bf16_parts(f, p);
                        for (int m = 0; m < 3; ++m) v[at + m * 64 * 8] = p[m];
                    }
                }
    }
}

}  // namespace wf
