// Products of fp32 values on fp32 MFMA, and of bf16-pair activations on bf16
// MFMA, in a fixed order of every sum: the layers of the hyper-decoder, and
// the plain product that hoists the hyperprior half of layer 1 before the
// resident driver's launch.
#pragma once

#include "wf_device.h"

namespace wf {

// What a tile computes: transposed conv 5x5 s2, conv 3x3, inverse GDN,
// transposed conv with the classes as columns, plain product (conv_tile: the
// first two and the last; synth_tile: all but conv 3x3).
enum { XM_DECONV = 0, XM_CONV3 = 1, XM_GDN = 2, XM_DECONV4 = 3, XM_GEMM = 4 };

// psi feeds the entropy parameters, and an encoder and a decoder have to agree
// on every bit of them, so the hyper-decoder's layers keep fp32 MFMA and one
// accumulation order per output, whatever the tile: the taps in raster order, each tap's
// input channels ascending.  Bound by the matrix cores (248 GFLOP at 4K,
// 157 TFLOP/s) on large grids, by the length of that chain on small ones.
//
// A workgroup owns 16 RT WR pixels of one class and 16 CT WC channels.  Each
// step is one tap's chunk of 32 input channels: its pixels are staged in LDS
// in operand order ([operand][k-group][pixel], 16 bytes each), double-buffered
// with one barrier a step, the loads two steps ahead of their use; weights
// come from L2 in operand order, also two steps ahead.  The four MFMAs of an
// fp32 k-block go round the wave's tiles, so that consecutive ones do not
// depend on each other.  Weights are the first operand: a lane holds four
// consecutive channels of one pixel and stores 16 bytes.  4K (N = 192,
// M = 320): 3.03 ms before (operands loaded per wave, 128 x 64 tiles, one
// k-block's MFMAs in a chain), 2.04 now (122 TFLOP/s); a 32x48 latent
// (N = 128, M = 192) 291 -> 100 us.
struct ConvArgs {
    const float* in;
    float* out;
    const void* wp[4];        // packed panel per output class
    const float* bias;        // [Co]
    int B, Hi, Wi, Ci;        // input [B][Hi][Wi][Ci]
    int Hq, Wq;               // output pixels of one class per image (rows = B Hq Wq)
    int Co, Cop;              // output channels, and padded to whole column tiles
    int Ho, Wo;               // output array [B][Ho][Wo][Co]; pixels outside are not stored
    int relu;
    int nrb, ncb;             // row and column blocks
};

template <int RT, int CT, int WC>
struct ConvShape {
    static constexpr int kWr = 4 / WC;                         // waves along the pixels
    static constexpr int kPx = 16 * RT * kWr, kCols = 16 * CT * WC;
    static constexpr int kItems = (kPx * 4 + kThreads - 1) / kThreads;   // 8-channel pieces a thread stages
};

// Workgroup `bid` of class `cls`.
template <class P, int MODE, int RT, int CT, int WC>
__device__ __forceinline__ void conv_tile(const ConvArgs& a, int bid, int cls) {
    using Bw = typename P::B;
    using S = ConvShape<RT, CT, WC>;
    constexpr int NI = S::kItems, PX = S::kPx, NB = 32 / P::kK;   // weight k-blocks of a chunk
    constexpr bool DEEP = RT * CT * NB < 16;                      // weights two steps ahead (else one: registers)
    __shared__ f4 tile[2][8][PX];      // fp32: [k-block][k-group]; bf16: [hi, lo][k-group]
    // neighbouring rows on one XCD, the column blocks of a row block together
    const int per = (a.nrb + kXcds - 1) / kXcds, l = bid / kXcds;
    const int rb = (bid % kXcds) * per + l / a.ncb, cb = l % a.ncb;
    if (rb >= a.nrb) return;
    const int py = cls >> 1, px = cls & 1;
    const int nky = MODE == XM_GEMM ? 1 : (MODE == XM_DECONV && py ? 2 : 3);
    const int nkx = MODE == XM_GEMM ? 1 : (MODE == XM_DECONV && px ? 2 : 3);
    const int nch = (a.Ci + 31) / 32, ns = nky * nkx * nch;       // steps
    const int cbn = a.Ci / P::kK, nkb = nky * nkx * cbn;          // weight k-blocks of a tap, of all
    const int nrows = a.B * a.Hq * a.Wq, nct = a.Cop / kTile;
    const int wave = wave_id(), lane = threadIdx.x & 63, kq = lane >> 4;
    const int wr = wave / WC, wc = wave % WC, ct0 = (cb * WC + wc) * CT;

    // staged pieces of this thread: pixel e / 4, channels 8 (e % 4) .. + 8
    int iy[NI], ix[NI], at[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int e = threadIdx.x + n * kThreads, r = rb * PX + (e >> 2);
        const bool ok = e < PX * 4 && r < nrows;
        const int rr = ok ? r : 0, b = rr / (a.Hq * a.Wq), rem = rr - b * a.Hq * a.Wq;
        iy[n] = ok ? rem / a.Wq : -4;                             // (-4: no tap of it lies on the grid)
        ix[n] = rem - rem / a.Wq * a.Wq;
        at[n] = ((b * a.Hi + rem / a.Wq) * a.Wi + ix[n]) * a.Ci + (e & 3) * 8;
    }
    struct Stage {
        f4 u[NI], v[NI];
    };
    // step s: tap (ty, tx), chunk ch
    auto load_in = [&](int ty, int tx, int ch, Stage& st) {
        const int dy = MODE == XM_GEMM ? 0 : (MODE == XM_DECONV ? 1 - ty : ty - 1);
        const int dx = MODE == XM_GEMM ? 0 : (MODE == XM_DECONV ? 1 - tx : tx - 1);
        const int off = (dy * a.Wi + dx) * a.Ci + ch * 32;
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int y = iy[n] + dy, x = ix[n] + dx;
            const bool ok = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi && ch * 32 + (threadIdx.x & 3) * 8 < a.Ci;
            st.u[n] = ld4<false>(a.in, (size_t)(at[n] + off), ok);
            st.v[n] = ld4<false>(a.in, (size_t)(at[n] + off + 4), ok);
        }
    };
    auto stage = [&](const Stage& st, f4 (*t)[PX]) {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int e = threadIdx.x + n * kThreads, p = e >> 2, g = e & 3;
            if (PX * 4 % kThreads && e >= PX * 4) continue;
            if constexpr (P::kBf16) {
                const b8x2 h = split8(st.u[n], st.v[n]);
                t[g][p] = __builtin_bit_cast(f4, h.hi);
                t[4 + g][p] = __builtin_bit_cast(f4, h.lo);
            } else {
                t[g * 2][p] = st.u[n];                            // (channels 8 g .. : k-block g / 2)
                t[g * 2 + 1][p] = st.v[n];
            }
        }
    };
    const Bw* w = static_cast<const Bw*>(a.wp[cls]) + lane;
    size_t wo[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) wo[j] = (size_t)(ct0 + j < nct ? ct0 + j : 0) * nkb * 64;
    struct Weights {
        Bw w[CT][NB];
    };
    auto load_w = [&](int tap, int ch, Weights& wv) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int k = min(tap * cbn + ch * NB + n, nkb - 1);
#pragma unroll
            for (int j = 0; j < CT; ++j) wv.w[j][n] = w[wo[j] + (size_t)k * 64];
        }
    };
    f4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = zero4();
    const int r0 = wr * RT * kTile + (lane & 15);
    auto products = [&](int ch, const Weights& wv, const f4 (*t)[PX]) {
        if constexpr (P::kBf16) {
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const b8 hi = __builtin_bit_cast(b8, t[kq][r0 + i * kTile]);
                const b8 lo = __builtin_bit_cast(b8, t[4 + kq][r0 + i * kTile]);
#pragma unroll
                for (int j = 0; j < CT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.w[j][0], hi, acc[i][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < CT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.w[j][0], lo, acc[i][j], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                if (n && ch * 32 + 16 >= a.Ci) break;             // (Ci = 16 mod 32: the last chunk is half)
                f4 x[RT];
#pragma unroll
                for (int i = 0; i < RT; ++i) x[i] = t[n * 4 + kq][r0 + i * kTile];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < RT; ++i)
#pragma unroll
                        for (int j = 0; j < CT; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv.w[j][n][q], x[i][q], acc[i][j], 0, 0, 0);
            }
        }
    };

    // Steps in order of (tap, chunk); `q*` is the step being loaded, two ahead
    // of the products (past the end: the last one again, not used).
    int ch = 0, qt = 0, qty = 0, qtx = 0, qch = 0, pt = 0, pch = 0;   // (p*: the step before q*)
    auto advance = [&] {
        pt = qt;
        pch = qch;
        if (++qch < nch) return;
        if (qt + 1 == nky * nkx) {
            qch = nch - 1;
            return;
        }
        qch = 0;
        ++qt;
        if (++qtx == nkx) {
            qtx = 0;
            ++qty;
        }
    };
    Stage s0, s1;
    Weights w0, w1, w2;
    load_in(0, 0, 0, s0);
    load_w(0, 0, w0);
    advance();
    load_in(qty, qtx, qch, s1);
    if (DEEP) load_w(qt, qch, w1);
    advance();
    stage(s0, tile[0]);
    __syncthreads();
    // one step: load step s + 2 into sl and step s + 2 (or s + 1) into wl,
    // products of step s, stage step s + 1
    auto step = [&](int s, Stage& sl, const Stage& sn, Weights& wl, const Weights& wu) {
        load_w(DEEP ? qt : pt, DEEP ? qch : pch, wl);
        load_in(qty, qtx, qch, sl);
        advance();
        __builtin_amdgcn_sched_barrier(0);
        products(ch, wu, tile[s & 1]);
        if (++ch == nch) ch = 0;
        stage(sn, tile[(s & 1) ^ 1]);
        __syncthreads();
    };
    if constexpr (DEEP) {
        for (int s = 0; s < ns; s += 6) {
            step(s, s0, s1, w2, w0);
            if (s + 1 < ns) step(s + 1, s1, s0, w0, w1);
            if (s + 2 < ns) step(s + 2, s0, s1, w1, w2);
            if (s + 3 < ns) step(s + 3, s1, s0, w2, w0);
            if (s + 4 < ns) step(s + 4, s0, s1, w0, w1);
            if (s + 5 < ns) step(s + 5, s1, s0, w1, w2);
        }
    } else {
        for (int s = 0; s < ns; s += 2) {
            step(s, s0, s1, w1, w0);
            if (s + 1 < ns) step(s + 1, s1, s0, w0, w1);
        }
    }

    // a lane holds channels 4 (lane / 16) + q of each column tile, pixel lane % 16
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int r = rb * PX + r0 + i * kTile;
        if (r >= nrows) continue;
        const int b = r / (a.Hq * a.Wq), rem = r - b * a.Hq * a.Wq, qy = rem / a.Wq, qx = rem - qy * a.Wq;
        const int oy = MODE == XM_DECONV ? 2 * qy + py : qy, ox = MODE == XM_DECONV ? 2 * qx + px : qx;
        if (oy >= a.Ho || ox >= a.Wo) continue;
        float* o = a.out + (((size_t)b * a.Ho + oy) * a.Wo + ox) * a.Co + kq * 4;
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            if (ct0 + j >= nct) continue;
            const int n = (ct0 + j) * kTile;
            f4 v = acc[i][j] + *reinterpret_cast<const f4*>(a.bias + n + kq * 4);
            if (a.relu) v = f4{fmaxf(v.x, 0.0f), fmaxf(v.y, 0.0f), fmaxf(v.z, 0.0f), fmaxf(v.w, 0.0f)};
            *reinterpret_cast<f4u*>(o + n) = v;      // (psi need only be aligned to 4 bytes)
        }
    }
}

}  // namespace wf
