// The transforms around the autoregressive decode (the latent pipeline of
// Sec. II-A): the hyper-decoder h_s (z_hat -> the hyperprior half psi of the
// entropy parameters) and the synthesis transform g_s (y_hat -> image), for
// an end-to-end decode timing with random weights.  Layer list (the paper
// names the models, not their layers; this is the mean-scale hyperprior model
// of the family the workloads are named after):
//   h_s: transposed conv 5x5 s2 (N -> M), ReLU; transposed conv 5x5 s2
//        (M -> 3M/2), ReLU; conv 3x3 s1 (3M/2 -> 2M), cropped to the H x W grid
//   g_s: 3 x (transposed conv 5x5 s2, inverse GDN) (M -> N -> N -> N), then
//        transposed conv 5x5 s2 (N -> 3)
//
// Every layer is an implicit GEMM on MFMA: k_conv for h_s, k_synth for g_s.  A stride-2 transposed
// conv (padding 2, output padding 1) splits into four output parity classes
// (oy mod 2, ox mod 2); class (py, px) is an ordinary product over the taps
// ky = py + 2 ty, kx = px + 2 tx, reading input pixel (qy + 1 - ty, qx + 1 - tx)
// for output pixel (2 qy + py, 2 qx + px).  Rows of the product are the class's
// output pixels, columns the output channels, k the (tap, input channel)
// pairs, tap-major.  Inverse GDN is the same product over the channels of
// the squared input, x_c sqrt(beta_c + sum_j gamma_cj x_j^2), with gamma^T
// as the weight panel.  Weights are packed per layer and class in the operand
// order of the step kernels.  A transposed conv with at most 4 output
// channels (the image's 3) puts all four classes into the columns instead:
// rows are input pixels, columns (class, channel), k the 3x3 input
// neighbourhood (taps a class does not use have zero weights), so one
// 16-column tile carries all 12 outputs of an input pixel.
#include <utility>
#include <vector>

#include "wf_conv.h"
#include "wf_device.h"
#include "wf_pack.h"
#include "wf_split.h"

namespace wf {

// ---- plan -------------------------------------------------------------------

struct Layer {
    int mode, Ci, Co, Cop, relu;
    const void* wp[4];
    const float* bias;        // h_s: [Co]; g_s: [Cop] (GDN: beta)
};

struct Xform {
    int N, M, B, H, W, Hz, Wz, precision;
    int device = 0;
    std::vector<void*> owned;
    Layer hs[3], gs[4], gdn[3];
    float *hs_a = nullptr, *hs_b = nullptr, *g_a = nullptr, *g_b = nullptr;
};

static int xf_fail_hip(hipError_t e, const char* what) {
    return fail(WF_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

template <class T>
static int xf_upload(Xform* x, const T** dst, const std::vector<T>& v) {
    T* p = nullptr;
    hipError_t e = hipMalloc((void**)&p, v.size() * sizeof(T));
    if (e != hipSuccess) return fail(WF_E_NOMEM, std::string("transform weights: ") + hipGetErrorString(e));
    x->owned.push_back(p);
    e = hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
    if (e != hipSuccess) return xf_fail_hip(e, "transform weights");
    *dst = p;
    return WF_OK;
}

static int xf_alloc(Xform* x, float** dst, size_t n) {
    hipError_t e = hipMalloc((void**)dst, n * sizeof(float));
    if (e != hipSuccess) return fail(WF_E_NOMEM, std::string("transform workspace: ") + hipGetErrorString(e));
    x->owned.push_back(*dst);
    return WF_OK;
}

// Pack one layer: wt(k, n) of class c over k = (tap, input channel), tap-major.
template <class F>
static int xf_pack(Xform* x, Layer& L, int nclass, F wt) {
    const bool bf = x->precision == WF_BF16;
    for (int c = 0; c < nclass; ++c) {
        const int nky = L.mode == XM_DECONV && (c >> 1) ? 2 : 3, nkx = L.mode == XM_DECONV && (c & 1) ? 2 : 3;
        const int K = nky * nkx * L.Ci;
        auto f = [&](int k, int n) { return wt(c, k / L.Ci, nkx, k % L.Ci, n); };
        int rc = bf ? xf_upload(x, reinterpret_cast<const uint16_t**>(&L.wp[c]), pack_panel_bf16(K, L.Co, K, L.Cop, f))
                    : xf_upload(x, reinterpret_cast<const float**>(&L.wp[c]), pack_panel(K, L.Co, K, L.Cop, f));
        if (rc != WF_OK) return rc;
    }
    for (int c = nclass; c < 4; ++c) L.wp[c] = L.wp[0];
    return WF_OK;
}

// Pack one layer of g_s for k_synth (see pack_split) and the bias (or beta) of
// every column.
template <class F, class G>
static int xf_pack_synth(Xform* x, Layer& L, int nclass, int ncol, F wt, G bias) {
    auto ntap = [&](int c, int& nkx) {
        nkx = L.mode == XM_GDN ? 1 : (L.mode == XM_DECONV && (c & 1) ? 2 : 3);
        return nkx * (L.mode == XM_GDN ? 1 : (L.mode == XM_DECONV && (c >> 1) ? 2 : 3));
    };
    std::vector<uint16_t> v[4];
    pack_split(x->precision == WF_BF16, nclass, L.Ci, ncol, L.Cop, ntap, wt, v);
    int rc = WF_OK;
    for (int c = 0; c < nclass && rc == WF_OK; ++c) rc = xf_upload(x, reinterpret_cast<const uint16_t**>(&L.wp[c]), v[c]);
    for (int c = nclass; c < 4; ++c) L.wp[c] = L.wp[0];
    std::vector<float> bv(L.Cop, 0.0f);
    for (int n = 0; n < ncol; ++n) bv[n] = bias(n);
    return rc != WF_OK ? rc : xf_upload(x, &L.bias, bv);
}

// Transposed conv weight W[ci][co][5][5]: tap t of class (py, px) is
// (ky, kx) = (py + 2 (t / nkx), px + 2 (t % nkx)).
static float deconv_w(const float* w, int Co, int c, int t, int nkx, int ci, int co) {
    const int ky = (c >> 1) + 2 * (t / nkx), kx = (c & 1) + 2 * (t % nkx);
    return w[(((size_t)ci * Co + co) * 5 + ky) * 5 + kx];
}

static int xf_deconv(Xform* x, Layer& L, const float* w, const float* b, int Ci, int Co, int relu) {
    L.mode = XM_DECONV; L.Ci = Ci; L.Co = Co; L.Cop = (Co + kTile - 1) / kTile * kTile; L.relu = relu;
    int rc = xf_pack(x, L, 4, [&](int c, int t, int nkx, int ci, int co) { return deconv_w(w, Co, c, t, nkx, ci, co); });
    if (rc != WF_OK) return rc;
    return xf_upload(x, &L.bias, std::vector<float>(b, b + Co));
}

static int xf_synth_deconv(Xform* x, Layer& L, const float* w, const float* b, int Ci, int Co) {
    L.mode = XM_DECONV; L.Ci = Ci; L.Co = Co; L.Cop = (Co + kTile - 1) / kTile * kTile; L.relu = 0;
    return xf_pack_synth(x, L, 4, Co,
        [&](int c, int t, int nkx, int ci, int co) { return deconv_w(w, Co, c, t, nkx, ci, co); },
        [&](int n) { return b[n]; });
}

// All four classes in the columns (Co <= 4): column n = class * Co + co, tap
// (dy, dx) = (t / 3 - 1, t % 3 - 1) of the input neighbourhood, which class
// (py, px) reaches through (ky, kx) = (py + 2 - 2 dy, px + 2 - 2 dx) when both
// are at most 4 (zero weight otherwise).
static int xf_synth_deconv4(Xform* x, Layer& L, const float* w, const float* b, int Ci, int Co) {
    L.mode = XM_DECONV4; L.Ci = Ci; L.Co = Co; L.Cop = (4 * Co + kTile - 1) / kTile * kTile; L.relu = 0;
    return xf_pack_synth(x, L, 1, 4 * Co,
        [&](int, int t, int, int ci, int n) -> float {
            const int cls = n / Co, co = n - cls * Co;
            const int ky = (cls >> 1) + 2 - 2 * (t / 3 - 1), kx = (cls & 1) + 2 - 2 * (t % 3 - 1);
            if (ky > 4 || kx > 4) return 0.0f;
            return w[(((size_t)ci * Co + co) * 5 + ky) * 5 + kx];
        },
        [&](int n) { return b[n % Co]; });
}

static int xf_conv3(Xform* x, Layer& L, const float* w, const float* b, int Ci, int Co) {
    L.mode = XM_CONV3; L.Ci = Ci; L.Co = Co; L.Cop = (Co + kTile - 1) / kTile * kTile; L.relu = 0;
    int rc = xf_pack(x, L, 1, [&](int, int t, int, int ci, int co) {
        return w[(((size_t)co * Ci + ci) * 3 + t / 3) * 3 + t % 3];
    });
    if (rc != WF_OK) return rc;
    return xf_upload(x, &L.bias, std::vector<float>(b, b + Co));
}

static int xf_synth_gdn(Xform* x, Layer& L, const float* beta, const float* gamma, int C) {
    L.mode = XM_GDN; L.Ci = C; L.Co = C; L.Cop = (C + kTile - 1) / kTile * kTile; L.relu = 0;
    return xf_pack_synth(x, L, 1, C, [&](int, int, int, int j, int c) { return gamma[(size_t)c * C + j]; },
                         [&](int n) { return beta[n]; });
}

constexpr long long kConvSmall = 1000000, kConvMidF32 = 2600000, kConvMidBf16 = 2000000, kConvWide = 8000000;

static int ceil_div(int a, int b) { return (a + b - 1) / b; }

template <class P, int MODE, int RT, int CT, int WC>
__global__ __launch_bounds__(kThreads, 2) void k_conv(ConvArgs a) {
    conv_tile<P, MODE, RT, CT, WC>(a, blockIdx.x, blockIdx.y);
}

template <class P, int MODE, int RT, int CT, int WC>
static void launch_conv(ConvArgs a, hipStream_t st) {
    using S = ConvShape<RT, CT, WC>;
    a.nrb = ceil_div(a.B * a.Hq * a.Wq, S::kPx);
    a.ncb = ceil_div(a.Cop, S::kCols);
    const dim3 grid(kXcds * ceil_div(a.nrb, kXcds) * a.ncb, MODE == XM_DECONV ? 4 : 1);
    hipLaunchKernelGGL((k_conv<P, MODE, RT, CT, WC>), grid, dim3(kThreads), 0, st, a);
}

template <class P, int MODE>
static void launch_layer(const Layer& L, const float* in, float* out, int B, int Hi, int Wi, int Hq, int Wq, int Ho,
                         int Wo, hipStream_t st) {
    ConvArgs a{};
    a.in = in; a.out = out; a.bias = L.bias;
    for (int c = 0; c < 4; ++c) a.wp[c] = L.wp[c];
    a.B = B; a.Hi = Hi; a.Wi = Wi; a.Ci = L.Ci; a.Hq = Hq; a.Wq = Wq;
    a.Co = L.Co; a.Cop = L.Cop; a.Ho = Ho; a.Wo = Wo; a.relu = L.relu;
    const long long rows = (long long)B * Hq * Wq * (MODE == XM_DECONV ? 4 : 1);
    // Pixels x channels of a workgroup by the layer's outputs, so that small
    // layers still spread over the chip (us per layer, 16 x 64 / 32 x 64 / the
    // larger tile).  fp32: 0.59 M outputs 56 / 64 / 67, 1.9 M 107 / 91 / 106,
    // 3.9 M 211 / 191 / 158; 4K's 20.7 M 2000 / 1700 / 1560 (before: 2170),
    // 128 x 160 1580.  bf16: 0.98 M 62 / 63 / 68, 2.4 M 145 / 96 / 89; 20.7 M
    // 1060 / 680 / 473, and 405 with 128 x 160 (before: 1373), which only pays
    // where 160 divides the channels (12.4 M outputs in 384: 197, 64 x 96 167).
    const long long outputs = rows * L.Cop;
    if (outputs < kConvSmall) launch_conv<P, MODE, 1, 1, 4>(a, st);
    else if (outputs < (P::kBf16 ? kConvMidBf16 : kConvMidF32)) launch_conv<P, MODE, 2, 1, 4>(a, st);
    else if constexpr (!P::kBf16) launch_conv<P, MODE, 4, 1, 4>(a, st);
    else if (outputs >= kConvWide && L.Cop % 160 == 0) launch_conv<P, MODE, 4, 5, 2>(a, st);
    else launch_conv<P, MODE, 2, 3, 2>(a, st);
}

template <class P>
static void run_layer(const Layer& L, const float* in, float* out, int B, int Hi, int Wi, int Ho, int Wo,
                      hipStream_t st) {
    if (L.mode == XM_DECONV) launch_layer<P, XM_DECONV>(L, in, out, B, Hi, Wi, Hi, Wi, Ho, Wo, st);
    else launch_layer<P, XM_CONV3>(L, in, out, B, Hi, Wi, Ho, Wo, Ho, Wo, st);
}

template <class P, int MODE, int RT, int CT, int WC, bool FUSE>
__global__ __launch_bounds__(kThreads, 2) void k_synth(SynthArgs a) {
    synth_tile<P, MODE, RT, CT, WC, FUSE>(a, blockIdx.x);
}

// Tiles of a launch: along x and y, for a tile 2^twl wide.
template <class S>
static int synth_tiles(SynthArgs& a, int twl) {
    const int tw = 1 << twl, th = S::kPx >> twl;
    a.twl = twl;
    a.ntx = ceil_div(a.Wi, tw);
    a.nty = ceil_div(a.Hi, th);
    return a.ntx * a.nty;
}

template <class P, int MODE, int RT, int CT, int WC, bool FUSE = false>
static void launch_synth(SynthArgs a, hipStream_t st) {
    using S = SynthShape<MODE, RT, CT, WC>;
    if (!S::kHalo) synth_tiles<S>(a, S::kPx == 128 ? 7 : 6);
    else if (synth_tiles<S>(a, 3) >= synth_tiles<S>(a, 4)) synth_tiles<S>(a, 4);   // the shape that pads less
    else synth_tiles<S>(a, 3);
    a.ncb = ceil_div(a.Cop, S::kCols);
    const int per = ceil_div(a.B * a.nty * a.ntx, kXcds);
    hipLaunchKernelGGL((k_synth<P, MODE, RT, CT, WC, FUSE>), dim3(kXcds * per * a.ncls * a.ncb), dim3(kThreads), 0, st, a);
}

static SynthArgs synth_args(const Layer& L, const float* in, float* out, int B, int h, int w) {
    SynthArgs a{};
    a.in = in; a.out = out; a.bias = L.bias;
    for (int c = 0; c < 4; ++c) a.wp[c] = L.wp[c];
    a.Ci = L.Ci; a.Co = L.Co; a.Cop = L.Cop; a.nch = ceil_div(L.Ci, 32);
    a.B = B; a.Hi = h; a.Wi = w; a.Ho = 2 * h; a.Wo = 2 * w; a.ncls = L.mode == XM_DECONV ? 4 : 1;
    return a;
}

// A transposed conv and its inverse GDN, [B][h][w][Ci] -> [B][2h][2w][Co]:
// in one kernel into `other` where a workgroup of 128 pixels holds every
// channel (up to 192) and the layer has enough of them.
// Otherwise the conv writes `other` and the GDN `own`, the buffer that may hold
// the conv's input.  Returns the output.
template <class P>
static float* run_synth(const Layer& L, const Layer& G, const float* in, float* own, float* other, int B, int h, int w,
                        hipStream_t st) {
    SynthArgs a = synth_args(L, in, other, B, h, w);
    const long long nb = 4LL * B * h * w / 128;
    if (nb >= kSynthMinBlocks<P> && L.Cop <= 192) {
        a.gwp = G.wp[0]; a.beta = G.bias;
        if (L.Cop <= 128) launch_synth<P, XM_DECONV, 8, 2, 4, true>(a, st);
        else launch_synth<P, XM_DECONV, 8, 3, 4, true>(a, st);
        return other;
    }
    SynthArgs g = synth_args(G, other, own, 1, 1, B * 4 * h * w);
    g.Ho = 1;
    g.Wo = g.Wi;
    if (nb * ceil_div(L.Cop, 192) >= kSynthMinBlocks<P>) {
        launch_synth<P, XM_DECONV, 8, 3, 4>(a, st);
        launch_synth<P, XM_GDN, 8, 3, 4>(g, st);
    } else {
        launch_synth<P, XM_DECONV, 4, 1, 4>(a, st);
        launch_synth<P, XM_GDN, 4, 1, 4>(g, st);
    }
    return own;
}

template <class P>
static void hyper(const Xform& x, const float* z, float* psi, hipStream_t st) {
    const int B = x.B, Hz = x.Hz, Wz = x.Wz;
    run_layer<P>(x.hs[0], z, x.hs_a, B, Hz, Wz, 2 * Hz, 2 * Wz, st);
    run_layer<P>(x.hs[1], x.hs_a, x.hs_b, B, 2 * Hz, 2 * Wz, 4 * Hz, 4 * Wz, st);
    run_layer<P>(x.hs[2], x.hs_b, psi, B, 4 * Hz, 4 * Wz, x.H, x.W, st);   // cropped to the latent grid
}

template <class P>
static void synth(const Xform& x, const float* y, float* img, hipStream_t st) {
    int h = x.H, w = x.W;
    const float* in = y;
    float *own = x.g_b, *other = x.g_a;
    for (int k = 0; k < 3; ++k) {
        float* out = run_synth<P>(x.gs[k], x.gdn[k], in, own, other, x.B, h, w, st);
        if (out == other) std::swap(own, other);
        in = out;
        h *= 2;
        w *= 2;
    }
    launch_synth<P, XM_DECONV4, 2, 1, 1>(synth_args(x.gs[3], in, img, x.B, h, w), st);
}

static void free_xform(Xform* x) {
    if (!x) return;
    for (void* p : x->owned)
        if (p) (void)hipFree(p);
    delete x;
}

}  // namespace wf

using namespace wf;

extern "C" {

int wf_xform_plan(const wf_xform_desc* d, wf_xform_t* out) {
    if (!out) return fail(WF_E_INVALID, "out is NULL");
    *out = nullptr;
    if (!d) return fail(WF_E_INVALID, "desc is NULL");
    if (d->N < 1 || d->M < 1 || d->B < 1 || d->H < 1 || d->W < 1)
        return fail(WF_E_INVALID, "N, M, B, H and W must be positive");
    if (d->precision != WF_FP32 && d->precision != WF_BF16) return fail(WF_E_INVALID, "unknown precision");
    if (!d->hs_w[0] || !d->hs_w[1] || !d->hs_w[2] || !d->hs_b[0] || !d->hs_b[1] || !d->hs_b[2])
        return fail(WF_E_INVALID, "a hyper-decoder weight pointer is NULL");
    for (int k = 0; k < 4; ++k)
        if (!d->gs_w[k] || !d->gs_b[k] || (k < 3 && (!d->gdn_beta[k] || !d->gdn_gamma[k])))
            return fail(WF_E_INVALID, "a synthesis weight pointer is NULL");
    const int kb = d->precision == WF_BF16 ? 32 : kTile;
    if (d->N % kb || d->M % kb || (d->M * 3 / 2) % kb || d->M % 2)
        return fail(WF_E_UNSUPPORTED, "N, M and 3M/2 must be multiples of the k-block (16 fp32, 32 bf16)");
    const long long big = (long long)d->B * 8 * d->H * 8 * d->W * d->N * 4;
    const long long lat = (long long)d->B * d->H * d->W * (long long)(d->M > 2 * d->M ? d->M : 2 * d->M) * 4;
    if (big >= kBufBytes || lat >= kBufBytes || (long long)d->B * 4 * ((d->H + 3) / 4) * 4 * ((d->W + 3) / 4) *
                                                     (d->M * 3 / 2) * 4 >= kBufBytes)
        return fail(WF_E_UNSUPPORTED, "transform activations exceed the 2 GiB buffer window");
    Xform* x = new (std::nothrow) Xform();
    if (!x) return fail(WF_E_NOMEM, "host allocation");
    x->N = d->N; x->M = d->M; x->B = d->B; x->H = d->H; x->W = d->W;
    x->Hz = (d->H + 3) / 4; x->Wz = (d->W + 3) / 4; x->precision = d->precision;
    hipError_t e = hipGetDevice(&x->device);
    int rc = e == hipSuccess ? WF_OK : xf_fail_hip(e, "hipGetDevice");
    const int N = d->N, M = d->M, C = M * 3 / 2;
    if (rc == WF_OK) rc = xf_deconv(x, x->hs[0], d->hs_w[0], d->hs_b[0], N, M, 1);
    if (rc == WF_OK) rc = xf_deconv(x, x->hs[1], d->hs_w[1], d->hs_b[1], M, C, 1);
    if (rc == WF_OK) rc = xf_conv3(x, x->hs[2], d->hs_w[2], d->hs_b[2], C, 2 * M);
    const int gi[4] = {M, N, N, N}, go[4] = {N, N, N, 3};
    for (int k = 0; k < 4 && rc == WF_OK; ++k) {
        rc = go[k] <= 4 ? xf_synth_deconv4(x, x->gs[k], d->gs_w[k], d->gs_b[k], gi[k], go[k])
                        : xf_synth_deconv(x, x->gs[k], d->gs_w[k], d->gs_b[k], gi[k], go[k]);
        if (rc == WF_OK && k < 3) rc = xf_synth_gdn(x, x->gdn[k], d->gdn_beta[k], d->gdn_gamma[k], N);
    }
    const size_t B = d->B;
    if (rc == WF_OK) rc = xf_alloc(x, &x->hs_a, B * 2 * x->Hz * 2 * x->Wz * M);
    if (rc == WF_OK) rc = xf_alloc(x, &x->hs_b, B * 4 * x->Hz * 4 * x->Wz * C);
    if (rc == WF_OK) rc = xf_alloc(x, &x->g_a, B * 8 * d->H * 8 * d->W * N);
    if (rc == WF_OK) rc = xf_alloc(x, &x->g_b, B * 8 * d->H * 8 * d->W * N);
    if (rc != WF_OK) {
        free_xform(x);
        return rc;
    }
    *out = reinterpret_cast<wf_xform_t>(x);
    return WF_OK;
}

int wf_hyper_synthesis(wf_xform_t plan, const float* z_hat, float* psi, hipStream_t stream) {
    if (!plan || !z_hat || !psi) return fail(WF_E_INVALID, "plan, z_hat or psi is NULL");
    const Xform& x = *reinterpret_cast<Xform*>(plan);
    if (x.precision == WF_BF16) hyper<PBF16>(x, z_hat, psi, stream);
    else hyper<PF32>(x, z_hat, psi, stream);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? WF_OK : xf_fail_hip(e, "transform launch");
}

int wf_synthesis(wf_xform_t plan, const float* y_hat, float* image, hipStream_t stream) {
    if (!plan || !y_hat || !image) return fail(WF_E_INVALID, "plan, y_hat or image is NULL");
    const Xform& x = *reinterpret_cast<Xform*>(plan);
    if (x.precision == WF_BF16) synth<SBF16>(x, y_hat, image, stream);
    else synth<SF32>(x, y_hat, image, stream);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? WF_OK : xf_fail_hip(e, "transform launch");
}

void wf_xform_destroy(wf_xform_t plan) { free_xform(reinterpret_cast<Xform*>(plan)); }

}  // extern "C"
