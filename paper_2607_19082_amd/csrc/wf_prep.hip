// What a call of the resident driver needs before its launch of k_resident
// (in a file of its own: the code of the roles then lies in memory as it was
// measured; with these kernels beside them the 1080p mixture decode, whose
// roles are the largest, took 5.38 ms instead of 5.29).
#include <algorithm>

#include "wf_split.h"

namespace wf {

static int ceil_div(int a, int b) { return (a + b - 1) / b; }

// One launch: the call's pointers, the counters at zero, fp32: h1 and h2 at
// the fill pattern that their readers check for, and (k_res_prep) the hoisted
// layer-1 part of every latent.
struct ResPrep {
    CallPtrs* dst;
    CallPtrs v;
    unsigned* cnt;            // ncnt counters, kResSlotWords words apart
    size_t ncnt;
    uint4 *h1, *h2;           // n1 and n2 16-byte words
    size_t n1, n2;
};
__device__ __forceinline__ void res_prep(const ResPrep& p, int b, int nb) {
    if (b == 0 && threadIdx.x == 0) *p.dst = p.v;
    const size_t i0 = (size_t)b * blockDim.x + threadIdx.x, st = (size_t)nb * blockDim.x;
    for (size_t i = i0; i < p.ncnt; i += st) p.cnt[i * kResSlotWords] = 0;
    const uint4 f{kResFill, kResFill, kResFill, kResFill};
    for (size_t i = i0; i < p.n1; i += st) p.h1[i] = f;
    for (size_t i = i0; i < p.n2; i += st) p.h2[i] = f;
}
__global__ __launch_bounds__(kThreads) void k_res_init(ResPrep p) { res_prep(p, blockIdx.x, gridDim.x); }

// The same in the first `np` workgroups, and the hoisted part
// P1 = b_hoist + W1[:, :2M] . psi in the others, as a product of f16 pairs
// (wf_split.h).  The fill is bound by memory and the product by the matrix
// cores, so they run side by side.  From the call's first launch to
// k_resident, before (fp32 MFMA, five launches) and now: 4K 680 us (the hoist
// 609) and 235, 16x16 88 us (the hoist 58 on 16 workgroups) and 26, of which
// 11 are the cooperative launch's own.
template <int RT, int CT>
__global__ __launch_bounds__(kThreads, 2) void k_res_prep(ResPrep p, SynthArgs a, int np) {
    if ((int)blockIdx.x < np) {
        res_prep(p, blockIdx.x, np);
        return;
    }
    synth_tile<SF16, XM_GEMM, RT, CT, 4, false>(a, blockIdx.x - np);
}

template <class T>
static int prep_alloc(Plan& p, T** dst, const std::vector<T>& v) {
    hipError_t e = hipMalloc((void**)dst, v.size() * sizeof(T));
    if (e != hipSuccess) return fail(WF_E_NOMEM, std::string("resident driver weights: ") + hipGetErrorString(e));
    p.owned.push_back((void*)*dst);
    e = hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
    return e == hipSuccess ? WF_OK : fail(WF_E_HIP, std::string("hipMemcpy: ") + hipGetErrorString(e));
}

int build_resident_prep(Plan& p, const float* w1) {
    if (p.precision == WF_BF16) return WF_OK;
    // the hoisted part's weights as f16 pairs
    const int M = p.M;
    std::vector<int> ce;
    std::vector<uint16_t> v[4];
    p.force_split = pack_split(false, 1, 2 * M, p.d1, p.Np1, [](int, int& nkx) { return nkx = 1; },
                               [&](int, int, int, int k, int n) { return w1[(size_t)n * 4 * M + k]; }, ce, v);
    uint16_t* wp = nullptr;
    int* dce = nullptr;
    int rc = prep_alloc(p, &wp, v[0]);
    if (rc == WF_OK) rc = prep_alloc(p, &dce, ce);
    p.wp_split = wp;
    p.ce_split = dce;
    return rc;
}

template <int RT, int CT>
static void launch_prep(const ResPrep& q, SynthArgs a, int np, hipStream_t stream) {
    using S = SynthShape<XM_GEMM, RT, CT, 4>;
    a.twl = RT == 1 ? 4 : (RT == 4 ? 6 : 7);
    a.ntx = ceil_div(a.Wi, S::kPx);
    a.nty = 1;
    a.ncb = ceil_div(a.Cop, S::kCols);
    const int nh = kXcds * ceil_div(a.ntx, kXcds) * a.ncb;
    hipLaunchKernelGGL((k_res_prep<RT, CT>), dim3(np + nh), dim3(kThreads), 0, stream, q, a, np);
}

int enqueue_resident_prep(Plan& p, const CallPtrs& c, hipStream_t stream) {
    const ResArgs& r = p.res;
    ResPrep q{};
    q.dst = p.d_call;
    q.v = c;
    q.cnt = r.cnt;
    q.ncnt = (size_t)(r.hoist ? kResRoles : RR_H) * r.ntasks * kXcds;   // (the last role's are the hoist's)
    if (p.precision != WF_BF16) {
        q.h1 = static_cast<uint4*>(r.h1);
        q.h2 = static_cast<uint4*>(r.h2);
        q.n1 = (size_t)r.ntasks * kTile * p.Np1 / 4;
        q.n2 = (size_t)r.ntasks * kTile * p.Np2 / 4;
    }
    // workgroups for the fills: every thread a few 16-byte words, at most half of the chip's slots
    const size_t words = q.ncnt + q.n1 + q.n2;
    const int np = kXcds * (int)std::min<size_t>(32, 1 + words / (kXcds * kThreads * 4));
    if (p.precision == WF_BF16) {
        hipLaunchKernelGGL(k_res_init, dim3(4 * np), dim3(kThreads), 0, stream, q);
        if (!r.hoist) {
            int rc = enqueue_hoist(p, stream);
            if (rc != WF_OK) return rc;
        }
    } else {
        SynthArgs a{};
        a.in = c.psi; a.out = p.args.p1; a.wp[0] = p.wp_split; a.ce = p.ce_split; a.bias = p.args.b_hoist;
        a.force_f32 = p.force_split;
        a.B = a.Hi = a.Ho = a.ncls = 1;
        a.Wi = a.Wo = p.B * p.H * p.W;
        a.Ci = 2 * p.M; a.nch = ceil_div(a.Ci, 32); a.Co = a.Cop = p.Np1;
        // 128 latents x 192 columns where that gives every compute unit work, else smaller tiles
        if ((long long)a.Wi * a.Cop >= 256LL * 128 * 192) launch_prep<8, 3>(q, a, np, stream);
        else if ((long long)a.Wi * a.Cop >= 256LL * 64 * 64) launch_prep<4, 1>(q, a, np, stream);
        else launch_prep<1, 1>(q, a, np, stream);
    }
    return WF_OK;
}

}  // namespace wf
