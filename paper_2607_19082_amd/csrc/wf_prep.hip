// What a call of the resident driver needs before its launch of k_resident.
#include <algorithm>

#include "wf_conv.h"

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
// P1 = b_hoist + W1[:, :2M] . psi in the others (wf_conv.h: each sum in the
// order of the other drivers' hoist, so a latent's bits depend neither on the
// grid nor on the latents beside it).  The fill is bound by memory and the
// product by the matrix cores, so they run side by side: 455 us at 4K (fp32
// MFMA: 44.5 GFLOP, 97 TFLOP/s with the fill's 0.3 GB beside them), where five
// launches took 680, the hoist 609 of it.
template <int RT>
__global__ __launch_bounds__(kThreads, 2) void k_res_prep(ResPrep p, ConvArgs a, int np) {
    if ((int)blockIdx.x < np) {
        res_prep(p, blockIdx.x, np);
        return;
    }
    conv_tile<PF32, XM_GEMM, RT, 1, 4>(a, blockIdx.x - np, 0);
}

template <int RT>
static void launch_prep(const ResPrep& q, ConvArgs a, int np, hipStream_t stream) {
    using S = ConvShape<RT, 1, 4>;
    a.nrb = ceil_div(a.Wq, S::kPx);
    a.ncb = ceil_div(a.Cop, S::kCols);
    const int nh = kXcds * ceil_div(a.nrb, kXcds) * a.ncb;
    hipLaunchKernelGGL(k_res_prep<RT>, dim3(np + nh), dim3(kThreads), 0, stream, q, a, np);
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
        ConvArgs a{};
        a.in = c.psi; a.out = p.args.p1; a.wp[0] = p.args.wp_hoist; a.bias = p.args.b_hoist;
        a.B = a.Hi = a.Hq = a.Ho = 1;
        a.Wi = a.Wq = a.Wo = p.B * p.H * p.W;
        a.Ci = 2 * p.M; a.Co = a.Cop = p.Np1;
        // Latents of a workgroup (16 RT, by 64 columns) by the size of the
        // product, so that small grids still spread over the chip.  us per
        // decode with 16 / 32 / 64 / 128: 16x16 (0.16 M outputs) 599 / 603 /
        // 606 / 616, 48x32 (0.98 M) 1343 / 1341 / 1343 / 1348, 80x48 (2.5 M)
        // 2124 / 2118 / 2120 / 2128, 120x68 mixture (5.2 M) 4766 / 4762 /
        // 4751 / 4752, 4K (34.7 M) 9678 / 9614 / 9536 / 9522.  (4K with 128
        // columns: 9523 with 128 latents, 9563 with 64.)
        const long long outputs = (long long)a.Wq * a.Cop;
        if (outputs < 500000) launch_prep<1>(q, a, np, stream);
        else if (outputs < 4000000) launch_prep<2>(q, a, np, stream);
        else launch_prep<8>(q, a, np, stream);
    }
    return WF_OK;
}

}  // namespace wf
