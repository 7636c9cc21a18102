// risk.hip -- the risk-set sums of one ISTA step as five launches, one per
// phase, or one for few subjects (the phases themselves are in risk_dev.h).
#include "risk_dev.h"

namespace cox {
namespace {

using namespace riskdev;

__global__ __launch_bounds__(kT) void risk_eta_kernel(RiskArgs a)
{
    __shared__ double sh[kNW];
    risk_eta_blk(a, blockIdx.x, blockIdx.y, sh);
}

__global__ __launch_bounds__(kT) void risk_scan_w_kernel(RiskArgs a)
{
    __shared__ double sh[kNW];
    risk_scan_w_blk(a, blockIdx.x, blockIdx.y, sh);
}

__global__ __launch_bounds__(kT) void risk_scan_q_kernel(RiskArgs a)
{
    __shared__ double sh[kNW];
    __shared__ double pre[kMaxTiles];
    risk_scan_q_blk(a, blockIdx.x, blockIdx.y, sh, pre);
}

__global__ __launch_bounds__(kT) void risk_resid_kernel(RiskArgs a)
{
    __shared__ double sh[kNW];
    __shared__ double suf[kMaxTiles];
    risk_resid_blk(a, blockIdx.x, blockIdx.y, sh, suf);
}

__global__ __launch_bounds__(kT) void risk_finish_kernel(RiskArgs a)
{
    __shared__ double sh[kNW];
    risk_finish_blk(a, blockIdx.x, sh);
}

// All five phases of one b in one workgroup, for at most kSide tiles: the kT
// threads of group g take tile g as the phases' workgroup g does, so every sum
// has the same terms in the same order and the results are the same, bit for bit.
// eta, w, S and T stay in LDS and the time order is loaded up front, so that the
// phases wait for barriers, not for memory: 17 us a step at n = 1,000, where five
// launches, at least 3 us each however little they do, took 22.
constexpr int kSide = 4;
constexpr int kSmallN = kSide * kSub;  // 4,096 subjects
__global__ __launch_bounds__(kSide* kT) void risk_small_kernel(RiskArgs a)
{
    __shared__ double se[kSmallN], sw[kSmallN], sS[kSmallN], sT[kSmallN];
    __shared__ double sh[kSide][kNW], off[kSide][kSide], tot[kSide], Lp[kSide], rp[kSide];
    const int b = blockIdx.x, g = threadIdx.x / kT, t = tid();
    if (skip_b(a, b)) return;
    const int n = (int)a.n;
    const int64_t bo = (int64_t)b * n;
    const int t0 = g * kSub, t1 = min(n, t0 + kSub), len = t1 - t0;  // len <= 0: no such tile
    // the time order at this thread's positions of each phase: t0 + 4 t + e (w), the tile's end - 4 t - e (q),
    // t0 + t + kT e (residual)
    int pw[4], gq[4], gr[4], pr[4];
    bool eq[4], er[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int kw = t0 + 4 * t + e, kq = t1 - 1 - 4 * t - e, kr = t0 + t + kT * e;
        pw[e] = kw < t1 ? a.ord.perm[kw] : 0;
        const bool q = 4 * t + e < len, r = kr < t1;
        eq[e] = q && a.ord.ev[kq];
        gq[e] = q ? a.ord.gend[kq] : 0;
        er[e] = r && a.ord.ev[kr];
        gr[e] = r ? a.ord.gstart[kr] : 0;
        pr[e] = r ? a.ord.perm[kr] : 0;
    }
    const bool addp = a.part != nullptr && *a.nsel > 0;
    const bool copy = addp || a.eta_in_f32 || a.eta_in != a.eta;
    double m = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = threadIdx.x + kSide * kT * e;
        if (i >= n) break;
        double v = a.eta_in_f32 ? (double)static_cast<const float*>(a.eta_in)[bo + i]
                                : static_cast<const double*>(a.eta_in)[bo + i];
        if (addp) {
#pragma unroll 8
            for (int c = 0; c < a.ncg; ++c) v += a.part[(int64_t)c * a.part_cstride + bo + i];
        }
        if (copy) a.eta[bo + i] = v;
        se[i] = v;
        m = fmax(m, v);
    }
    m = block_max(m, sh[g]);
    if (t == 0) tot[g] = m;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSide; ++q) m = fmax(m, tot[q]);
    // w and its cumulative sum within the tile
    double v[4], es[4], ts = 0.0, sum;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        es[e] = se[pw[e]];
        v[e] = t0 + 4 * t + e < t1 ? exp(es[e] - m) : 0.0;
        ts += v[e];
    }
    double run = block_excl_scan(ts, sh[g], &sum);  // every thread has read se by the first barrier in it
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = t0 + 4 * t + e;
        run += v[e];
        if (k < t1) {
            se[k] = es[e];  // from here in time order
            sw[k] = v[e];
            sS[k] = run;
            a.w[bo + k] = v[e];
        }
    }
    if (t == 0) tot[g] = sum;
    __syncthreads();
    block_offsets(tot, a.ntile, false, off[g], sh[g]);
    // W at the end of the tie group, the log-likelihood terms, the reverse cumulative sum of delta / W
    double Lacc = 0.0;
    ts = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = 0.0;
        if (eq[e]) {
            const double W = sS[gq[e]] + off[g][gq[e] / kSub];
            v[e] = 1.0 / W;
            Lacc += se[t1 - 1 - 4 * t - e] - m - log(W);
        }
        ts += v[e];
    }
    run = block_excl_scan(ts, sh[g], &sum);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        run += v[e];
        if (4 * t + e < len) sT[t1 - 1 - 4 * t - e] = run;
    }
    Lacc = block_sum(Lacc, sh[g]);
    if (t == 0) {
        tot[g] = sum;
        Lp[g] = Lacc;
        a.mshift[b] = m;
    }
    __syncthreads();
    block_offsets(tot, a.ntile, true, off[g], sh[g]);
    // c at the start of the tie group, the residual
    double sr = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = t0 + t + kT * e;
        if (k >= t1) break;
        const double c = sT[gr[e]] + off[g][gr[e] / kSub];
        const double r = (er[e] ? 1.0 : 0.0) - sw[k] * c;
        if (a.r32) {
            const float rf = (float)r;
            a.r32[(int64_t)b * a.rstride + pr[e]] = rf;
            sr += (double)rf;
        } else {
            sr += r;
        }
        if (a.r64) a.r64[bo + pr[e]] = r;
    }
    sr = block_sum(sr, sh[g]);
    if (t == 0) rp[g] = sr;
    __syncthreads();
    if (g > 0) return;  // the barriers below are this group's alone
    RiskArgs f = a;
    f.Lpart = Lp - (int64_t)b * a.ntile;
    f.rpart = rp - (int64_t)b * a.ntile;
    risk_finish_blk(f, b, sh[0]);
}

}  // namespace

hipError_t launch_risk(const RiskArgs& a, hipStream_t s)
{
    if (a.bpad) return launch_risk_rows(a, s);
    if (a.ntile > kMaxTiles || a.ntile < 1 || a.nfin < 1) return hipErrorInvalidValue;
    if (a.ntile <= kSide && a.tile == kSub) {
        hipLaunchKernelGGL(risk_small_kernel, dim3(a.B), dim3(kSide * kT), 0, s, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(risk_eta_kernel, dim3(a.nfin, a.B), dim3(kT), 0, s, a);
    hipLaunchKernelGGL(risk_scan_w_kernel, dim3(a.ntile, a.B), dim3(kT), 0, s, a);
    hipLaunchKernelGGL(risk_scan_q_kernel, dim3(a.ntile, a.B), dim3(kT), 0, s, a);
    hipLaunchKernelGGL(risk_resid_kernel, dim3(a.ntile, a.B), dim3(kT), 0, s, a);
    hipLaunchKernelGGL(risk_finish_kernel, dim3(a.B), dim3(kT), 0, s, a);
    return hipGetLastError();
}

}  // namespace cox
