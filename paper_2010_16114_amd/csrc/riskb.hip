// riskb.hip -- the risk-set sums of one batched ISTA step (B > 8 lambdas over
// allele counts), and the quantisation of its residuals.
//
// The quantities are those of risk_dev.h.  Here eta, w and r are stored in
// rows, [subject or position][bpad] with bpad = B rounded up to 16: the gather of
// eta and the scatter of r through the time order move whole 128- to 512-byte
// rows (in [B][n] every 8-byte value cost a cache line of its own), and 16
// adjacent lanes hold 16 adjacent vectors, so every running sum is one lane's
// serial sum and no lane waits for another.
//
// A unit of 16 lanes takes one b group of 16 vectors over one tile of a.tile
// consecutive sorted positions; a workgroup's kUnits units are `tpw` consecutive
// tiles of all groups.  Event groups are the tie groups with events, in time
// order, a.egrank[k] of them ending before position k.  Four passes:
//   max    m_b = max_i eta_bi, by atomic maxima of order-preserving keys (exact,
//          so the order of arrival does not matter)
//   w      w_k = exp(eta - m) and its running sum in the tile; the sum at each
//          event group's last position to sg[group] (the whole tie group is at
//          risk, Breslow); tile and workgroup totals; sum of delta (eta - m)
//   q      W = sg + the totals before the tile; q_g = d_g / W for the group's
//          d_g events, in place of sg; L terms d_g log W; totals of q
//   r      positions in descending order: c grows by q_g at each event group's
//          last position, so that every member of the group sees it; r =
//          delta - w c to subject order, and max |r| by atomic maxima
// then the fixed-order sums of the L terms with the stopping rule.  Every sum
// has a fixed order: results are reproducible bit for bit.
//
// It is bound by memory: eta read twice, w written and read, r written, and
// two reads and writes of a row per event group: about 1.2 GB at 400,000
// subjects, 64 vectors and 20% events.  The passes take 33, 90, 41 and 109 us
// there (4.2 GB/ms; a large copy 4.9); in [B][n] with the vector form's kernels
// it was 1,204 us, and quantising r 175 us (65 now).
#include "risk_dev.h"

#include "mfma.h"

namespace cox {
namespace {

constexpr int kBT = 512;            // threads per workgroup
constexpr int kUnits = kBT / 16;    // 16-lane units per workgroup
constexpr int kWgs = 512;           // workgroups a pass is spread over (two per compute unit)
constexpr int kMinTile = 8;
constexpr int kPf = 8;              // rows in flight per unit
// Copies of every atomically updated key or sum, one per workgroup modulo
// kKeySets: updates of one address follow each other at about 50 ns, so 512
// workgroups on one set of keys took 26 us.
static_assert(kKeySets * kKeyRow == kBT, "one thread clears each key");

// Order-preserving keys of doubles: larger value, larger key; 0 is below all.
__device__ __forceinline__ unsigned long long key_of(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    return (u >> 63) ? ~u : u | (1ull << 63);
}
__device__ __forceinline__ double of_key(unsigned long long k)
{
    return __longlong_as_double((long long)((k >> 63) ? k & ~(1ull << 63) : ~k));
}

// The largest of b's keys over the sets.
__device__ __forceinline__ unsigned long long top_key(const unsigned long long* __restrict__ keys, int b)
{
    unsigned long long k = 0;
#pragma unroll
    for (int q = 0; q < kKeySets; ++q) k = max(k, keys[q * kKeyRow + b]);
    return k;
}

// A unit's place: its vector b, its tile of the workgroup, its positions [t0, t1).
struct Unit {
    int b, tl;        // vector of this lane; tile within the workgroup
    int64_t t0, t1;   // sorted positions
    bool on;          // a live vector over a non-empty tile
};

__device__ __forceinline__ Unit unit_of(const RiskArgs& a)
{
    const int ng = a.bpad / 16, tpw = kUnits / ng;
    const int u = threadIdx.x / 16;
    Unit x;
    x.tl = u / ng;
    x.b = (u % ng) * 16 + (threadIdx.x & 15);
    x.t0 = ((int64_t)blockIdx.x * tpw + x.tl) * a.tile;
    x.t1 = min(a.n, x.t0 + a.tile);
    x.on = x.tl < tpw && x.t0 < a.n && x.b < a.B && !riskdev::skip_b(a, x.b);
    return x;
}

// sum_{w < blockIdx.x} (or, reverse, > blockIdx.x) of tot[w][b] for every b, into
// out[b]: kBT / bpad slices of the workgroups, added in slice order.
__device__ void outer_sum(const double* __restrict__ tot, int bpad, bool reverse, double* slice, double* out)
{
    const int ns = kBT / bpad, s = threadIdx.x / bpad, b = threadIdx.x % bpad;
    const int lo = reverse ? blockIdx.x + 1 : 0, hi = reverse ? gridDim.x : blockIdx.x;
    const int per = (hi - lo + ns - 1) / ns;
    if (s < ns) {
        const int w0 = lo + s * per, w1 = min(hi, w0 + per);
        double v = 0.0;
#pragma unroll 8
        for (int w = w0; w < w1; ++w) v += tot[(int64_t)w * bpad + b];
        slice[s * bpad + b] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < bpad) {
        double v = 0.0;
        for (int q = 0; q < ns; ++q) v += slice[q * bpad + threadIdx.x];
        out[threadIdx.x] = v;
    }
    __syncthreads();
}

__global__ __launch_bounds__(kBT) void riskb_max_kernel(RiskArgs a)
{
    __shared__ double sh[kBT];
    const int rows = kBT / a.bpad, s = threadIdx.x / a.bpad, b = threadIdx.x % a.bpad;
    const bool on = s < rows && b < a.B && !riskdev::skip_b(a, b);
    double m = -INFINITY;
    if (on) {
        const int64_t step = (int64_t)gridDim.x * rows;
        const double* __restrict__ eta = a.eta + b;
#pragma unroll 4
        for (int64_t i = (int64_t)blockIdx.x * rows + s; i < a.n; i += step) m = fmax(m, eta[i * a.bpad]);
    }
    sh[threadIdx.x] = m;
    __syncthreads();
    if (s == 0 && on) {
        for (int q = 1; q < rows; ++q) m = fmax(m, sh[q * a.bpad + b]);
        atomicMax(&a.mkey[(blockIdx.x % kKeySets) * kKeyRow + b], key_of(m));
    }
}

// A tile's w and the tiles' and workgroups' L terms are added with their rounding
// errors kept (Knuth's TwoSum: t + err = hi + v exactly), and the objective adds lambda |beta|_1 before its last
// rounding.  Near the top of a path the w of a step are a few values just below 1,
// whose additions all round the same way, and -L and the penalty change by 1e3 units
// in the last place of L, their sum by none: with plain sums the objective of the
// first step at 400,000 x 500,000 came out one unit above the start's.  The adds hide
// behind the loads.
__device__ __forceinline__ void add2(double& hi, double& lo, double v, double vlo)
{
    const double t = hi + v, z = t - hi;
    lo += (hi - (t - z)) + (v - z) + vlo;
    hi = t;
}

__global__ __launch_bounds__(kBT) void riskb_w_kernel(RiskArgs a)
{
    __shared__ double st[kUnits * 16], sl[kUnits * 16];
    const Unit x = unit_of(a);
    const int bpad = a.bpad;
    if (blockIdx.x == 0) a.rkey[threadIdx.x] = 0;  // for the r pass of this step
    double run = 0.0, rlo = 0.0, l1 = 0.0;
    if (x.on) {
        const double m = of_key(top_key(a.mkey, x.b));
        const int32_t* __restrict__ perm = a.ord.perm;
        const int32_t* __restrict__ rank = a.egrank;
        const uint8_t* __restrict__ ev = a.ord.ev;
        const double* __restrict__ eta = a.eta + x.b;
        double* __restrict__ w = a.w + x.b;
        double* __restrict__ sg = a.S + x.b;
        int32_t g = rank[x.t0];
        for (int64_t k0 = x.t0; k0 < x.t1; k0 += kPf) {
            double e[kPf];
            int32_t rk[kPf];
            uint8_t d[kPf];
#pragma unroll
            for (int q = 0; q < kPf; ++q) {
                const int64_t k = min(k0 + q, x.t1 - 1);
                e[q] = eta[(int64_t)perm[k] * bpad];
                rk[q] = rank[k + 1];
                d[q] = ev[k];
            }
#pragma unroll
            for (int q = 0; q < kPf; ++q) {
                if (k0 + q >= x.t1) break;
                const double v = e[q] - m, wk = exp(v);
                add2(run, rlo, wk, 0.0);
                if (d[q]) l1 += v;
                w[(k0 + q) * bpad] = wk;
                if (rk[q] != g) {  // an event group ends here
                    sg[(int64_t)g * bpad] = run + rlo;
                    g = rk[q];
                }
            }
        }
    }
    const int ng = bpad / 16, tpw = kUnits / ng;
    if (x.tl < tpw) {
        run += rlo;
        st[x.tl * bpad + x.b] = run;
        sl[x.tl * bpad + x.b] = l1;
        a.stot[((int64_t)blockIdx.x * tpw + x.tl) * bpad + x.b] = run;
    }
    __syncthreads();
    if ((int)threadIdx.x < bpad) {
        double s = 0.0, l = 0.0;
        for (int t = 0; t < tpw; ++t) {
            s += st[t * bpad + threadIdx.x];
            l += sl[t * bpad + threadIdx.x];
        }
        a.wgS[(int64_t)blockIdx.x * bpad + threadIdx.x] = s;
        a.Lpart[(int64_t)blockIdx.x * bpad + threadIdx.x] = l;
    }
}

__global__ __launch_bounds__(kBT) void riskb_q_kernel(RiskArgs a)
{
    __shared__ double slice[kBT], off[64], sq[kUnits * 16], sl[kUnits * 16];
    const Unit x = unit_of(a);
    const int bpad = a.bpad, ng = bpad / 16, tpw = kUnits / ng;
    if (blockIdx.x == 0) a.mkey[threadIdx.x] = 0;  // for the next step's maxima
    outer_sum(a.wgS, bpad, false, slice, off);
    double q = 0.0, l = 0.0;
    if (x.on) {
        double before = 0.0;
        for (int t = 0; t < x.tl; ++t) before += a.stot[((int64_t)blockIdx.x * tpw + t) * bpad + x.b];
        before += off[x.b];
        double* __restrict__ sg = a.S + x.b;
        const int32_t* __restrict__ cnt = a.egcnt;
        const int32_t g1 = a.egrank[x.t1];
        for (int32_t g0 = a.egrank[x.t0]; g0 < g1; g0 += kPf) {
            double s[kPf];
            int32_t d[kPf];
#pragma unroll
            for (int u = 0; u < kPf; ++u) {
                const int32_t g = min(g0 + u, g1 - 1);
                s[u] = sg[(int64_t)g * bpad];
                d[u] = cnt[g];
            }
#pragma unroll
            for (int u = 0; u < kPf; ++u) {
                if (g0 + u >= g1) break;
                const double W = s[u] + before, dg = (double)d[u], qg = dg / W;
                l += dg * log(W);
                q += qg;
                sg[(int64_t)(g0 + u) * bpad] = qg;
            }
        }
    }
    if (x.tl < tpw) {
        sq[x.tl * bpad + x.b] = q;
        sl[x.tl * bpad + x.b] = l;
        a.qtot[((int64_t)blockIdx.x * tpw + x.tl) * bpad + x.b] = q;
    }
    __syncthreads();
    if ((int)threadIdx.x < bpad) {
        double s = 0.0, t = 0.0, lo = 0.0;
        for (int u = 0; u < tpw; ++u) {
            s += sq[u * bpad + threadIdx.x];
            add2(t, lo, sl[u * bpad + threadIdx.x], 0.0);
        }
        if (isfinite(t)) t += lo;
        a.wgQ[(int64_t)blockIdx.x * bpad + threadIdx.x] = s;
        a.Lpart[(int64_t)blockIdx.x * bpad + threadIdx.x] -= t;
    }
}

__global__ __launch_bounds__(kBT) void riskb_r_kernel(RiskArgs a)
{
    __shared__ double slice[kBT], off[64], sm[kUnits * 16];
    const Unit x = unit_of(a);
    const int bpad = a.bpad, ng = bpad / 16, tpw = kUnits / ng;
    outer_sum(a.wgQ, bpad, true, slice, off);
    double rm = 0.0;
    if (x.on) {
        double c = off[x.b];
        for (int t = tpw - 1; t > x.tl; --t) c += a.qtot[((int64_t)blockIdx.x * tpw + t) * bpad + x.b];
        const int32_t* __restrict__ perm = a.ord.perm;
        const int32_t* __restrict__ rank = a.egrank;
        const uint8_t* __restrict__ ev = a.ord.ev;
        const double* __restrict__ w = a.w + x.b;
        const double* __restrict__ qg = a.S + x.b;
        double* __restrict__ r = a.r64 + x.b;
        int32_t g = rank[x.t1];  // event groups that end before the position above
        for (int64_t k1 = x.t1; k1 > x.t0; k1 -= kPf) {
            double wk[kPf], qk[kPf];
            int32_t at[kPf];
            uint8_t d[kPf];
            int32_t gq = g;
#pragma unroll
            for (int q = 0; q < kPf; ++q) {
                const int64_t k = max(k1 - 1 - q, x.t0);
                wk[q] = w[k * bpad];
                at[q] = perm[k];
                d[q] = ev[k];
                const int32_t rk = rank[k];
                qk[q] = rk != gq ? qg[(int64_t)rk * bpad] : 0.0;  // rk = gq - 1: a group ends at k
                gq = rk;
            }
            g = gq;
#pragma unroll
            for (int q = 0; q < kPf; ++q) {
                if (k1 - 1 - q < x.t0) break;
                c += qk[q];
                const double v = (d[q] ? 1.0 : 0.0) - wk[q] * c;
                rm = fmax(rm, fabs(v));
                r[(int64_t)at[q] * bpad] = v;
            }
        }
    }
    if (x.tl < tpw) sm[x.tl * bpad + x.b] = rm;
    __syncthreads();
    if ((int)threadIdx.x < bpad) {
        double m = 0.0;
        for (int t = 0; t < tpw; ++t) m = fmax(m, sm[t * bpad + threadIdx.x]);
        if (m > 0.0) atomicMax(&a.rkey[(blockIdx.x % kKeySets) * kKeyRow + threadIdx.x], key_of(m));
    }
}

__global__ __launch_bounds__(riskdev::kT) void riskb_finish_kernel(RiskArgs a)
{
    __shared__ double sh[riskdev::kNW], sl[riskdev::kNW];
    const int b = blockIdx.x;
    if (riskdev::skip_b(a, b)) return;
    double L = 0.0, lo = 0.0;
    for (int q = threadIdx.x; q < a.ntile; q += riskdev::kT) add2(L, lo, a.Lpart[(int64_t)q * a.bpad + b], 0.0);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) add2(L, lo, __shfl_xor(L, o, kWave), __shfl_xor(lo, o, kWave));
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    if (lane == 0) sh[wid] = L, sl[wid] = lo;
    __syncthreads();
    L = 0.0, lo = 0.0;
#pragma unroll
    for (int q = 0; q < riskdev::kNW; ++q) add2(L, lo, sh[q], sl[q]);
    __syncthreads();
    if (!isfinite(L)) lo = 0.0;
    if (threadIdx.x == 0) a.L[b] = L + lo;
    if (a.use_ctl) riskdev::stop_rule(a, b, L, sh, lo);
}

// The residual limbs of 16 subjects and one vector per thread, 16 adjacent lanes
// for 16 adjacent vectors: rows of r in, one 16-byte run of each limb out (limb
// layout and rounding as described in mfma.hip).  The exact sums of R arrive by
// integer atomics; the last workgroup to finish writes sumr_b = q_b sum_i R_bi
// and clears the sums for the next launch.  Few, large workgroups: each counts
// itself on one address (at 400,000 x 64: 153 us with 2,048 workgroups of 256
// threads, 101 with 1,024).
constexpr int kQT = 1024;
__global__ __launch_bounds__(kQT) void quantize_rows_kernel(const double* __restrict__ r, int64_t n, int B,
                                                            const unsigned long long* __restrict__ rkey,
                                                            int8_t* __restrict__ limbs, int bpad, int nlimb,
                                                            double* __restrict__ qscale,
                                                            unsigned long long* __restrict__ rsum,
                                                            unsigned* __restrict__ done, double* __restrict__ sumr)
{
    __shared__ long long sh[kQT];
    __shared__ int last;
    const int per = kQT / bpad, s = threadIdx.x / bpad, b = threadIdx.x % bpad;
    const int64_t nchunk = (n + 255) / 256 * 16;  // chunks of 16 subjects, up to round_up(n, 256)
    const bool on = s < per && b < B;
    long long sum = 0;
    double q = 1.0;
    if (on) {
        const unsigned long long key = top_key(rkey, b);
        const double mx = key ? of_key(key) : 0.0;
        q = mx > 0.0 ? mx / (double)(1 << (nlimb == 2 ? 14 : 22)) : 1.0;
        if (blockIdx.x == 0 && s == 0) qscale[b] = q;
        for (int64_t c = (int64_t)blockIdx.x * per + s; c < nchunk; c += (int64_t)gridDim.x * per) {
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = c * 16 + e < n ? r[(c * 16 + e) * bpad + b] : 0.0;
            uint32_t o0[4] = {}, o1[4] = {}, o2[4] = {};
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int R = (int)llrint(v[e] / q);
                const int d0 = ((R + 128) & 255) - 128;
                const int R1 = (R - d0) >> 8;
                const int sft = 8 * (e & 3);
                o0[e >> 2] |= (uint32_t)(d0 & 255) << sft;
                if (nlimb == 2) {
                    o1[e >> 2] |= (uint32_t)(R1 & 255) << sft;  // |R1| <= 64 when |R| <= 2^14
                } else {
                    const int d1 = ((R1 + 128) & 255) - 128;
                    o1[e >> 2] |= (uint32_t)(d1 & 255) << sft;
                    o2[e >> 2] |= (uint32_t)(((R1 - d1) >> 8) & 255) << sft;
                }
                sum += R;
            }
            uint4* dst = reinterpret_cast<uint4*>(limbs + (c * (nlimb * bpad) + b) * 16);
            dst[0] = make_uint4(o0[0], o0[1], o0[2], o0[3]);
            dst[bpad] = make_uint4(o1[0], o1[1], o1[2], o1[3]);
            if (nlimb == 3) dst[2 * bpad] = make_uint4(o2[0], o2[1], o2[2], o2[3]);
        }
    }
    sh[threadIdx.x] = sum;
    __syncthreads();
    if (s == 0 && on) {
        for (int u = 1; u < per; ++u) sum += sh[u * bpad + b];
        atomicAdd(&rsum[(blockIdx.x % kKeySets) * kKeyRow + b], (unsigned long long)sum);
        __threadfence();  // the sums are in before this workgroup counts as done
    }
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(done, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    if (s == 0 && on) {
        unsigned long long tot = 0;
#pragma unroll
        for (int u = 0; u < kKeySets; ++u) tot += atomicExch(&rsum[u * kKeyRow + b], 0ull);
        sumr[b] = q * (double)(long long)tot;
    }
    if (threadIdx.x == 0) *done = 0;
}

}  // namespace

void riskb_shape(int64_t n, int bpad, int64_t* tile, int* nwg)
{
    const int tpw = kUnits / (bpad / 16);
    *tile = max((int64_t)kMinTile, (n + (int64_t)kWgs * tpw - 1) / ((int64_t)kWgs * tpw));
    *nwg = (int)((n + *tile * tpw - 1) / (*tile * tpw));
}

int64_t riskb_tiles() { return (int64_t)kWgs * kUnits; }
int riskb_wgs() { return kWgs; }

hipError_t launch_risk_rows(RiskArgs a, hipStream_t s)
{
    if (a.bpad < 16 || a.bpad > 64 || a.bpad % 16 || a.B > a.bpad || !a.egrank || !a.mkey || !a.rkey)
        return hipErrorInvalidValue;
    int nwg = 0;
    riskb_shape(a.n, a.bpad, &a.tile, &nwg);
    a.ntile = nwg;  // rows of Lpart
    if (nwg > kWgs) return hipErrorInvalidValue;
    hipLaunchKernelGGL(riskb_max_kernel, dim3(nwg), dim3(kBT), 0, s, a);
    hipLaunchKernelGGL(riskb_w_kernel, dim3(nwg), dim3(kBT), 0, s, a);
    hipLaunchKernelGGL(riskb_q_kernel, dim3(nwg), dim3(kBT), 0, s, a);
    if (a.r64) hipLaunchKernelGGL(riskb_r_kernel, dim3(nwg), dim3(kBT), 0, s, a);
    hipLaunchKernelGGL(riskb_finish_kernel, dim3(a.B), dim3(riskdev::kT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_quantize_rows(const double* r, int64_t n, int B, const unsigned long long* rkey, int8_t* limbs,
                                int64_t lstride, int bpad, int nlimb, double* qscale, unsigned long long* rsum,
                                unsigned* done, double* sumr, hipStream_t s)
{
    if (lstride % 256 || lstride < n || bpad < B || bpad > 64 || bpad % 16 || (nlimb != 2 && nlimb != 3))
        return hipErrorInvalidValue;
    const int64_t nchunk = (n + 255) / 256 * 16, per = kQT / bpad;
    const unsigned grid = (unsigned)min((int64_t)256, (nchunk + per - 1) / per);
    hipLaunchKernelGGL(quantize_rows_kernel, dim3(grid), dim3(kQT), 0, s, r, n, B, rkey, limbs, bpad, nlimb, qscale,
                       rsum, done, sumr);
    return hipGetLastError();
}

}  // namespace cox
