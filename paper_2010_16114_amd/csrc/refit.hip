// refit.hip -- the unpenalised Cox refit on a chosen set of columns.
//
// Section 6 ranks the SNPs that the lasso path selects, then refits the
// unpenalised Cox model on them together with the covariates and keeps those
// whose Wald p-value passes a Bonferroni threshold.  The refit here is
// Newton's method on L over the M chosen columns, gathered into a dense FP32
// block D (M columns of ldd rows, rows in the sorted order of the times,
// zero past n; genotype columns standardised as (g - mu_j) s_j, formed in FP64
// and rounded once).
//
// With w = exp(eta - max eta), r = delta - w c (the risk-set pass), and in the
// sorted order S1(k) = sum_{k' <= k} w_k' d_k' (the risk-set sums of the rows
// of D), the negative Hessian of L in the coefficients is
//     -H = sum_i w_i c_i d_i d_i'  -  sum_G n_G S1(G) S1(G)' / W(G)^2
// where the first sum runs over subjects (w_i c_i = delta_i - r_i) and the
// second over tie groups G with n_G > 0 events, read at the group's last
// sorted position (Breslow).  Both terms are Gram matrices of tall arrays: D
// with row weights delta - r, and P with one row S1(G) per event group and
// row weights n_G / W(G)^2.  They are formed on the FP64 matrix cores from
// fixed-order partial sums.  -H is factorised by a blocked Cholesky; the Newton direction
// and the diagonal of (-H)^{-1} (squared standard errors) come from blocked
// triangular solves with that factor.
#include "device_common.h"

namespace cox {
namespace {

constexpr int kT = 256;
constexpr int kGT = 128;         // Gram output tile (kGT x kGT), 32 rows of it per wavefront
constexpr int kGR = 32;          // row chunks of the Gram kernel start on multiples of this
constexpr int kScanChunk = 4096; // sorted positions per workgroup of the risk-set scans
constexpr int kCB = 32;          // block size of the Cholesky factorisation and the triangular solves

__device__ double block_sum256(double v, double* sh)
{
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double s = 0.0;
    for (int q = 0; q < kT / kWave; ++q) s += sh[q];
    return s;
}

// D[a][k] = x~(perm[k], cols[a]) for k < n, 0 for n <= k < ldd
__global__ __launch_bounds__(kT) void gather_kernel(XDesc x, const int32_t* __restrict__ cols,
                                                    const int32_t* __restrict__ perm, float* __restrict__ D,
                                                    int64_t ldd)
{
    const int a = blockIdx.y;
    const int64_t j = cols[a];
    double mu = 0.0, sc = 1.0;
    if (x.xt != XT_F32) {
        if (x.center) mu = x.center[j];
        if (x.scale) sc = x.scale[j];
    }
    for (int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x; k < ldd; k += (int64_t)gridDim.x * kT) {
        double v = 0.0;
        if (k < x.n) {
            const int64_t off = j * x.ldx + perm[k];
            if (x.xt == XT_F32)
                v = load_x1<XT_F32>(x.X, off);
            else if (x.xt == XT_FP8)
                v = ((double)load_x1<XT_FP8>(x.X, off) - mu) * sc;
            else
                v = ((double)load_x1<XT_I8>(x.X, off) - mu) * sc;
        }
        D[(int64_t)a * ldd + k] = (float)v;
    }
}

// D[a][k] = Z[a][perm[k]] for k < n, 0 for n <= k < ldd (Z column-major, ldz)
__global__ __launch_bounds__(kT) void gather_z_kernel(const float* __restrict__ Z, int64_t ldz, int64_t n,
                                                      const int32_t* __restrict__ perm, float* __restrict__ D,
                                                      int64_t ldd)
{
    const int a = blockIdx.y;
    for (int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x; k < ldd; k += (int64_t)gridDim.x * kT)
        D[(int64_t)a * ldd + k] = k < n ? Z[(int64_t)a * ldz + perm[k]] : 0.0f;
}

// eta[perm[k]] = sum_a D[a][k] b[a]  (eta in subject order).  A workgroup takes 256
// positions, a lane 4 of them and a wavefront every fourth column, 8 16-byte loads
// in flight; the four wavefronts' sums are added in order.  Bound by reading D:
// with a position per lane and all columns in one chain of 4-byte loads it took
// 182 us at 400,000 x 344, 111 now (5.0 TB/s).
__global__ __launch_bounds__(kT) void refit_eta_kernel(const float* __restrict__ D, int64_t ldd, int64_t n, int M,
                                                       const int32_t* __restrict__ perm,
                                                       const double* __restrict__ b, double* __restrict__ eta)
{
    constexpr int NW = kT / kWave;
    __shared__ double sh[NW][4][kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t k0 = (int64_t)blockIdx.x * kT, k = k0 + 4 * lane;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (k < ldd) {
        const float* Dk = D + k;
#pragma unroll 8
        for (int a = wid; a < M; a += NW) {
            const float4 d = *reinterpret_cast<const float4*>(Dk + (int64_t)a * ldd);
            const double ba = b[a];
            s[0] += (double)d.x * ba, s[1] += (double)d.y * ba, s[2] += (double)d.z * ba, s[3] += (double)d.w * ba;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sh[wid][e][lane] = s[e];
    __syncthreads();
    const int t = threadIdx.x;
    if (k0 + t >= n) return;
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) v += sh[q][t & 3][t >> 2];
    eta[perm[k0 + t]] = v;
}

// rs[k] = r[perm[k]]: the residuals in the sorted order
__global__ void sort_r_kernel(const int32_t* __restrict__ perm, const double* __restrict__ r, int64_t n,
                              double* __restrict__ rs)
{
    for (int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x; k < n; k += (int64_t)gridDim.x * kT) rs[k] = r[perm[k]];
}

// row weights of the first Hessian term in the sorted order: wt[k] = delta - r
// of subject perm[k] for k < n, 0 for n <= k < ldd
__global__ void hess_weight_kernel(const int32_t* __restrict__ perm, const uint8_t* __restrict__ ev,
                                   const double* __restrict__ r, int64_t n, int64_t ldd, double* __restrict__ wt)
{
    for (int64_t k = (int64_t)blockIdx.x * kT + threadIdx.x; k < ldd; k += (int64_t)gridDim.x * kT)
        wt[k] = k < n ? (ev[k] ? 1.0 : 0.0) - r[perm[k]] : 0.0;
}

constexpr int kScanJ = kScanChunk / (4 * kT);  // sub-blocks of 4 kT positions in a scan chunk

// v[j][e] = w[k] at position k = k0 + 4 kT j + 4 t + e of thread t: consecutive
// threads read consecutive 16-byte pieces.  0 at or past n.  k0 is a multiple of
// 4 kT.
__device__ __forceinline__ void scan_weights(const double* __restrict__ w, int64_t k0, int64_t n, double (*v)[4])
{
#pragma unroll
    for (int j = 0; j < kScanJ; ++j) {
        const int64_t kb = k0 + 4 * kT * j + 4 * (int64_t)threadIdx.x;
        if (kb + 4 <= n) {
            const double2 x0 = *reinterpret_cast<const double2*>(w + kb);
            const double2 x1 = *reinterpret_cast<const double2*>(w + kb + 2);
            v[j][0] = x0.x, v[j][1] = x0.y, v[j][2] = x1.x, v[j][3] = x1.y;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[j][e] = kb + e < n ? w[kb + e] : 0.0;
        }
    }
}

// the column's values at the same positions; 0 at or past ldd, as in its padding
// (ldd a multiple of 8)
__device__ __forceinline__ void scan_column(const float* __restrict__ Dcol, int64_t k0, int64_t ldd, float4* d)
{
#pragma unroll
    for (int j = 0; j < kScanJ; ++j) {
        const int64_t kb = k0 + 4 * kT * j + 4 * (int64_t)threadIdx.x;
        d[j] = kb < ldd ? *reinterpret_cast<const float4*>(Dcol + kb) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}

// The two sums over D at one coefficient vector, in one pass: per chunk ch of
// kScanChunk sorted positions gpart[a][ch] = sum_k D[a][k] rs[k] (the gradient) and
// csum[a][ch] = sum_k D[a][k] w[k], csum[M][ch] = sum_k w[k] (the risk-set scans of
// the Hessian).  A workgroup keeps the chunk's rs and w in registers over kSumCols
// columns, the next column's loads under way.  Bound by reading D: 115 us at
// 400,000 x 344 (4.8 TB/s), where one pass for each sum, reading rs or w again for
// every column, took 170 and 127.
constexpr int kSumCols = 8;
__global__ __launch_bounds__(kT) void refit_sums_kernel(const float* __restrict__ D, int64_t ldd, int64_t n, int M,
                                                        const double* __restrict__ rs, const double* __restrict__ w,
                                                        int nch, double* __restrict__ gpart,
                                                        double* __restrict__ csum)
{
    constexpr int NW = kT / kWave;
    __shared__ double sh[kSumCols + 1][2][NW];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int ch = blockIdx.x, a0 = blockIdx.y * kSumCols, na = min(kSumCols, M - a0);
    const int64_t k0 = (int64_t)ch * kScanChunk;
    float4 d[kScanJ], dn[kScanJ];
    scan_column(D + (int64_t)a0 * ldd, k0, ldd, dn);
    double rv[kScanJ][4], wv[kScanJ][4];
    scan_weights(rs, k0, n, rv);
    scan_weights(w, k0, n, wv);
    for (int c = 0; c < na; ++c) {
#pragma unroll
        for (int j = 0; j < kScanJ; ++j) d[j] = dn[j];
        if (c + 1 < na) scan_column(D + (int64_t)(a0 + c + 1) * ldd, k0, ldd, dn);
        double sr = 0.0, sw = 0.0;
#pragma unroll
        for (int j = 0; j < kScanJ; ++j) {
            const double v[4] = {(double)d[j].x, (double)d[j].y, (double)d[j].z, (double)d[j].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) sr += v[e] * rv[j][e], sw += v[e] * wv[j][e];
        }
        sr = wave_sum(sr);
        sw = wave_sum(sw);
        if (lane == 0) sh[c][0][wid] = sr, sh[c][1][wid] = sw;
    }
    double sw = 0.0;
    if (a0 == 0) {
#pragma unroll
        for (int j = 0; j < kScanJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) sw += wv[j][e];
        sw = wave_sum(sw);
        if (lane == 0) sh[kSumCols][1][wid] = sw;
    }
    __syncthreads();
    const int c = threadIdx.x >> 1, which = threadIdx.x & 1;
    if (c < na || (c == kSumCols && which && a0 == 0)) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) v += sh[c][which][q];
        const int a = c == kSumCols ? M : a0 + c;
        (which ? csum : gpart)[(int64_t)a * nch + ch] = v;
    }
}

// g[a] = sum_ch gpart[a][ch], one wavefront per a, in a fixed order
__global__ __launch_bounds__(kT) void refit_sum_kernel(const double* __restrict__ gpart, int nch, int M,
                                                       double* __restrict__ g)
{
    const int lane = threadIdx.x & (kWave - 1), a = blockIdx.x * (kT / kWave) + threadIdx.x / kWave;
    if (a >= M) return;
    double s = 0.0;
    for (int ch = lane; ch < nch; ch += kWave) s += gpart[(int64_t)a * nch + ch];
    s = wave_sum(s);
    if (lane == 0) g[a] = s;
}

// The prefix sums at the event groups: with P_a(k) = sum_{k' <= k} w[k'] D[a][k']
// (a < M) and P_M(k) = sum_{k' <= k} w[k'] in the sorted order, P[a][g] =
// P_a(k) at the last position k of event group g (egidx[k] = g; -1 at every
// other position).  Workgroup (ch, y) scans chunk ch of kScanCols columns, starting
// from the sums of the earlier chunks: each thread's 4 positions in each
// sub-block are summed in place, every sub-block is scanned across the
// wavefront, and one exchange of the wavefront totals places them.  The chunk's
// w and egidx stay in registers over the columns, the next column's loads are under
// way meanwhile: read again for every column, three bytes of them to each of D, the
// scan took 246 us at 400,000 x 344, now 213.  Chunk 0 also clears P's padding
// rows G .. ldp - 1.
constexpr int kScanCols = kT / kWave;  // a wavefront sums the earlier chunks of each
__global__ __launch_bounds__(kT) void scan_p_kernel(const float* __restrict__ D, int64_t ldd, int64_t n, int M,
                                                    const double* __restrict__ w, const double* __restrict__ csum,
                                                    int nch, const int32_t* __restrict__ egidx, int64_t G,
                                                    int64_t ldp, double* __restrict__ P)
{
    constexpr int NW = kT / kWave;
    __shared__ double sv[2][kScanJ][NW], scv[kScanCols];
    const int ch = blockIdx.x, a0 = blockIdx.y * kScanCols, na = min(kScanCols, M + 1 - a0);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int64_t k0 = (int64_t)ch * kScanChunk;
    float4 d[kScanJ], dn[kScanJ];
    if (a0 < M) scan_column(D + (int64_t)a0 * ldd, k0, ldd, dn);
    double wv[kScanJ][4];
    int32_t g[kScanJ][4];
    scan_weights(w, k0, n, wv);
#pragma unroll
    for (int j = 0; j < kScanJ; ++j) {
        const int64_t kb = k0 + 4 * kT * j + 4 * (int64_t)threadIdx.x;
        if (kb + 4 <= n) {
            const int4 q = *reinterpret_cast<const int4*>(egidx + kb);
            g[j][0] = q.x, g[j][1] = q.y, g[j][2] = q.z, g[j][3] = q.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) g[j][e] = kb + e < n ? egidx[kb + e] : -1;
        }
    }
    if (wid < na) {
        double cv = 0.0;
        for (int c = lane; c < ch; c += kWave) cv += csum[(int64_t)(a0 + wid) * nch + c];
        cv = wave_sum(cv);
        if (lane == 0) scv[wid] = cv;
    }
    for (int c = 0; c < na; ++c) {
        const int a = a0 + c;
#pragma unroll
        for (int j = 0; j < kScanJ; ++j) d[j] = dn[j];
        if (c + 1 < na && a + 1 < M) scan_column(D + (int64_t)(a + 1) * ldd, k0, ldd, dn);
        double v[kScanJ][4], iv[kScanJ];
#pragma unroll
        for (int j = 0; j < kScanJ; ++j) {
            const float de[4] = {d[j].x, d[j].y, d[j].z, d[j].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[j][e] = a < M ? wv[j][e] * (double)de[e] : wv[j][e];
                if (e) v[j][e] += v[j][e - 1];
            }
            iv[j] = wave_incl_scan(v[j][3], lane);
            if (lane == kWave - 1) sv[c & 1][j][wid] = iv[j];
        }
        __syncthreads();
        double* Pa = P + (int64_t)a * ldp;
        if (ch == 0 && threadIdx.x < ldp - G) Pa[G + threadIdx.x] = 0.0;
        double before = scv[c];  // the earlier chunks and sub-blocks
#pragma unroll
        for (int j = 0; j < kScanJ; ++j) {
            // plus the earlier wavefronts of this sub-block and the earlier lanes
            double bv = before + iv[j] - v[j][3];
            for (int q = 0; q < wid; ++q) bv += sv[c & 1][j][q];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (g[j][e] >= 0) Pa[g[j][e]] = bv + v[j][e];
            for (int q = 0; q < NW; ++q) before += sv[c & 1][j][q];
        }
    }
}

// Row weights of the second Hessian term: wg[g] = n_G / W(G)^2 with W(G) =
// P[M][g], so that sum_g wg[g] P_a(g) P_b(g) = sum_G n_G S1_a S1_b / W^2; 0 on
// the padding rows G .. ldp - 1.
__global__ void event_weight_kernel(const double* __restrict__ PM, const int32_t* __restrict__ egcnt, int64_t G,
                                    int64_t ldp, double* __restrict__ wg)
{
    for (int64_t g = (int64_t)blockIdx.x * kT + threadIdx.x; g < ldp; g += (int64_t)gridDim.x * kT) {
        double v = 0.0;
        if (g < G) {
            const double W = PM[g];
            v = (double)egcnt[g] / (W * W);
        }
        wg[g] = v;
    }
}

// Gram terms: for a 128 x 128 output tile (ta, tb), ta <= tb, and a chunk of the rows
// k, sum_k wt_k A[a][k] A[b][k], a <= b.  A is column-major (lda a multiple of 8, 0
// past the rows, wt likewise); every chunk starts on a multiple of kGR rows.
//
// On the FP64 matrix cores with v_mfma_f64_4x4x4f64, four independent 4 x 4 x 4
// products: per lane, block l / 4 mod 4 holds A (row l % 4, k l / 16), B (k l / 16,
// column l % 4) and D (row l / 16, column l % 4).  Every block takes the same four
// rows, so an instruction multiplies 4 rows by 16 columns.  It sustains 67 to 72
// TFLOP/s here, v_mfma_f64_16x16x4f64 31 to 44 in the same loop.  Any vector
// instruction between takes its issue slots from the matrix pipe, so the operands are
// converted and weighted once per workgroup, on their way into LDS, not per
// wavefront.
//
// A step is one 128-byte line of every column (32 FP32 rows, 16 FP64); 8 lanes load a
// line.  The weighted columns of ta and the plain ones of tb lie in LDS as doubles,
// with column strides that put a read of 16 columns on mostly distinct banks; the
// next step's lines load into registers meanwhile.
// Wavefront w takes the blocks of 16 rows w and 7 - w and leaves out the 16 x 16
// blocks below the diagonal or past M (the reduction reads the upper triangle), so
// that on the diagonal too the four have the same work: 9 blocks each.
//
// Bound by the matrix cores and the steps' latency.  At 400,000 x 344 the FP32 term
// took 1360 us and the FP64 term (80,000 event groups) 366 with one wavefront per
// 64 x 64 tile straight from memory on v_mfma_f64_16x16x4f64; now 1110 and 266
// (its products alone take 660 us at the instruction's rate).  That form on the 4x4x4
// instruction, its columns rotated across lanes, took 2030: the conversions and
// rotations of every wavefront stood in the matrix pipe's way.

// A tile's place in the list of workgroups: those of chunk ch of its kind start at
// first + ch * count, its own is idx further on.
struct GramTile {
    int ta, tb, first, count, idx, chunks;
};
__device__ __forceinline__ int gram_tiles(int M) { return (M - 1) / kGT; }  // but the last
__device__ __forceinline__ GramTile gram_find(const GramPlan& g, int M, int ta, int tb)
{
    const int nt1 = gram_tiles(M), pairs = nt1 * (nt1 - 1) / 2;
    const int edge = pairs * g.full, diag = edge + nt1 * g.edge, last = diag + nt1 * g.diag;
    if (ta != tb) {
        if (tb == nt1) return GramTile{ta, tb, edge, nt1, ta, g.edge};
        return GramTile{ta, tb, 0, pairs, ta * (nt1 - 1) - ta * (ta - 1) / 2 + tb - ta - 1, g.full};
    }
    if (tb == nt1) return GramTile{ta, tb, last, 1, 0, g.last};
    return GramTile{ta, tb, diag, nt1, ta, g.diag};
}

template <class T>
struct GramStep;
template <>
struct GramStep<float> {
    static constexpr int K = 32, E = 4, S = 38;
    using V = float4;
};
template <>
struct GramStep<double> {
    static constexpr int K = 16, E = 2, S = 18;
    using V = double2;
};
__device__ __forceinline__ void unpack(const float4& v, double* o)
{
    o[0] = (double)v.x, o[1] = (double)v.y, o[2] = (double)v.z, o[3] = (double)v.w;
}
__device__ __forceinline__ void unpack(const double2& v, double* o) { o[0] = v.x, o[1] = v.y; }

// one step's products of a wavefront: rows 16 of block h (as0, as1) by block t of 16
// columns if bit 8 h + t of mask is set
template <int K, int S>
__device__ __forceinline__ void gram_step(const double (*__restrict__ as0)[S], const double (*__restrict__ as1)[S],
                                          const double (*__restrict__ bs)[S], int lane, int mask, double (*acc)[8])
{
#pragma unroll 1
    for (int kk = 0; kk < K; kk += 8) {
        // a lane's k-slot l / 16 takes two neighbouring rows, in both operands
        const int k = kk + 2 * (lane >> 4);
        double2 av[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            av[q] = *reinterpret_cast<const double2*>(&as0[q * 4 + (lane & 3)][k]);
            av[4 + q] = *reinterpret_cast<const double2*>(&as1[q * 4 + (lane & 3)][k]);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const double2 bv = *reinterpret_cast<const double2*>(&bs[t * 16 + (lane & 15)][k]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (!((mask >> (8 * h + t)) & 1)) continue;
#pragma unroll
                for (int q = 4 * h; q < 4 * h + 4; ++q)
                    acc[q][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[q].x, bv.x, acc[q][t], 0, 0, 0);
#pragma unroll
                for (int q = 4 * h; q < 4 * h + 4; ++q)
                    acc[q][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[q].y, bv.y, acc[q][t], 0, 0, 0);
            }
        }
    }
}

template <class T>
__global__ __launch_bounds__(kT, 2) void gram_kernel(const T* __restrict__ A, int64_t lda, int64_t n, int M,
                                                     const double* __restrict__ wt, GramPlan g,
                                                     double* __restrict__ part)
{
    using V = typename GramStep<T>::V;
    constexpr int K = GramStep<T>::K, E = GramStep<T>::E, LS = GramStep<T>::S, P = kGT / 32;
    __shared__ __attribute__((aligned(16))) double as[kGT][LS], bs[kGT][LS];
    // workgroup -> (tile, chunk): the full tiles above the diagonal, those of the last
    // column, those on the diagonal, the last one; within a kind the chunks outermost
    const int nt1 = gram_tiles(M), pairs = nt1 * (nt1 - 1) / 2;
    int idx = blockIdx.x, ta, tb, ch, nc;
    if (idx < pairs * g.full) {
        ch = idx / pairs, nc = g.full;
        idx -= ch * pairs;
        ta = 0;
        while (idx >= nt1 - 1 - ta) {
            idx -= nt1 - 1 - ta;
            ++ta;
        }
        tb = ta + 1 + idx;
    } else if ((idx -= pairs * g.full) < nt1 * g.edge) {
        ch = idx / nt1, nc = g.edge, ta = idx - ch * nt1, tb = nt1;
    } else if ((idx -= nt1 * g.edge) < nt1 * g.diag) {
        ch = idx / nt1, nc = g.diag, ta = tb = idx - ch * nt1;
    } else {
        ch = idx - nt1 * g.diag, nc = g.last, ta = tb = nt1;
    }
    const bool diag = ta == tb;
    // the wavefront's blocks of 16 rows, wid and 7 - wid, by 8 blocks of 16 columns:
    // those with an entry on or above the diagonal, of rows and columns below M
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int u0 = wid * 16, u1 = (7 - wid) * 16;
    int mask = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int b = tb * kGT + t * 16;
        mask |= (ta * kGT + u0 <= b && b < M) << t;
        mask |= (ta * kGT + u1 <= b && b < M) << (8 + t);
    }
    const int64_t rows = ((n + nc - 1) / nc + kGR - 1) / kGR * kGR;
    const int64_t r0 = ch * rows, r1 = min(n, r0 + rows);
    double acc[8][8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[u][t] = 0.0;
    // thread: rows E (tid % 8) .. of the step, columns tid / 8 + 32 p.  Columns past
    // M are read from column M - 1: they only reach outputs that are not stored.  A
    // piece at or past r1 is read at r0 with weight 0 (one that starts before r1
    // ends before lda: r1 <= the rows, lda >= them rounded up to 8).
    const int piece = threadIdx.x & 7, c0 = threadIdx.x >> 3;
    V va[P], vb[P];
    double vw[E];
    bool in = false;
    auto fetch = [&](int64_t s0) {
        const int64_t k = s0 + E * piece;
        in = k < r1;
        const int64_t kl = in ? k : r0;
#pragma unroll
        for (int p = 0; p < P; ++p)
            va[p] = *reinterpret_cast<const V*>(A + (int64_t)min(ta * kGT + c0 + 32 * p, M - 1) * lda + kl);
        if (!diag) {
#pragma unroll
            for (int p = 0; p < P; ++p)
                vb[p] = *reinterpret_cast<const V*>(A + (int64_t)min(tb * kGT + c0 + 32 * p, M - 1) * lda + kl);
        }
#pragma unroll
        for (int e = 0; e < E; e += 2) {
            const double2 x = *reinterpret_cast<const double2*>(wt + kl + e);
            vw[e] = x.x, vw[e + 1] = x.y;
        }
    };
    if (r0 < r1) fetch(r0);
    for (int64_t s0 = r0; s0 < r1; s0 += K) {
        double w[E];
#pragma unroll
        for (int e = 0; e < E; ++e) w[e] = in ? vw[e] : 0.0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            double x[E], y[E];
            unpack(va[p], x);
            unpack(diag ? va[p] : vb[p], y);
#pragma unroll
            for (int e = 0; e < E; e += 2) {
                *reinterpret_cast<double2*>(&as[c0 + 32 * p][E * piece + e]) = double2{x[e] * w[e], x[e + 1] * w[e + 1]};
                *reinterpret_cast<double2*>(&bs[c0 + 32 * p][E * piece + e]) = double2{y[e], y[e + 1]};
            }
        }
        __syncthreads();
        if (s0 + K < r1) fetch(s0 + K);
        if (mask) gram_step<K, LS>(as + u0, as + u1, bs, lane, mask, acc);
        __syncthreads();
    }
    const int S = min(M, kGT);
    part += (int64_t)blockIdx.x * S * S;
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int a = (u < 4 ? u0 : u1) + (u & 3) * 4 + (lane >> 4), b = t * 16 + (lane & 15);
            const int ga = ta * kGT + a, gb = tb * kGT + b;
            if (gb < M && ga <= gb) part[a * S + b] = acc[u][t];
        }
}

// H[a][b] = H[b][a] = sum_c p1[c][a][b] - sum_c p2[c][a][b], a <= b, over the chunks c
// of the entry's tile: the Gram kernel writes every entry of the upper triangle.
__global__ void gram_reduce_kernel(const double* __restrict__ p1, GramPlan g1, const double* __restrict__ p2,
                                   GramPlan g2, int M, double* __restrict__ H)
{
    const int S = min(M, kGT);
    for (int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x; t < (int64_t)M * M; t += (int64_t)gridDim.x * kT) {
        const int a = (int)(t / M), b = (int)(t % M);
        if (a > b) continue;
        const int ta = a / kGT, tb = b / kGT;
        const int64_t at = (a - ta * kGT) * S + b - tb * kGT;
        const GramTile t1 = gram_find(g1, M, ta, tb), t2 = gram_find(g2, M, ta, tb);
        const double *q1 = p1 + (int64_t)(t1.first + t1.idx) * S * S + at, *q2 = p2 + (int64_t)(t2.first + t2.idx) * S * S + at;
        double s = 0.0;
#pragma unroll 8
        for (int c = 0; c < t1.chunks; ++c) s += q1[(int64_t)c * t1.count * S * S];
#pragma unroll 8
        for (int c = 0; c < t2.chunks; ++c) s -= q2[(int64_t)c * t2.count * S * S];
        H[t] = s;
        H[(int64_t)b * M + a] = s;
    }
}

// Blocked right-looking Cholesky A = L L' of the symmetric positive definite
// M x M matrix (row-major; the lower triangle receives L, the upper one is
// left as it was), in blocks of kCB.  Step J runs chol_panel_kernel, then
// chol_update_kernel on the trailing lower blocks.

// lane `src`'s v (src the same in every lane)
__device__ __forceinline__ double bcast(double v, int src)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                            __builtin_amdgcn_readlane(__double2loint(v), src));
}

// a / d from inv = 1 / d: the rounded product and one correction by its remainder, which an
// fma gives exactly (the last step of Markstein's division), a chain of three where the
// division's own is about ten
__device__ __forceinline__ double quotient(double a, double d, double inv)
{
    const double q = a * inv;
    return fma(fma(-d, q, a), inv, q);
}

// One wavefront per workgroup: lanes 0 .. kCB - 1 hold the rows of the diagonal
// block J in registers (every workgroup factorises it, the same arithmetic in each),
// lanes kCB .. 2 kCB - 1 those of block row J + b of the panel, b = blockIdx.x, which
// the same column steps turn into X with X L_JJ' = A_(J+b)J.  Workgroup 0 stores the
// factorised block, to `diag` (row-major, kCB wide) unless it is alone, because the
// others may still have to read A's, and the flag; workgroup b > 0 its panel rows.
// chol_update_kernel moves `diag` into A.  ok[0] = 1 after the
// first step, set to 0 by any step that meets a pivot that is not positive (the
// pivot is then taken as 1 and the factorisation runs on).  A chain of kCB square
// roots, divisions and rank-1 updates: in LDS, with four barriers per column and
// the panel solved afterwards, it took 28.5 us a step at M = 344, now 19.7.
__global__ __launch_bounds__(kWave) void chol_panel_kernel(double* __restrict__ A, int M, int J,
                                                            double* __restrict__ diag, int* __restrict__ ok)
{
    static_assert(2 * kCB == kWave && kCB * kCB == kCholDiag, "a lane per row of the two blocks");
    __shared__ double T[2 * kCB][kCB + 1];
    const int lane = threadIdx.x;
    const int j0 = J * kCB, bs = min(kCB, M - j0), i0 = (J + blockIdx.x) * kCB;
    // a panel block exists only below a full diagonal block (bs == kCB)
    const int rs = blockIdx.x ? min(kCB, M - i0) : 0;
#pragma unroll
    for (int t = 0; t < kCB; ++t) {  // two rows of kCB at a time
        const int r = 2 * t + lane / kCB, c = lane % kCB;
        const bool top = r < kCB;
        const int row = top ? j0 + r : i0 + r - kCB;
        T[r][c] = c < bs && (top ? r < bs : r - kCB < rs) ? A[(int64_t)row * M + j0 + c] : 0.0;
    }
    __syncthreads();
    double x[kCB];
#pragma unroll
    for (int c = 0; c < kCB; ++c) x[c] = T[lane][c];
    // entries right of the diagonal are carried along in lanes that no other reads
    bool good = true;
#pragma unroll
    for (int j = 0; j < kCB; ++j) {
        if (j < bs) {
            const double d = bcast(x[j], j);
            good = good && d > 0.0;
            const double piv = d > 0.0 ? sqrt(d) : 1.0;
            x[j] = lane == j ? piv : quotient(x[j], piv, 1.0 / piv);
#pragma unroll
            for (int k = j + 1; k < kCB; ++k) x[k] -= x[j] * bcast(x[j], k);
        }
    }
#pragma unroll
    for (int c = 0; c < kCB; ++c) T[lane][c] = x[c];
    __syncthreads();
    if (blockIdx.x == 0) {
        for (int e = lane; e < kCB * kCB; e += kWave) {
            const int r = e / kCB, c = e % kCB;
            if (gridDim.x > 1)
                diag[e] = T[r][c];
            else if (r < bs && c <= r)
                A[(int64_t)(j0 + r) * M + j0 + c] = T[r][c];
        }
        if (lane == 0) {
            if (J == 0)
                ok[0] = good;
            else if (!good)
                ok[0] = 0;
        }
        return;
    }
    for (int e = lane; e < kCB * kCB; e += kWave) {
        const int r = e / kCB, c = e % kCB;
        if (r < rs) A[(int64_t)(i0 + r) * M + j0 + c] = T[kCB + r][c];
    }
}

// A_IK -= L_IJ L_KJ' for the trailing lower blocks J < K <= I (in a diagonal
// block only on and below the diagonal); one block per workgroup, and the last
// workgroup stores step J's factorised diagonal block.
__global__ __launch_bounds__(kT) void chol_update_kernel(double* __restrict__ A, int M, int J,
                                                         const double* __restrict__ diag)
{
    __shared__ double Pi[kCB][kCB + 1], Pk[kCB][kCB + 1];
    if (blockIdx.x == gridDim.x - 1) {
        for (int e = threadIdx.x; e < kCB * kCB; e += kT) {
            const int r = e / kCB, c = e % kCB;
            if (c <= r) A[(int64_t)(J * kCB + r) * M + J * kCB + c] = diag[e];
        }
        return;
    }
    int64_t t = blockIdx.x;
    int ii = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((int64_t)ii * (ii + 1) / 2 > t) --ii;
    while ((int64_t)(ii + 1) * (ii + 2) / 2 <= t) ++ii;
    const int kk = (int)(t - (int64_t)ii * (ii + 1) / 2);
    const int I = J + 1 + ii, K = J + 1 + kk, j0 = J * kCB;
    for (int e = threadIdx.x; e < kCB * kCB; e += kT) {
        const int r = e / kCB, c = e % kCB;
        const int ri = I * kCB + r, rk = K * kCB + r;
        Pi[r][c] = ri < M ? A[(int64_t)ri * M + j0 + c] : 0.0;
        Pk[r][c] = rk < M ? A[(int64_t)rk * M + j0 + c] : 0.0;
    }
    __syncthreads();
    const int r = threadIdx.x >> 3;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int qq = 0; qq < kCB; ++qq) {
        const double pi = Pi[r][qq];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] += pi * Pk[(threadIdx.x & 7) + 8 * u][qq];
    }
    const int row = I * kCB + r;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int cc = (threadIdx.x & 7) + 8 * u, col = K * kCB + cc;
        if (row < M && col < M && (I != K || cc <= r)) A[(int64_t)row * M + col] -= acc[u];
    }
}

// Forward substitution L y = e on rows from block I0 on (L from the blocked
// Cholesky, y in LDS ys[], whose entries below I0 kCB are not read); e is g
// (rows i) or, with g null, the unit vector at row `unit`.  Per block: the
// known part of each row's sum with 8 threads per row, then the kCB x kCB
// diagonal block in one wavefront, lane r holding row r of it in registers, loaded
// before the sums.  The chain over the rows is the time: with a division and a shuffle
// through LDS per row the two solves took 146 us at M = 344, now 120 (the sums' loads
// and barriers, 22 blocks one after the other).
__device__ void lower_solve(const double* __restrict__ L, int M, int I0, const double* __restrict__ g, int unit,
                            double* ys, double* red)
{
    const int nb = (M + kCB - 1) / kCB;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int I = I0; I < nb; ++I) {
        const int i0 = I * kCB, rb = min(kCB, M - i0);
        double lr[kCB], ld = 1.0;
        if (wid == 0) {
#pragma unroll
            for (int c = 0; c < kCB; ++c) lr[c] = (lane < rb && c <= lane) ? L[(int64_t)(i0 + lane) * M + i0 + c] : 0.0;
            if (lane < rb) ld = L[(int64_t)(i0 + lane) * M + i0 + lane];
        }
        {
            const int r = threadIdx.x >> 3, s = threadIdx.x & 7;
            double part = 0.0;
            if (r < rb)
#pragma unroll 8
                for (int k = I0 * kCB + s; k < i0; k += 8) part += L[(int64_t)(i0 + r) * M + k] * ys[k];
            part += __shfl_xor(part, 1, kWave);
            part += __shfl_xor(part, 2, kWave);
            part += __shfl_xor(part, 4, kWave);
            if (s == 0) red[r] = part;
        }
        __syncthreads();
        if (wid == 0) {
            double b = 0.0;
            const double inv = 1.0 / ld;
            if (lane < rb) b = (g ? g[i0 + lane] : (i0 + lane == unit ? 1.0 : 0.0)) - red[lane];
#pragma unroll
            for (int c = 0; c < kCB; ++c) {
                if (c < rb) {
                    const double yc = bcast(quotient(b, ld, inv), c);
                    if (lane > c) b -= lr[c] * yc;
                    if (lane == c) b = yc;
                }
            }
            if (lane < rb) ys[i0 + lane] = b;
        }
        __syncthreads();
    }
}

// Back substitution L' x = y in place in ys[] (all M rows), the same blocking:
// the known part of each row's sum reads row k of L across 32 columns (8
// slices of k), and lane r holds column r of the diagonal block.
__device__ void upper_solve(const double* __restrict__ L, int M, double* ys, double (*red8)[kCB])
{
    const int nb = (M + kCB - 1) / kCB;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int I = nb - 1; I >= 0; --I) {
        const int i0 = I * kCB, rb = min(kCB, M - i0), k0 = i0 + rb;
        double lc[kCB], ld = 1.0;
        if (wid == 0) {
#pragma unroll
            for (int c = 0; c < kCB; ++c)
                lc[c] = (lane < rb && c >= lane && c < rb) ? L[(int64_t)(i0 + c) * M + i0 + lane] : 0.0;
            if (lane < rb) ld = L[(int64_t)(i0 + lane) * M + i0 + lane];
        }
        {
            const int r = threadIdx.x & (kCB - 1), s = threadIdx.x / kCB;
            double part = 0.0;
            if (r < rb)
#pragma unroll 8
                for (int k = k0 + s; k < M; k += kT / kCB) part += L[(int64_t)k * M + i0 + r] * ys[k];
            red8[s][r] = part;
        }
        __syncthreads();
        if (wid == 0) {
            double b = 0.0;
            const double inv = 1.0 / ld;
            if (lane < rb) {
                b = ys[i0 + lane];
                for (int s = 0; s < kT / kCB; ++s) b -= red8[s][lane];
            }
#pragma unroll
            for (int c = kCB - 1; c >= 0; --c) {
                if (c < rb) {
                    const double xc = bcast(quotient(b, ld, inv), c);
                    if (lane < c) b -= lc[c] * xc;
                    if (lane == c) b = xc;
                }
            }
            if (lane < rb) ys[i0 + lane] = b;
        }
        __syncthreads();
    }
}

// x = (L L')^{-1} g with the factor from the blocked Cholesky.  One workgroup.
__global__ __launch_bounds__(kT) void chol_solve_kernel(const double* __restrict__ L, int M,
                                                        const double* __restrict__ g, double* __restrict__ x)
{
    __shared__ double ys[kMaxRefit];
    __shared__ double red8[kT / kCB][kCB];
    lower_solve(L, M, 0, g, -1, ys, red8[0]);
    upper_solve(L, M, ys, red8);
    for (int k = threadIdx.x; k < M; k += kT) x[k] = ys[k];
}

// Wald statistics from the factor, one workgroup per coefficient a: L y = e_a,
// so ((L L')^{-1})_aa = |y|^2 (y_k = 0 for k < a); se_a = its square root,
// z_a = b_a / se_a, p_a = erfc(|z_a| / sqrt 2).
__global__ __launch_bounds__(kT) void wald_kernel(const double* __restrict__ L, int M, const double* __restrict__ b,
                                                  double* __restrict__ se, double* __restrict__ pval)
{
    __shared__ double ys[kMaxRefit];
    __shared__ double red[kCB];
    __shared__ double sh[kT / kWave];
    const int a = blockIdx.x;
    lower_solve(L, M, a / kCB, nullptr, a, ys, red);
    double s2 = 0.0;
    for (int k = a + threadIdx.x; k < M; k += kT) s2 += ys[k] * ys[k];
    s2 = block_sum256(s2, sh);
    if (threadIdx.x == 0) {
        const double sd = sqrt(s2);
        se[a] = sd;
        pval[a] = erfc(fabs(b[a] / sd) * 0.70710678118654752440);
    }
}

// out = b + t d
__global__ void axpy_kernel(const double* __restrict__ b, const double* __restrict__ d, double t, int M,
                            double* __restrict__ out)
{
    const int a = blockIdx.x * kT + threadIdx.x;
    if (a < M) out[a] = b[a] + t * d[a];
}

// first sorted position with a nonzero coefficient per column: entry[j] = the
// smallest l with path[l][j] != 0 (or -1), coef[j] = |path[entry][j]|
__global__ void entry_kernel(const float* __restrict__ path, int L, int64_t ptot, int64_t p,
                             int32_t* __restrict__ entry, float* __restrict__ coef)
{
    for (int64_t j = (int64_t)blockIdx.x * kT + threadIdx.x; j < p; j += (int64_t)gridDim.x * kT) {
        int e = -1;
        float c = 0.0f;
        for (int l = 0; l < L; ++l) {
            const float v = path[(int64_t)l * ptot + j];
            if (v != 0.0f) {
                e = l;
                c = fabsf(v);
                break;
            }
        }
        entry[j] = e;
        coef[j] = c;
    }
}

inline unsigned grid_for(int64_t m) { return (unsigned)min((int64_t)8192, max((int64_t)1, (m + kT - 1) / kT)); }

}  // namespace

int64_t refit_ld(int64_t rows) { return max((int64_t)8, (rows + 7) / 8 * 8); }

hipError_t launch_gather_cols(const XDesc& x, const int32_t* cols, int m, const int32_t* perm, float* D, int64_t ldd,
                              hipStream_t s)
{
    if (m < 1 || ldd < refit_ld(x.n)) return hipErrorInvalidValue;
    const unsigned gx = (unsigned)min((int64_t)512, (ldd + kT - 1) / kT);
    hipLaunchKernelGGL(gather_kernel, dim3(gx, m), dim3(kT), 0, s, x, cols, perm, D, ldd);
    return hipGetLastError();
}

hipError_t launch_gather_z(const float* Z, int64_t ldz, int64_t n, int q, const int32_t* perm, float* D, int64_t ldd,
                           hipStream_t s)
{
    if (q < 1 || ldd < refit_ld(n)) return hipErrorInvalidValue;
    const unsigned gx = (unsigned)min((int64_t)512, (ldd + kT - 1) / kT);
    hipLaunchKernelGGL(gather_z_kernel, dim3(gx, q), dim3(kT), 0, s, Z, ldz, n, perm, D, ldd);
    return hipGetLastError();
}

hipError_t launch_refit_eta(const float* D, int64_t ldd, int64_t n, int M, const int32_t* perm, const double* b,
                            double* eta, hipStream_t s)
{
    if (ldd < refit_ld(n)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(refit_eta_kernel, dim3((unsigned)((n + kT - 1) / kT)), dim3(kT), 0, s, D, ldd, n, M, perm, b,
                       eta);
    return hipGetLastError();
}

hipError_t launch_refit_grad(const float* D, int64_t ldd, int64_t n, int M, const int32_t* perm, const double* r,
                             const double* w, double* rs, double* part, double* csum, double* g, hipStream_t s)
{
    if (ldd < refit_ld(n)) return hipErrorInvalidValue;
    const int nch = scan_chunks(n);
    hipLaunchKernelGGL(sort_r_kernel, dim3(grid_for(n)), dim3(kT), 0, s, perm, r, n, rs);
    hipLaunchKernelGGL(refit_sums_kernel, dim3(nch, (M + kSumCols - 1) / kSumCols), dim3(kT), 0, s, D, ldd, n, M, rs, w,
                       nch, part, csum);
    hipLaunchKernelGGL(refit_sum_kernel, dim3((M + kT / kWave - 1) / (kT / kWave)), dim3(kT), 0, s, part, nch, M, g);
    return hipGetLastError();
}

// Chunks of each kind of tile in proportion to what a step of it costs, so that
// every workgroup takes the same time, in all at most two workgroups of four
// wavefronts per CU: one round.  A step costs its wavefronts' blocks (16 for a tile
// above the diagonal, 9 for one on it) plus the loads, barriers and LDS writes,
// about kGramStep blocks' time: the two terms at 400,000 x 344 took 1324 and 312 us
// with as many chunks for every tile, 1379 and 308 in proportion to the blocks
// alone, 1110 and 266 with 10 (1129 and 266 with 20, 1163 and 265 with 40).
constexpr int kGramStep = 10;
GramPlan gram_plan(int64_t rows, int M)
{
    const int nt1 = (M - 1) / kGT, last = (M - nt1 * kGT + 15) / 16;
    const int cf = 16 + kGramStep, ce = 2 * last + kGramStep, cd = 9 + kGramStep,
              cl = (last * (last + 1) / 2 + 3) / 4 + kGramStep;
    const int total = nt1 * (nt1 - 1) / 2 * cf + nt1 * (ce + cd) + cl;
    const int64_t cap = max((int64_t)1, min((int64_t)kGramChunks, rows / 1024));
    auto chunks = [&](int cost) { return (int)max((int64_t)1, min(cap, (int64_t)(512 * cost / total))); };
    return GramPlan{chunks(cf), chunks(ce), chunks(cd), chunks(cl)};
}

static int gram_grid(const GramPlan& g, int M)
{
    const int nt1 = (M - 1) / kGT;
    return nt1 * (nt1 - 1) / 2 * g.full + nt1 * (g.edge + g.diag) + g.last;
}

size_t gram_part(int64_t rows, int M)
{
    const size_t S = min(M, kGT);
    return (size_t)gram_grid(gram_plan(rows, M), M) * S * S;
}

int scan_chunks(int64_t n) { return (int)max((int64_t)1, (n + kScanChunk - 1) / kScanChunk); }

hipError_t launch_refit_hessian(const RefitHess& h, hipStream_t s)
{
    const int M = h.M;
    if (M < 1 || M > kMaxRefit || h.ldd < refit_ld(h.n) || h.ldp < refit_ld(h.G)) return hipErrorInvalidValue;
    const GramPlan g1 = gram_plan(h.n, M), g2 = gram_plan(h.G, M);
    const int nch = scan_chunks(h.n);
    hipLaunchKernelGGL(hess_weight_kernel, dim3(grid_for(h.ldd)), dim3(kT), 0, s, h.perm, h.ev, h.r, h.n, h.ldd,
                       h.wt);
    hipLaunchKernelGGL((gram_kernel<float>), dim3(gram_grid(g1, M)), dim3(kT), 0, s, h.D, h.ldd, h.n, M, h.wt, g1,
                       h.part1);
    hipLaunchKernelGGL(scan_p_kernel, dim3(nch, M / kScanCols + 1), dim3(kT), 0, s, h.D, h.ldd, h.n, M, h.w, h.csum, nch, h.egidx,
                       h.G, h.ldp, h.P);
    hipLaunchKernelGGL(event_weight_kernel, dim3(grid_for(h.ldp)), dim3(kT), 0, s, h.P + (int64_t)M * h.ldp, h.egcnt,
                       h.G, h.ldp, h.wg);
    hipLaunchKernelGGL((gram_kernel<double>), dim3(gram_grid(g2, M)), dim3(kT), 0, s, h.P, h.ldp, h.G, M, h.wg, g2,
                       h.part2);
    hipLaunchKernelGGL(gram_reduce_kernel, dim3(grid_for((int64_t)M * M)), dim3(kT), 0, s, h.part1, g1, h.part2,
                       g2, M, h.H);
    return hipGetLastError();
}

hipError_t launch_chol(double* A, int M, double* diag, int* ok, hipStream_t s)
{
    if (M < 1 || M > kMaxRefit) return hipErrorInvalidValue;
    const int nb = (M + kCB - 1) / kCB;
    for (int J = 0; J < nb; ++J) {
        hipLaunchKernelGGL(chol_panel_kernel, dim3(nb - J), dim3(kWave), 0, s, A, M, J, diag, ok);
        const int nt = nb - J - 1;
        if (nt > 0)
            hipLaunchKernelGGL(chol_update_kernel, dim3(nt * (nt + 1) / 2 + 1), dim3(kT), 0, s, A, M, J, diag);
    }
    return hipGetLastError();
}

hipError_t launch_chol_solve(const double* L, int M, const double* g, double* x, hipStream_t s)
{
    if (M < 1 || M > kMaxRefit) return hipErrorInvalidValue;
    hipLaunchKernelGGL(chol_solve_kernel, dim3(1), dim3(kT), 0, s, L, M, g, x);
    return hipGetLastError();
}

hipError_t launch_wald(const double* L, int M, const double* b, double* se, double* pval, hipStream_t s)
{
    if (M < 1 || M > kMaxRefit) return hipErrorInvalidValue;
    hipLaunchKernelGGL(wald_kernel, dim3(M), dim3(kT), 0, s, L, M, b, se, pval);
    return hipGetLastError();
}

hipError_t launch_axpy(const double* b, const double* d, double t, int M, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(axpy_kernel, dim3((M + kT - 1) / kT), dim3(kT), 0, s, b, d, t, M, out);
    return hipGetLastError();
}

hipError_t launch_entry(const float* path, int L, int64_t ptot, int64_t p, int32_t* entry, float* coef, hipStream_t s)
{
    hipLaunchKernelGGL(entry_kernel, dim3(grid_for(p)), dim3(kT), 0, s, path, L, ptot, p, entry, coef);
    return hipGetLastError();
}

}  // namespace cox
