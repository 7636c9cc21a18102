// nmf.hip -- nonnegative matrix factorisation X ~ V W (Section 5.1) on one GPU,
// and its C ABI (include/nmf.h).
//
// X is m x n FP32, row-major (row i at X + i * ldx), borrowed.  The factors are
// stored as the paper's loop stores them, V' (r x m) and W (r x n), row-major,
// in FP64: they are small (r (m + n) doubles) and every product with X is
// formed and summed in FP64, so the only rounding is in the order of the sums.
//
// One iteration (Section 5.1, the loop's order):
//   W X'   (r x m)  nmf_wxt_kernel: workgroups over (256 or 128 rows of X, a
//                   split of the columns); a step's X tile of 32 columns and
//                   r x 32 W tile pass through LDS into FP64 matrix-core
//                   tiles, the next step's tiles loading into registers
//                   meanwhile.  nmf_reduce_gram_kernel adds the split partials.
//   W W'   (r x r)  the same launch, one workgroup per entry of the upper
//                   triangle, fixed-order reduction.
//   V' <- update    nmf_update_kernel, 4 threads per column of V': the r x r
//                   product with W W', then the multiplicative update
//                   V .* (X W') ./ (V W W' + eps) or the projected step
//                   max(0, V - sigma (V W W' - X W')), sigma = 1/(2||W W'||_F^2 + eps).
//   V' X   (r x n)  nmf_vtx_kernel: workgroups over (256 or 128 columns of X, a
//                   split of the rows); an X tile of 32 rows and the r x 32 V'
//                   tile, the same way.
//   V' V   (r x r), then the W update the same way with tau = 1/(2||V'V||_F^2 + eps).
// Both passes over X read it once each; the r x r products and the updates
// are O(r^2 (m + n)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "cox.h"
#include "device_common.h"
#include "nmf.h"

namespace cox {
namespace {

constexpr int kT = 256;
constexpr int kTJ = 32;  // columns of X per LDS step of W X'
constexpr int kTI = 32;  // rows of X per LDS step of V' X

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

// Both passes run on the FP64 matrix cores with v_mfma_f64_4x4x4f64, four
// independent 4 x 4 x 4 products: per lane, block l / 4 mod 4 holds A (row l % 4,
// k l / 16), B (k l / 16, column l % 4) and D (row l / 16, column l % 4).  Every
// block takes the same four rows of the factor as A, so an instruction multiplies
// 4 rank rows by 16 rows (or columns) of X, lane % 16, over 4 steps of the inner
// dimension, and the rank is padded to QT quads of 4.  v_mfma_f64_16x16x4f64 does
// 4 times the work an instruction, but sustained 44 TFLOP/s here, 31 with one
// wavefront on a SIMD, against 72 and 67, and pads the rank to 16 (r = 20 did the
// work of 32).  At 10,000 x 10,000, r = 20, W X' took 153 us and V' X 148 with it;
// they take 127 and 120 (r = 5: 91 and 74; r = 60: 283 and 260).  Reading X alone
// takes 82 us at the rate of a large copy and the products at r = 60 167 us at
// 72 TFLOP/s: a pass is bound by X up to about r = 20 and by the matrix cores, fed
// through LDS, above.
__device__ __forceinline__ double mfma_f64(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// N tiles of 16 rows (or columns) of X per wavefront: 4 up to rank 32, 2 above, where
// 4 would take the accumulators past two wavefronts per SIMD (at 10,000 x 10,000, r = 60
// one wavefront per SIMD made a pass 315 us).  A workgroup of 4 wavefronts owns 64
// times as many.
constexpr int n_tiles(int QT) { return QT <= 8 ? 4 : 2; }
int rows_per_wg(int r) { return 64 * n_tiles((r + 3) / 4); }

// LDS strides of the tiles.  A read of X takes 16 rows (or columns) by 4 inner
// positions, one of a factor 4 rows by 4 positions for every block.  With rows of
// 36 floats for the X tile of W X', 16 past a multiple of 64 floats for that of
// V' X and 36 doubles for a factor tile, a read's addresses fall on distinct banks.
constexpr int kXRow = kTJ + 4;
template <int NT>
constexpr int x_col() { return 64 * NT + 16; }
constexpr int kFRow = 36;
static_assert(kTJ <= kFRow && kTI <= kFRow, "a factor tile's row holds a step");

// part[split][a][i] = sum over the split's columns j of W[a][j] X[i][j]:
// M = a (the rank), N = i (64 NT rows of X per workgroup), K = j.  VEC: rows of X and
// of W start 16-byte aligned (X aligned, ldx a multiple of 4; W aligned, n even),
// and whole 16-byte pieces are loaded.
template <int QT, bool VEC>
__global__ __launch_bounds__(kT, 2) void nmf_wxt_kernel(const float* __restrict__ X, int64_t m, int64_t n, int64_t ldx,
                                                     int r, const double* __restrict__ W, int64_t cols,
                                                     double* __restrict__ part)
{
    constexpr int R = 4 * QT, NT = n_tiles(QT), ROWS = 64 * NT;
    __shared__ __attribute__((aligned(16))) float Xs[ROWS][kXRow];
    __shared__ __attribute__((aligned(16))) double Ws[R][kFRow];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * ROWS;
    const int64_t j0 = (int64_t)blockIdx.y * cols, j1 = min(n, j0 + cols);
    double acc[QT][NT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[qt][nt] = 0.0;
    // the next step's tiles are loaded into registers while the current one is
    // multiplied out of LDS
    constexpr int XE = ROWS * kTJ / (4 * kT);
    constexpr int WE = (R * kTJ / 2 + kT - 1) / kT;  // pairs of W
    float4 xr[XE];
    double2 wr[WE];
    auto fetch = [&](int64_t js) {
#pragma unroll
        for (int e = 0; e < XE; ++e) {
            const int li = threadIdx.x + kT * e;
            const int64_t i = i0 + li / (kTJ / 4), j = js + (li % (kTJ / 4)) * 4;
            const float* x = X + i * ldx + j;
            if (VEC && i < m && j + 4 <= j1)
                xr[e] = *reinterpret_cast<const float4*>(x);
            else
                xr[e] = make_float4(i < m && j < j1 ? x[0] : 0.0f, i < m && j + 1 < j1 ? x[1] : 0.0f,
                                    i < m && j + 2 < j1 ? x[2] : 0.0f, i < m && j + 3 < j1 ? x[3] : 0.0f);
        }
#pragma unroll
        for (int e = 0; e < WE; ++e) {
            const int li = threadIdx.x + kT * e;
            const int a = li / (kTJ / 2);
            const int64_t j = js + 2 * (li % (kTJ / 2));
            const double* w = W + (int64_t)a * n + j;
            const bool ok = li < R * kTJ / 2 && a < r;
            if (VEC && ok && j + 2 <= j1)
                wr[e] = *reinterpret_cast<const double2*>(w);
            else
                wr[e] = double2{ok && j < j1 ? w[0] : 0.0, ok && j + 1 < j1 ? w[1] : 0.0};
        }
    };
    if (j0 < j1) fetch(j0);
    for (int64_t js = j0; js < j1; js += kTJ) {
#pragma unroll
        for (int e = 0; e < XE; ++e) {
            const int li = threadIdx.x + kT * e;
            *reinterpret_cast<float4*>(&Xs[li / (kTJ / 4)][(li % (kTJ / 4)) * 4]) = xr[e];
        }
#pragma unroll
        for (int e = 0; e < WE; ++e) {
            const int li = threadIdx.x + kT * e;
            if (li < R * kTJ / 2) *reinterpret_cast<double2*>(&Ws[li / (kTJ / 2)][2 * (li % (kTJ / 2))]) = wr[e];
        }
        __syncthreads();
        if (js + kTJ < j1) fetch(js + kTJ);
#pragma unroll
        for (int kk = 0; kk < kTJ; kk += 4) {
            const int k = kk + (lane >> 4);
            double av[QT], bv[NT];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) av[qt] = Ws[qt * 4 + (lane & 3)][k];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bv[nt] = (double)Xs[wid * (16 * NT) + nt * 16 + (lane & 15)][k];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[qt][nt] = mfma_f64(av[qt], bv[nt], acc[qt][nt]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int a = qt * 4 + (lane >> 4);
            const int64_t i = i0 + wid * (16 * NT) + nt * 16 + (lane & 15);
            if (a < r && i < m) part[((int64_t)blockIdx.y * r + a) * m + i] = acc[qt][nt];
        }
}

// part[split][a][j] = sum over the split's rows i of Vt[a][i] X[i][j]:
// M = a, N = j (64 NT columns of X per workgroup), K = i
template <int QT>
__global__ __launch_bounds__(kT, 2) void nmf_vtx_kernel(const float* __restrict__ X, int64_t m, int64_t n, int64_t ldx,
                                                     int r, const double* __restrict__ Vt, int64_t rows,
                                                     double* __restrict__ part)
{
    constexpr int R = 4 * QT, NT = n_tiles(QT), COLS = 64 * NT, RPT = kT / COLS;
    __shared__ float Xs[kTI][x_col<NT>()];
    __shared__ double Vs[R][kFRow];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t jb = (int64_t)blockIdx.x * COLS;
    const int64_t i0 = (int64_t)blockIdx.y * rows, i1 = min(m, i0 + rows);
    double acc[QT][NT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[qt][nt] = 0.0;
    // the next step's tiles (kTI rows x COLS columns of X, one column per thread,
    // and the r x kTI tile of V') are loaded into registers during this one
    constexpr int VE = (R * kTI + kT - 1) / kT;
    const int row0 = RPT == 1 ? 0 : threadIdx.x / COLS, col = RPT == 1 ? threadIdx.x : threadIdx.x % COLS;
    float xr[kTI / RPT];
    double vr[VE];
    auto fetch = [&](int64_t is) {
#pragma unroll
        for (int ii = 0; ii < kTI / RPT; ++ii) {
            const int64_t i = is + RPT * ii + row0, j = jb + col;
            xr[ii] = (i < i1 && j < n) ? X[i * ldx + j] : 0.0f;
        }
#pragma unroll
        for (int e = 0; e < VE; ++e) {
            const int li = threadIdx.x + kT * e;
            const int a = li / kTI, ii = li % kTI;
            const int64_t i = is + ii;
            vr[e] = (li < R * kTI && a < r && i < i1) ? Vt[(int64_t)a * m + i] : 0.0;
        }
    };
    if (i0 < i1) fetch(i0);
    for (int64_t is = i0; is < i1; is += kTI) {
#pragma unroll
        for (int ii = 0; ii < kTI / RPT; ++ii) Xs[RPT * ii + row0][col] = xr[ii];
#pragma unroll
        for (int e = 0; e < VE; ++e) {
            const int li = threadIdx.x + kT * e;
            if (li < R * kTI) Vs[li / kTI][li % kTI] = vr[e];
        }
        __syncthreads();
        if (is + kTI < i1) fetch(is + kTI);
#pragma unroll
        for (int kk = 0; kk < kTI; kk += 4) {
            const int k = kk + (lane >> 4);
            double av[QT], bv[NT];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) av[qt] = Vs[qt * 4 + (lane & 3)][k];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bv[nt] = (double)Xs[k][wid * (16 * NT) + nt * 16 + (lane & 15)];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[qt][nt] = mfma_f64(av[qt], bv[nt], acc[qt][nt]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int a = qt * 4 + (lane >> 4);
            const int64_t j = jb + wid * (16 * NT) + nt * 16 + (lane & 15);
            if (a < r && j < n) part[((int64_t)blockIdx.y * r + a) * n + j] = acc[qt][nt];
        }
}

// num[t] = sum over splits of part[split][t], t < count, in split order: workgroup bx of nred
__device__ __forceinline__ void nmf_reduce_blk(const double* __restrict__ part, int nsplit, int64_t count,
                                               double* __restrict__ num, int bx, int nred)
{
    for (int64_t t = (int64_t)bx * kT + threadIdx.x; t < count; t += (int64_t)nred * kT) {
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < nsplit; ++q) s += part[(int64_t)q * count + t];
        num[t] = s;
    }
}

// G[a][b] = G[b][a] = sum_k F[a][k] F[b][k] over len, one workgroup per a <= b (idx)
__device__ __forceinline__ void nmf_gram_blk(const double* __restrict__ F, int r, int64_t len,
                                             double* __restrict__ G, int idx, double* sh)
{
    int a = 0;
    while (idx >= r - a) {
        idx -= r - a;
        ++a;
    }
    const int b = a + idx;
    const double *Fa = F + (int64_t)a * len, *Fb = F + (int64_t)b * len;
    double s = 0.0;
#pragma unroll 8
    for (int64_t k = threadIdx.x; k < len; k += kT) s += Fa[k] * Fb[k];
    s = block_sum256(s, sh);
    if (threadIdx.x == 0) {
        G[a * r + b] = s;
        G[b * r + a] = s;
    }
}

// The split sums of a pass over X and the Gram matrix of the factor it used, side
// by side in one launch (neither reads the other's output): workgroups below
// nred the sums, the others one entry of the Gram's upper triangle each.  Both are
// chains of loads: at 10,000 x 10,000, r = 20 they took 10 and 15 us one after the
// other, 12 us together.
__global__ __launch_bounds__(kT) void nmf_reduce_gram_kernel(const double* __restrict__ part, int nsplit,
                                                             int64_t count, double* __restrict__ num, int nred,
                                                             const double* __restrict__ F, int r, int64_t len,
                                                             double* __restrict__ G)
{
    __shared__ double sh[kT / kWave];
    if ((int)blockIdx.x < nred)
        nmf_reduce_blk(part, nsplit, count, num, blockIdx.x, nred);
    else
        nmf_gram_blk(F, r, len, G, blockIdx.x - nred, sh);
}

// One factor's update, kUP threads per column k of F (r x len), thread p
// taking the rows a = p, p + kUP, ...:
//   num[a][k]                                (X W' or V' X, the split sums)
//   den = (G F)[a][k]                        (W W' V' or V' V W)
//   multiplicative: F <- F num / (den + eps); APG: F <- max(0, F - step (den - num)),
//   step = 1 / (2 ||G||_F^2 + eps)
// Every old value of the workgroup's columns is read before any is written.
constexpr int kUC = 64;         // columns per workgroup of the update
constexpr int kUP = kT / kUC;   // threads per column
template <int R>
__global__ __launch_bounds__(kT) void nmf_update_kernel(double* __restrict__ F, int r, int64_t len,
                                                        const double* __restrict__ num_, const double* __restrict__ G,
                                                        int algo, double eps)
{
    __shared__ double Gs[R * R];
    __shared__ double sh[kT / kWave];
    for (int q = threadIdx.x; q < R * R; q += kT) {
        const int a = q / R, b = q % R;
        Gs[q] = (a < r && b < r) ? G[a * r + b] : 0.0;
    }
    __syncthreads();
    double step = 0.0;
    if (algo == 1) {
        double s2 = 0.0;
        for (int q = threadIdx.x; q < R * R; q += kT) s2 += Gs[q] * Gs[q];
        step = 1.0 / (2.0 * block_sum256(s2, sh) + eps);
    }
    const int p = threadIdx.x / kUC;
    const int64_t k = (int64_t)blockIdx.x * kUC + threadIdx.x % kUC;
    const bool live = k < len;
    double old[R];
#pragma unroll
    for (int a = 0; a < R; ++a) old[a] = (live && a < r) ? F[(int64_t)a * len + k] : 0.0;
    __syncthreads();
    if (!live) return;
    for (int a = p; a < r; a += kUP) {
        const double num = num_[(int64_t)a * len + k];
        double den = 0.0;
#pragma unroll
        for (int b = 0; b < R; ++b) den += Gs[a * R + b] * old[b];
        // only this thread writes row a of column k, so F[a][k] is still the old value
        const double oa = F[(int64_t)a * len + k];
        F[(int64_t)a * len + k] = algo == 0 ? oa * num / (den + eps) : fmax(0.0, oa - step * (den - num));
    }
}

// The objective's two inner products in one launch: workgroups below ninner sum
// F num over a run of the r len entries each, into part; the others one entry each
// of G = F F'.
__global__ __launch_bounds__(kT) void nmf_inner_gram_kernel(const double* __restrict__ F, int r, int64_t len,
                                                            const double* __restrict__ num, double* __restrict__ part,
                                                            int ninner, double* __restrict__ G)
{
    __shared__ double sh[kT / kWave];
    if ((int)blockIdx.x >= ninner) {
        nmf_gram_blk(F, r, len, G, blockIdx.x - ninner, sh);
        return;
    }
    const int64_t m = (int64_t)r * len, per = (m + ninner - 1) / ninner;
    const int64_t t0 = (int64_t)blockIdx.x * per, t1 = min(m, t0 + per);
    double s = 0.0;
    for (int64_t t = t0 + threadIdx.x; t < t1; t += kT) s += F[t] * num[t];
    s = block_sum256(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// partial sums of X_ij^2 per row block, then their sum in a fixed order
__global__ __launch_bounds__(kT) void nmf_xnorm_kernel(const float* __restrict__ X, int64_t m, int64_t n,
                                                       int64_t ldx, double* __restrict__ part)
{
    __shared__ double sh[kT / kWave];
    const int64_t i = blockIdx.x;
    double s = 0.0;
    for (int64_t j = threadIdx.x; j < n; j += kT) {
        const double x = X[i * ldx + j];
        s += x * x;
    }
    s = block_sum256(s, sh);
    if (threadIdx.x == 0) part[i] = s;
}

__global__ __launch_bounds__(kT) void nmf_sum_kernel(const double* __restrict__ v, int64_t len,
                                                     double* __restrict__ out)
{
    __shared__ double sh[kT / kWave];
    double s = 0.0;
    for (int64_t k = threadIdx.x; k < len; k += kT) s += v[k];
    s = block_sum256(s, sh);
    if (threadIdx.x == 0) out[0] = s;
}

// f = ||X||^2 - 2 <W, V'X> + <V'V, W W'>, the middle term from its ninner <= kT parts
constexpr int kInner = 256;
static_assert(kInner <= kT, "one thread per part");
__global__ __launch_bounds__(kT) void nmf_objective_kernel(const double* __restrict__ scal,
                                                           const double* __restrict__ part, int ninner,
                                                           const double* __restrict__ VtV,
                                                           const double* __restrict__ WWt, int r,
                                                           double* __restrict__ f)
{
    __shared__ double sh[kT / kWave];
    const double inner = block_sum256((int)threadIdx.x < ninner ? part[threadIdx.x] : 0.0, sh);
    double c = 0.0;
    for (int q = threadIdx.x; q < r * r; q += kT) c += VtV[q] * WWt[q];
    c = block_sum256(c, sh);
    if (threadIdx.x == 0) f[0] = scal[0] - 2.0 * inner + c;
}

inline unsigned grid_for(int64_t m) { return (unsigned)min((int64_t)8192, max((int64_t)1, (m + kT - 1) / kT)); }

}  // namespace
}  // namespace cox

using namespace cox;

struct nmf_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    const float* X = nullptr;
    int64_t m = 0, n = 0, ldx = 0;
    int r = 0;
    int ns_wxt = 1, ns_vtx = 1;
    int64_t cols = 0, rows = 0;
    double *part = nullptr, *num = nullptr, *WWt = nullptr, *VtV = nullptr, *scal = nullptr, *xpart = nullptr, *ipart = nullptr;
    std::vector<void*> allocs;
    std::string err;
    bool timing = false;
    std::vector<hipEvent_t> tev[2];
    double tms[2] = {};
    int64_t tcount[2] = {};
};

namespace {

cox_status nfail(nmf_ctx* c, cox_status s, const std::string& msg)
{
    if (c) c->err = msg;
    return s;
}

#define NCHK(expr, what)                                                                              \
    do {                                                                                              \
        hipError_t _e = (expr);                                                                       \
        if (_e != hipSuccess) return nfail(c, COX_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(_e)); \
    } while (0)

void nmf_release(nmf_ctx* c)
{
    for (int ph = 0; ph < 2; ++ph) {
        for (hipEvent_t e : c->tev[ph]) (void)hipEventDestroy(e);
        c->tev[ph].clear();
    }
    for (void* p : c->allocs) (void)hipFree(p);
    c->allocs.clear();
}

template <class T>
bool nalloc(nmf_ctx* c, T** out, size_t count)
{
    void* p = nullptr;
    if (hipMalloc(&p, std::max<size_t>(count, 1) * sizeof(T)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    c->allocs.push_back(p);
    *out = static_cast<T*>(p);
    return true;
}

void nmark(nmf_ctx* c, int ph)
{
    if (!c->timing) return;
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    (void)hipEventRecord(e, c->stream);
    c->tev[ph].push_back(e);
}

// the rows of X and of W start 16-byte aligned: W X' loads whole 16-byte pieces
bool nmf_aligned(const nmf_ctx* c, const double* W)
{
    return reinterpret_cast<uintptr_t>(c->X) % 16 == 0 && c->ldx % 4 == 0 && c->n % 2 == 0 &&
           reinterpret_cast<uintptr_t>(W) % 16 == 0;
}

// num (r x len) from the split partials, G (r x r) from the factor F (r x flen)
void nmf_reduce_gram(nmf_ctx* c, int nsplit, int64_t len, const double* F, int64_t flen, double* G)
{
    const int64_t count = (int64_t)c->r * len;
    const unsigned nred = grid_for(count), ngram = (unsigned)(c->r * (c->r + 1) / 2);
    hipLaunchKernelGGL(nmf_reduce_gram_kernel, dim3(nred + ngram), dim3(kT), 0, c->stream, c->part, nsplit, count,
                       c->num, (int)nred, F, c->r, flen, G);
}

template <int QT>
void nmf_vtx_gram(nmf_ctx* c, const double* Vt)
{
    const unsigned gn = (unsigned)((c->n + 64 * n_tiles(QT) - 1) / (64 * n_tiles(QT)));
    nmark(c, 1);
    hipLaunchKernelGGL(nmf_vtx_kernel<QT>, dim3(gn, c->ns_vtx), dim3(kT), 0, c->stream, c->X, c->m, c->n, c->ldx, c->r,
                       Vt, c->rows, c->part);
    nmark(c, 1);
    nmf_reduce_gram(c, c->ns_vtx, c->n, Vt, c->m, c->VtV);
}

template <int R>
void nmf_update(nmf_ctx* c, double* F, int64_t len, const double* G, int algo, double eps)
{
    hipLaunchKernelGGL(nmf_update_kernel<R>, dim3((unsigned)((len + kUC - 1) / kUC)), dim3(kT), 0, c->stream, F, c->r,
                       len, c->num, G, algo, eps);
}

template <int QT>
hipError_t nmf_iteration(nmf_ctx* c, int algo, double eps, double* Vt, double* W)
{
    constexpr int R = (4 * QT + 15) / 16 * 16;  // the update's rank, padded to 16
    const unsigned gm = (unsigned)((c->m + 64 * n_tiles(QT) - 1) / (64 * n_tiles(QT)));
    nmark(c, 0);
    if (nmf_aligned(c, W))
        hipLaunchKernelGGL((nmf_wxt_kernel<QT, true>), dim3(gm, c->ns_wxt), dim3(kT), 0, c->stream, c->X, c->m, c->n,
                           c->ldx, c->r, W, c->cols, c->part);
    else
        hipLaunchKernelGGL((nmf_wxt_kernel<QT, false>), dim3(gm, c->ns_wxt), dim3(kT), 0, c->stream, c->X, c->m, c->n,
                           c->ldx, c->r, W, c->cols, c->part);
    nmark(c, 0);
    nmf_reduce_gram(c, c->ns_wxt, c->m, W, c->n, c->WWt);
    nmf_update<R>(c, Vt, c->m, c->WWt, algo, eps);
    nmf_vtx_gram<QT>(c, Vt);
    nmf_update<R>(c, W, c->n, c->VtV, algo, eps);
    return hipGetLastError();
}

// iters iterations, or V'X and V'V alone, with the kernels of rank quads QT = ceil(r / 4) <= 16
template <int QT = 1>
hipError_t nmf_dispatch(nmf_ctx* c, int algo, double eps, double* Vt, double* W, int iters, bool vtx_only)
{
    if constexpr (QT < NMF_MAX_RANK / 4) {
        if (c->r > 4 * QT) return nmf_dispatch<QT + 1>(c, algo, eps, Vt, W, iters, vtx_only);
    }
    if (vtx_only) {
        nmf_vtx_gram<QT>(c, Vt);
        return hipGetLastError();
    }
    for (int k = 0; k < iters; ++k) {
        const hipError_t e = nmf_iteration<QT>(c, algo, eps, Vt, W);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

extern "C" {

cox_status nmf_setup(nmf_ctx** out, const float* X, int64_t m, int64_t n, int64_t ldx, int32_t r, void* hip_stream)
{
    if (!out) return COX_ERR_INVALID_ARG;
    *out = nullptr;
    if (!X || m < 1 || n < 1 || ldx < n || r < 1 || r > NMF_MAX_RANK || m >= (1LL << 31) || n >= (1LL << 31))
        return COX_ERR_INVALID_ARG;
    nmf_ctx* c = new (std::nothrow) nmf_ctx;
    if (!c) return COX_ERR_OUT_OF_MEMORY;
    c->stream = static_cast<hipStream_t>(hip_stream);
    if (hipGetDevice(&c->device) != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return COX_ERR_DEVICE;
    }
    c->X = X;
    c->m = m;
    c->n = n;
    c->ldx = ldx;
    c->r = r;
    // split the inner dimension so each pass has several workgroups per CU
    const int64_t rw = rows_per_wg(r), gm = (m + rw - 1) / rw, gn = (n + rw - 1) / rw;
    c->ns_wxt = (int)std::max<int64_t>(1, std::min<int64_t>((n + kTJ - 1) / kTJ, (1024 + gm - 1) / gm));
    c->ns_vtx = (int)std::max<int64_t>(1, std::min<int64_t>((m + kTI - 1) / kTI, (1024 + gn - 1) / gn));
    c->cols = ((n + c->ns_wxt - 1) / c->ns_wxt + kTJ - 1) / kTJ * kTJ;
    c->ns_wxt = (int)((n + c->cols - 1) / c->cols);
    c->rows = ((m + c->ns_vtx - 1) / c->ns_vtx + kTI - 1) / kTI * kTI;
    c->ns_vtx = (int)((m + c->rows - 1) / c->rows);
    const size_t pmax = std::max((size_t)c->ns_wxt * r * m, (size_t)c->ns_vtx * r * n);
    if (!(nalloc(c, &c->part, pmax) && nalloc(c, &c->num, (size_t)r * std::max(m, n)) &&
          nalloc(c, &c->WWt, (size_t)r * r) && nalloc(c, &c->VtV, (size_t)r * r) &&
          nalloc(c, &c->scal, 4) && nalloc(c, &c->xpart, m) && nalloc(c, &c->ipart, kInner))) {
        nmf_release(c);
        delete c;
        return COX_ERR_OUT_OF_MEMORY;
    }
    // ||X||_F^2 once, for the objective
    hipLaunchKernelGGL(nmf_xnorm_kernel, dim3((unsigned)m), dim3(kT), 0, c->stream, X, m, n, ldx, c->xpart);
    hipLaunchKernelGGL(nmf_sum_kernel, dim3(1), dim3(kT), 0, c->stream, c->xpart, m, c->scal);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(c->stream) != hipSuccess) {
        (void)hipGetLastError();
        nmf_release(c);
        delete c;
        return COX_ERR_DEVICE;
    }
    *out = c;
    return COX_OK;
}

cox_status nmf_destroy(nmf_ctx* c)
{
    if (!c) return COX_OK;
    (void)hipSetDevice(c->device);
    (void)hipStreamSynchronize(c->stream);
    nmf_release(c);
    delete c;
    return COX_OK;
}

cox_status nmf_last_error(const nmf_ctx* c, char* buf, size_t len)
{
    if (!c || !buf || len == 0) return COX_ERR_INVALID_ARG;
    const size_t k = std::min(len - 1, c->err.size());
    std::memcpy(buf, c->err.data(), k);
    buf[k] = '\0';
    return COX_OK;
}

cox_status nmf_run(nmf_ctx* c, int32_t algo, int32_t iters, double eps, double* Vt, double* W, double* obj)
{
    if (!c) return COX_ERR_INVALID_ARG;
    c->err.clear();
    if (hipSetDevice(c->device) != hipSuccess) return nfail(c, COX_ERR_DEVICE, "hipSetDevice failed");
    if ((algo != NMF_MULTIPLICATIVE && algo != NMF_APG) || iters < 0 || !(eps >= 0) || !std::isfinite(eps) || !Vt ||
        !W)
        return nfail(c, COX_ERR_INVALID_ARG, "bad nmf_run arguments");
    NCHK(nmf_dispatch(c, algo, eps, Vt, W, iters, false), "NMF iteration");
    if (obj) {
        const int r = c->r;
        // V'X and V'V of the final V are still in the workspace after an
        // iteration; with none, form them
        if (iters == 0) NCHK(nmf_dispatch(c, algo, eps, Vt, W, 0, true), "V'X");
        const int ninner = (int)std::min<int64_t>(kInner, ((int64_t)r * c->n + 1023) / 1024);
        hipLaunchKernelGGL(nmf_inner_gram_kernel, dim3((unsigned)(ninner + r * (r + 1) / 2)), dim3(kT), 0, c->stream, W,
                           r, c->n, c->num, c->ipart, ninner, c->WWt);
        hipLaunchKernelGGL(nmf_objective_kernel, dim3(1), dim3(kT), 0, c->stream, c->scal, c->ipart, ninner, c->VtV,
                           c->WWt, r, c->scal + 2);
        NCHK(hipGetLastError(), "objective");
        NCHK(hipMemcpyAsync(obj, c->scal + 2, sizeof(double), hipMemcpyDeviceToHost, c->stream), "objective");
        NCHK(hipStreamSynchronize(c->stream), "synchronise");
        if (!std::isfinite(*obj)) return nfail(c, COX_ERR_NUMERIC, "non-finite objective");
    }
    return COX_OK;
}

cox_status nmf_timing_enable(nmf_ctx* c, int32_t enable)
{
    if (!c) return COX_ERR_INVALID_ARG;
    NCHK(hipStreamSynchronize(c->stream), "synchronise");
    for (int ph = 0; ph < 2; ++ph) {
        for (hipEvent_t e : c->tev[ph]) (void)hipEventDestroy(e);
        c->tev[ph].clear();
        c->tms[ph] = 0;
        c->tcount[ph] = 0;
    }
    c->timing = enable != 0;
    return COX_OK;
}

cox_status nmf_timing_read(nmf_ctx* c, int32_t phase, double* total_ms, int64_t* count)
{
    if (!c || phase < 0 || phase > 1 || !total_ms) return COX_ERR_INVALID_ARG;
    NCHK(hipStreamSynchronize(c->stream), "synchronise");
    auto& ev = c->tev[phase];
    for (size_t q = 0; q + 1 < ev.size(); q += 2) {
        float ms = 0;
        NCHK(hipEventElapsedTime(&ms, ev[q], ev[q + 1]), "event time");
        c->tms[phase] += ms;
        c->tcount[phase] += 1;
    }
    for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    ev.clear();
    *total_ms = c->tms[phase];
    if (count) *count = c->tcount[phase];
    return COX_OK;
}

}  // extern "C"
