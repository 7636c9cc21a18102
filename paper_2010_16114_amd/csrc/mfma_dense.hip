// mfma_dense.hip -- eta = X C for B > 8 coefficient vectors over allele counts, to
// FP64 accuracy, in one pass over X per 32 vectors on the int8 matrix cores.
//
// Each coefficient is taken as c = q0 R0 + q1 R1 + q2 R2 + rest with integers
// |R| <= 2^22 (R1 is what R0's rounding leaves, on a scale 2^23 times finer, and so
// on): q0_b = max_j |c_bj| / 2^22, q1 = 2^-23 q0, q2 = 2^-46 q0, rest at most
// 2^-69 max|c_b|.  Every R goes as three signed int8 limbs (mfma.hip), so one
// read of X meets nine limb columns per vector; the integer sums are exact (over more
// than kMfmaMaxSum columns they are taken in shares, mfma_plan.h), and
// eta = q0 S0 + q1 S1 + q2 S2 is three roundings.
//
// Up to 32 vectors go in one launch (48 and 64 in two, each reading X).  A
// workgroup of 8 wavefronts owns SUB subjects and every vector of its launch:
// wavefront (s, g) takes 64 subjects and the 16 vectors of group g, all nine limbs
// of each (4 x 9 accumulator tiles of 16 x 16); SUB = 256 with two groups, 512
// with one.  A stage is 64 columns: its G tile (SUB subjects of each, decoded to
// counts) and its D tile (nine limbs of every vector) go through LDS, three stages
// of them, and every wavefront loads and stores a share of both.  While stage t is
// computed, stage t + 2 is stored and D of stage t + 3 and X of stage t + 4 are
// loaded.  Of the two wavefronts on a SIMD one stores before its matrix-core work
// and the other after, so that the matrix cores have work meanwhile.  Blocks of
// neighbouring subjects run on one XCD, whose L2 then serves the second half of a
// 128-byte line that two blocks share.
//
// What bounds it is the path of a compute unit's loads: every byte of G and D
// comes through it at about 17 bytes a cycle, and the accumulators limit how many
// subjects share a D tile.  At 200,000 x 50,000: 1.71 ms for 16 vectors (5.8 TB/s),
// 2.6 for 32, 5.2 for 64 (6.4 in one launch with 128 subjects to a workgroup, 45 KB
// a stage; 6.3 as three passes of the eta update's kernel, one per R, which take
// that for any number of vectors above 16).
#include "device_common.h"
#include "mfma.h"
#include "mfma_dev.h"

namespace cox {
namespace {

constexpr int kT = 256;
constexpr int kSets = 3;                  // R0, R1, R2
constexpr int kLC = kSets * kLimbs;       // limb columns per vector
constexpr double kFiner = 0x1p-23;        // scale of each R below the one before
constexpr int kDT = 512;                  // threads of the product kernel
constexpr int kWidth = 32;                // vectors per launch

// Largest |c_b| over a tile of 4096 columns; flag[b] = 1 (cleared by the caller)
// if some c_bj is a NaN or an infinity.
__global__ __launch_bounds__(kT) void dense_max_kernel(const double* __restrict__ coef, int64_t p,
                                                       double* __restrict__ part, int ntile,
                                                       int32_t* __restrict__ flag)
{
    __shared__ double sh[kT / 64];
    const int b = blockIdx.y;
    const int64_t j1 = min(p, (int64_t)(blockIdx.x + 1) * 4096);
    double mx = 0.0;
    bool bad = false;
    for (int64_t j = (int64_t)blockIdx.x * 4096 + threadIdx.x; j < j1; j += kT) {
        const double v = coef[(int64_t)b * p + j];
        mx = fmax(mx, fabs(v));
        bad |= !isfinite(v);
    }
    if (bad) flag[b] = 1;  // every writer stores 1
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) part[(int64_t)b * ntile + blockIdx.x] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

// The limbs of 16 columns of one vector per thread.  Each launch's vectors have
// an array of their own, one after another: [j / 16][limb column * width + b - b0]
// [j % 16], limb column 3 set + limb, width the launch's vectors rounded up to 16;
// columns p .. round_up(p, 64) - 1 are zero.
__global__ __launch_bounds__(kT) void dense_quant_kernel(const double* __restrict__ coef, int64_t p,
                                                         const double* __restrict__ part, int ntile,
                                                         int8_t* __restrict__ dlimbs, int64_t dstride, int bpad,
                                                         double* __restrict__ dscale)
{
    const int b = blockIdx.y;
    double mx = 0.0;
    for (int t = threadIdx.x & 63; t < ntile; t += 64) mx = fmax(mx, part[(int64_t)b * ntile + t]);
    mx = wave_max(mx);
    const double q0 = mx > 0.0 ? mx / (double)(1 << kQBits) : 1.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) dscale[b] = q0;
    const int64_t u = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (u >= (p + 63) / 64 * 4) return;
    uint32_t o[kLC][4] = {};
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int64_t j = 16 * u + e;
        double v = j < p ? coef[(int64_t)b * p + j] : 0.0;
        double q = q0;
#pragma unroll
        for (int k = 0; k < kSets; ++k) {
            // a scale that underflows to zero leaves nothing to carry
            const double Rd = q > 0.0 ? rint(v / q) : 0.0;
            v = fma(-q, Rd, v);
            q *= kFiner;
            int d[3];
            split_limbs((int)Rd, d[0], d[1], d[2]);
#pragma unroll
            for (int l = 0; l < 3; ++l) o[3 * k + l][e >> 2] |= (uint32_t)(d[l] & 255) << (8 * (e & 3));
        }
    }
    const int b0 = b / kWidth * kWidth, width = min(kWidth, bpad - b0);
    int8_t* dst = dlimbs + dstride * kLC * b0 + (u * (kLC * width) + b - b0) * 16;
#pragma unroll
    for (int c = 0; c < kLC; ++c)
        *reinterpret_cast<uint4*>(dst + c * width * 16) = make_uint4(o[c][0], o[c][1], o[c][2], o[c][3]);
}

// NG groups of 16 vectors from a.b0 on; SUB subjects per block.  Blocks from a.nfull on are split a.ksplit ways over
// columns: their exact sums go to a.part ([share][block - nfull][subject][3][16 NG]),
// added by dense_sum_kernel.
template <int XT, int NG, int SUB>
__global__ __launch_bounds__(kDT, 2) void mfma_dense_kernel(MfmaDenseArgs a)
{
    constexpr int NS = SUB / 64;          // subject groups of a block
    static_assert(NS * NG == 8, "eight wavefronts cover the block");
    constexpr int SW = SUB / 4;           // dwords per column of the G tile
    constexpr int RB = SUB / 16;          // 16-byte chunks per column of the G tile
    constexpr int NCOL = 16 * NG * kLC;   // limb columns
    constexpr int DCH = 4 * NCOL;         // 16-byte chunks of D per stage
    constexpr int GPT = 64 * RB / kDT;    // chunks of G per thread
    constexpr int DPT = (DCH + kDT - 1) / kDT;
    static_assert(GPT * kDT == 64 * RB, "the G tile splits evenly");
    constexpr bool DALL = DCH % kDT == 0;
    // dword position of dword w of column c: the four 16-column groups of a fragment read hit distinct banks
    auto gpos = [](int c, int w) { return c * SW + (w ^ (((c >> 4) & 3) << 4)); };
    __shared__ __attribute__((aligned(16))) uint32_t sG[3][64 * SW];
    __shared__ v4i sD[3][DCH];

    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int ws = wid % NS, wg = wid / NS;  // subject group, vector group
    const int64_t n = a.n, p = a.p, ldx = a.ldx;
    const uint8_t* __restrict__ X = static_cast<const uint8_t*>(a.X);
    const int nstage = (int)((p + 63) / 64);
    int64_t blk = blockIdx.x;
    int t0 = 0, t1 = nstage, share = -1;
    if (blk >= a.nfull) {
        const int64_t v = blk - a.nfull;
        blk = a.nfull + v / a.ksplit;
        if (a.ksplit > 1) share = (int)(v % a.ksplit);
        t0 = (int)((int64_t)nstage * (v % a.ksplit) / a.ksplit);
        t1 = (int)((int64_t)nstage * (v % a.ksplit + 1) / a.ksplit);
    } else if (a.nfull % 8 == 0) {
        blk = (blk % 8) * (a.nfull / 8) + blk / 8;  // workgroups go to the 8 XCDs in turn
    }
    const int64_t i0 = blk * SUB;

    // this thread's G chunks (column of the stage, 16 subjects) and D chunks
    int gcol[GPT], gdst[GPT];
    int64_t grow[GPT];
#pragma unroll
    for (int k = 0; k < GPT; ++k) {
        const int ch = threadIdx.x + kDT * k;
        gcol[k] = ch / RB;
        grow[k] = i0 + 16 * (ch % RB);
        gdst[k] = gpos(gcol[k], 4 * (ch % RB));
    }
    const v4i* __restrict__ D = reinterpret_cast<const v4i*>(a.dlimbs);
    v4i gr[2][GPT], dr[DPT];
    // a column past p, or a chunk that starts at or after n, loads the start of X: the limbs of columns past p are
    // zero, and subjects past n reach only outputs that are never written
    auto fetch_g = [&](int t, v4i (&g)[GPT]) {
#pragma unroll
        for (int k = 0; k < GPT; ++k) {
            const int64_t col = (int64_t)t * 64 + gcol[k];
            g[k] = *reinterpret_cast<const v4i*>(X + (col < p && grow[k] < n ? col * ldx + grow[k] : 0));
        }
    };
    auto fetch_d = [&](int t) {
        const int64_t at = (int64_t)min(t, nstage - 1) * DCH;
#pragma unroll
        for (int k = 0; k < DPT; ++k)
            if (DALL || (int)threadIdx.x + kDT * k < DCH) dr[k] = D[at + threadIdx.x + kDT * k];
    };
    auto store = [&](int buf, const v4i (&g)[GPT]) {
#pragma unroll
        for (int k = 0; k < GPT; ++k) *reinterpret_cast<v4i*>(&sG[buf][gdst[k]]) = decode_a<XT>(g[k]);
#pragma unroll
        for (int k = 0; k < DPT; ++k)
            if (DALL || (int)threadIdx.x + kDT * k < DCH) sD[buf][threadIdx.x + kDT * k] = dr[k];
    };

    v4i acc[4][kLC];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int c = 0; c < kLC; ++c) acc[mt][c] = v4i{0, 0, 0, 0};
    const int xr = ws * 16 + (lane & 15);  // this lane's dword (4 subjects) within a column
    auto compute = [&](int buf) {
        // three limb columns' fragments are read while the three before are multiplied: one ahead left the chain of
        // LDS reads longer than the matrix-core work (1.27 us a stage of 64 columns, 0.6 us of it matrix cores)
        constexpr int BG = 3;
        const v4i* sb = &sD[buf][(lane >> 4) * NCOL + wg * 16 + (lane & 15)];
        v4i br[2][BG];
        uint32_t d[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) d[q][e] = sG[buf][gpos(16 * (lane >> 4) + 4 * q + e, xr)];
#pragma unroll
        for (int u = 0; u < BG; ++u) br[0][u] = sb[u * 16 * NG];
        __builtin_amdgcn_sched_barrier(0);
        v4i A[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t o[4];
            transpose4x4(d[q], o);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) A[mt][q] = (int)o[mt];
        }
#pragma unroll
        for (int g = 0; g < kLC / BG; ++g) {
            if (g + 1 < kLC / BG) {
#pragma unroll
                for (int u = 0; u < BG; ++u) br[(g + 1) & 1][u] = sb[((g + 1) * BG + u) * 16 * NG];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < BG; ++u)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    acc[mt][g * BG + u] =
                        __builtin_amdgcn_mfma_i32_16x16x64_i8(A[mt], br[g & 1][u], acc[mt][g * BG + u], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const bool early = wid < 4;
    int buf = 0;  // stage t's
    auto step = [&](int t, v4i (&g)[GPT]) {  // g holds X of stage t + 2, dr D of it
        const int b1 = buf == 2 ? 0 : buf + 1, b2 = b1 == 2 ? 0 : b1 + 1;
        if (!early) compute(buf);
        __builtin_amdgcn_sched_barrier(0);
        store(b2, g);
        fetch_d(t + 3);
        fetch_g(t + 4, g);
        __builtin_amdgcn_sched_barrier(0);
        if (early) compute(buf);
        buf = b1;
        __syncthreads();
    };

    fetch_g(t0, gr[0]);
    fetch_d(t0);
    fetch_g(t0 + 1, gr[1]);
    store(0, gr[0]);
    fetch_d(t0 + 1);
    fetch_g(t0 + 2, gr[0]);
    store(1, gr[1]);
    fetch_d(t0 + 2);
    fetch_g(t0 + 3, gr[1]);
    __syncthreads();
    int t = t0;
    for (; t + 1 < t1; t += 2) {
        step(t, gr[0]);
        step(t + 1, gr[1]);
    }
    if (t < t1) step(t, gr[0]);

    const int bl = wg * 16 + (lane & 15), b = a.b0 + bl;
    if (b >= a.B) return;
    const double q0 = a.dscale[b], q1 = q0 * kFiner, q2 = q1 * kFiner;
    const bool poison = a.nonfin[b] != 0;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int r = 64 * ws + 4 * mfma_c_row(lane, v) + mt;
            if (i0 + r >= n) continue;
            int64_t tot[kSets];
#pragma unroll
            for (int k = 0; k < kSets; ++k)
                tot[k] = (int64_t)acc[mt][3 * k][v] + 256 * (int64_t)acc[mt][3 * k + 1][v] +
                         65536 * (int64_t)acc[mt][3 * k + 2][v];
            if (share < 0) {
                const double e = fma(q2, (double)tot[2], fma(q1, (double)tot[1], q0 * (double)tot[0]));
                a.eta[(i0 + r) * a.bpad + b] = poison ? __builtin_nan("") : e;
            } else {
                long long* out = a.part + ((share * (a.nblk - a.nfull) + blk - a.nfull) * SUB + r) * (kSets * 16 * NG) + bl;
#pragma unroll
                for (int k = 0; k < kSets; ++k) out[k * 16 * NG] = tot[k];
            }
        }
}

// eta of the split blocks: the shares' exact sums added, then as above.
__global__ __launch_bounds__(kT) void dense_sum_kernel(MfmaDenseArgs a, int sub, int width)
{
    const int64_t i0 = a.nfull * sub, m = (a.n - i0) * width;
    const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (e >= m) return;
    const int64_t r = e / width;
    const int bl = (int)(e % width), b = a.b0 + bl;
    if (b >= a.B) return;
    const int64_t rows = (a.nblk - a.nfull) * sub;
    long long tot[kSets] = {};
#pragma unroll 4
    for (int s = 0; s < a.ksplit; ++s)
#pragma unroll
        for (int k = 0; k < kSets; ++k) tot[k] += a.part[((s * rows + r) * kSets + k) * width + bl];
    const double q0 = a.dscale[b], q1 = q0 * kFiner, q2 = q1 * kFiner;
    const double v = fma(q2, (double)tot[2], fma(q1, (double)tot[1], q0 * (double)tot[0]));
    a.eta[(i0 + r) * a.bpad + b] = a.nonfin[b] ? __builtin_nan("") : v;
}

template <int XT, int NG, int SUB>
hipError_t launch_ng(MfmaDenseArgs a, hipStream_t s)
{
    a.nblk = (a.n + SUB - 1) / SUB;
    const DensePlan d = dense_plan(a.nblk, (a.p + 63) / 64, a.ncu, (int64_t)SUB * kSets * 16 * NG, a.part_room);
    if (d.ksplit < 1) return hipErrorInvalidValue;
    a.nfull = d.nfull;
    a.ksplit = d.ksplit;
    hipLaunchKernelGGL((mfma_dense_kernel<XT, NG, SUB>), dim3((unsigned)(a.nfull + (a.nblk - a.nfull) * a.ksplit)),
                       dim3(kDT), 0, s, a);
    if (a.ksplit > 1) {
        const int64_t m = (a.n - a.nfull * SUB) * 16 * NG;
        hipLaunchKernelGGL(dense_sum_kernel, dim3((unsigned)((m + kT - 1) / kT)), dim3(kT), 0, s, a, SUB, 16 * NG);
    }
    return hipGetLastError();
}

template <int XT>
hipError_t launch_xt(MfmaDenseArgs a, hipStream_t s)
{
    const int8_t* limbs = a.dlimbs;
    hipError_t e = hipSuccess;
    for (a.b0 = 0; a.b0 < a.bpad && e == hipSuccess; a.b0 += kWidth) {
        a.dlimbs = limbs + a.dstride * kLC * a.b0;
        e = a.bpad - a.b0 >= kWidth ? launch_ng<XT, 2, 256>(a, s) : launch_ng<XT, 1, 512>(a, s);
    }
    return e;
}

}  // namespace

hipError_t launch_dense_quant(const double* coef, int64_t p, int B, double* dmaxp, int8_t* dlimbs, int64_t dstride,
                              int bpad, double* dscale, int32_t* nonfin, hipStream_t s)
{
    if (p < 1 || B < 1 || dstride % 64 || dstride < p || bpad < B || bpad % 16) return hipErrorInvalidValue;
    const int nt = (int)((p + 4095) / 4096);
    hipLaunchKernelGGL(dense_max_kernel, dim3(nt, B), dim3(kT), 0, s, coef, p, dmaxp, nt, nonfin);
    const int64_t chunks = (p + 63) / 64 * 4;
    hipLaunchKernelGGL(dense_quant_kernel, dim3((unsigned)((chunks + kT - 1) / kT), B), dim3(kT), 0, s, coef, p, dmaxp,
                       nt, dlimbs, dstride, bpad, dscale);
    return hipGetLastError();
}

hipError_t launch_mfma_dense(const MfmaDenseArgs& a, hipStream_t s)
{
    if (a.bpad < 16 || a.bpad > 64 || a.bpad % 16 || a.B > a.bpad || (a.part_room > 0 && !a.part))
        return hipErrorInvalidValue;
    return a.xt == XT_FP8 ? launch_xt<XT_FP8>(a, s) : launch_xt<XT_I8>(a, s);
}

}  // namespace cox
