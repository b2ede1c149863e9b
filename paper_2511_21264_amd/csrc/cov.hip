// Covariance adaptation and full-covariance sampling (Alg. 1: sampling from
// N(nu_m, Sigma_m); Eqs. mean_update and cov_update with the weights of
// Eq. s_formula).  A sequence is the n = 14 H vector of its joint velocities
// in step-major order (index 14 k + d), so Sigma is n x n, row-major, FP64.
//
//   cov_syrk_kernel    Sigma' = (1 - eta) Sigma + eta sum_j w_j D_j D_j^T / sum w
//                      + eps I with D_j = u_j - nu_{m+1}: one workgroup per
//                      32 x 32 lower tile, four or eight waves split the samples,
//                      FP64 MFMA 16x16x4 with the deviation and the weight
//                      formed in the operand load; each symmetric pair is
//                      written by one lane (so the update may run in place)
//   chol_*_kernel      blocked right-looking Cholesky in FP64, 32-wide block
//                      columns, one launch per block column: every trailing
//                      lower tile (r, c) forms the panel blocks A_rb L_bb^-T
//                      and A_cb L_bb^-T itself and subtracts their product
//                      (FP64 MFMA); the tile (r, r) also stores its panel block
//                      as the factor, and the workgroup of the next diagonal
//                      tile factors and inverts it in one wave's registers
//   sample_*_kernel    U = clip(nu + Z L^T, +-u_max): both factors as three
//                      bf16 parts in operand order, bf16 MFMA 16x16x32 over
//                      32 x 64 tiles, skipping the zero upper triangle of L
//
// MFMA 16x16x4 operand layout: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; result element v of lane l is D[4 (l / 16) + v][l % 16]
// for f32 and D[l / 16 + 4 v][l % 16] for f64 (measured on gfx950).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "team.h"

namespace mppi {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int CT = 32;  // covariance output tile edge
constexpr int CB = 32;  // Cholesky block edge

// t -> (row, col) of the t-th lower tile, enumerated row by row
__device__ __forceinline__ void tri_index(int t, int &row, int &col)
{
    int b = (int)((sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while (b * (b + 1) / 2 > t) --b;
    while ((b + 1) * (b + 2) / 2 <= t) ++b;
    row = b;
    col = t - b * (b + 1) / 2;
}

// Workgroups are dealt to the eight XCDs (each with its own L2) in turn by
// their index b; this maps b to a logical tile so that every XCD takes one
// contiguous range of tiles (a bijection on 0 .. nb - 1): tiles that share
// input rows then share an L2.
__device__ __forceinline__ int xcd_order(int b, int nb)
{
    const int x = b & 7, q = nb >> 3, r = nb & 7;
    return x * q + min(x, r) + (b >> 3);
}

__device__ __forceinline__ double wave_sum_f64(double x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

}  // namespace

// ------------------------------------------------------------ covariance update
constexpr int CG = 8;  // groups of four samples per wave and step

// CW: waves per tile.  Bound by issue: per group of four samples a wave's four
// FP64 MFMAs (64 cycles each) and its vector instructions, which run one after
// the other.  So indices past K or n are clamped instead of tested (their
// columns are not stored, their weight is 0) and offsets are 32-bit where they
// fit.  K = 1024, n = 896: 40.3 -> 37.4 us; K = 4096, n = 1400: 268 -> 233 us
// (17 TFLOP/s of the lower triangle).  What is left at n = 896 is the tail: 406 tiles on
// 256 CUs, so some CUs have two.
template <int CW, typename Off>
__global__ void __launch_bounds__(64 * CW) cov_syrk_kernel(CovArgs a)
{
    __shared__ double red[CW][CT][CT + 1];
    __shared__ double wred[CW];
    int bi, bl;
    tri_index(xcd_order(blockIdx.x, gridDim.x), bi, bl);  // consecutive rows of tiles share an XCD
    const int n = a.n, K = a.K;
    const int i0 = bi * CT, l0 = bl * CT;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    const int ia0 = min(i0 + r, n - 1), ia1 = min(i0 + r + 16, n - 1), lb0 = min(l0 + r, n - 1), lb1 = min(l0 + r + 16, n - 1);
    const double na0 = a.nu[ia0], na1 = a.nu[ia1], nl0 = a.nu[lb0], nl1 = a.nu[lb1];
    d4 c00 = {0.0, 0.0, 0.0, 0.0}, c01 = c00, c10 = c00, c11 = c00;
    double ws = 0.0;
    // wave wv takes the groups of four samples j0 = 4 wv, 4 wv + 4 CW, ...,
    // CG groups per step; the loads of step s + 1 are issued before the
    // products of step s.  Sample values do not wait on their weight: a
    // weightless sample's are dropped by a select afterwards (so a non-finite
    // entry in it still contributes nothing).
    float uc[CG][4], un[CG][4] = {};
    double wc[CG], wn[CG] = {};
    auto load = [&](int j0, float (&u4)[CG][4], double (&w2)[CG]) {
#pragma unroll
        for (int g = 0; g < CG; ++g) {
            const int j = j0 + 4 * CW * g + q, jc = min(j, K - 1);
            const double w = a.w[jc];
            w2[g] = j < K ? w : 0.0;
            const Off o = (Off)jc * (Off)n;
            u4[g][0] = a.U[o + (Off)ia0];
            u4[g][1] = a.U[o + (Off)ia1];
            u4[g][2] = a.U[o + (Off)lb0];
            u4[g][3] = a.U[o + (Off)lb1];
        }
    };
    load(4 * wv, uc, wc);
    for (int j0 = 4 * wv; j0 < K; j0 += 4 * CW * CG) {
        if (j0 + 4 * CW * CG < K) load(j0 + 4 * CW * CG, un, wn);
        bool any = false;
#pragma unroll
        for (int g = 0; g < CG; ++g) {
            ws += wc[g];  // on each of the 16 lanes that share the sample
            any = any || wc[g] != 0.0;
        }
        if (__ballot(any) != 0) {  // skipped when no group of the step carries weight
#pragma unroll
            for (int g = 0; g < CG; ++g) {
                const bool on = wc[g] != 0.0;
                const double x0 = on ? (double)uc[g][0] - na0 : 0.0, x1 = on ? (double)uc[g][1] - na1 : 0.0;
                const double y0 = on ? wc[g] * ((double)uc[g][2] - nl0) : 0.0;
                const double y1 = on ? wc[g] * ((double)uc[g][3] - nl1) : 0.0;
                c00 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y0, c00, 0, 0, 0);
                c01 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, y1, c01, 0, 0, 0);
                c10 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y0, c10, 0, 0, 0);
                c11 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, y1, c11, 0, 0, 0);
            }
        }
#pragma unroll
        for (int g = 0; g < CG; ++g) {
            wc[g] = wn[g];
#pragma unroll
            for (int e = 0; e < 4; ++e) uc[g][e] = un[g][e];
        }
    }
    if (r != 0) ws = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        red[wv][q + 4 * v][r] = c00[v];
        red[wv][q + 4 * v][16 + r] = c01[v];
        red[wv][16 + q + 4 * v][r] = c10[v];
        red[wv][16 + q + 4 * v][16 + r] = c11[v];
    }
    ws = wave_sum_f64(ws);
    if (lane == 0) wred[wv] = ws;
    __syncthreads();
    double wsum = wred[0];
#pragma unroll
    for (int w = 1; w < CW; ++w) wsum += wred[w];
    for (int e = threadIdx.x; e < CT * CT; e += 64 * CW) {
        const int ti = e / CT, tl = e % CT;
        const int i = i0 + ti, l = l0 + tl;
        if (i >= n || l >= n || (bi == bl && ti < tl)) continue;
        double g = red[0][ti][tl];
#pragma unroll
        for (int w = 1; w < CW; ++w) g += red[w][ti][tl];
        const double s_old = a.S_in[(long)i * n + l];
        // no weight at all (no finite cost): Sigma is kept, as the mean is
        double v = s_old;
        if (wsum > 0.0) {
            v = (1.0 - a.eta) * s_old + a.eta * (g / wsum);
            if (i == l) v += a.eps;
        }
        a.S_out[(long)i * n + l] = v;
        red[0][ti][tl] = v;  // read above by this thread only
    }
    __syncthreads();
    // the mirrored upper half, written along its rows
    for (int e = threadIdx.x; e < CT * CT; e += 64 * CW) {
        const int tl = e / CT, ti = e % CT;
        const int i = i0 + ti, l = l0 + tl;
        if (i >= n || l >= n || i == l || (bi == bl && ti < tl)) continue;
        a.S_out[(long)l * n + i] = red[0][ti][tl];
    }
}

void launch_cov_update(const CovArgs &a, hipStream_t s)
{
    const int nt = (a.n + CT - 1) / CT, tiles = nt * (nt + 1) / 2;
    const bool small = (long)a.K * a.n < (1l << 30);
    // up to a tile a CU (256), eight waves share it: two a SIMD, half the
    // samples each (K = 1000, n = 462: 21.9 us against 29.9 with four).  Past
    // that two tiles share a CU and eight waves only add to the reduction
    // (K = 256, n = 1400: 30.7 us against 28.3); at 128 samples or fewer four
    // waves have one step each already (K = 64, n = 280: 14.6 us either way).
    if (tiles <= 256 && a.K > 16 * CG) {
        // 22 tile rows at most (n <= 704), so K n stays below 2^30 up to K = 2^20
        static_assert(MPPI_MAX_K <= 1 << 20, "32-bit offsets of the eight-wave form");
        hipLaunchKernelGGL((cov_syrk_kernel<8, uint32_t>), dim3(tiles), dim3(512), 0, s, a);
    } else {
        if (small)
            hipLaunchKernelGGL((cov_syrk_kernel<4, uint32_t>), dim3(tiles), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((cov_syrk_kernel<4, long>), dim3(tiles), dim3(256), 0, s, a);
    }
}

// ------------------------------------------------------------------ Cholesky
__global__ void __launch_bounds__(256) chol_init_kernel(CholArgs a)
{
    const long n = a.n, N = n * n;
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
        const long i = e / n, l = e - i * n;
        if (l <= i) {
            a.A[e] = a.S[e];
        } else {
            a.L[e] = 0.0;
        }
    }
    if (a.reset_flag && blockIdx.x == 0 && threadIdx.x == 0) *a.flag = a.n;
}

// x of lane N of each row of 16 lanes, on all of them
template <int N>
__device__ __forceinline__ double row_bcast(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x150 + N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x150 + N, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// a[k] -= l bcast(l, lane k), e[k] -= m bcast(l, lane k) for k = K .. 15
template <int K>
__device__ __forceinline__ void rank1(double (&a)[16], double (&e)[16], double l, double m)
{
    if constexpr (K < 16) {
        const double lk = row_bcast<K>(l);
        a[K] = fma(-l, lk, a[K]);
        e[K] = fma(-m, lk, e[K]);
        rank1<K + 1>(a, e, l, m);
    }
}

// Columns J .. 15 of the factorization of a 16 x 16 block: lane r of each row
// of 16 lanes holds row r of the block (a) and a row e of its own that becomes
// e L^-T.  A pivot that is not positive and finite makes its column NaN.
template <int J>
__device__ __forceinline__ void factor16(double (&a)[16], double (&e)[16])
{
    if constexpr (J < 16) {
        const double id = rsqrt(row_bcast<J>(a[J]));
        a[J] *= id;
        e[J] *= id;
        rank1<J + 1>(a, e, a[J], e[J]);
        factor16<J + 1>(a, e);
    }
}

// Factor the diagonal block held in s (zero above the diagonal, the identity
// in rows and columns past nbk), invert it, and store the factor block of
// columns c0b.. into L and the inverse into Linv.  256 threads; x is scratch.
//
// A serial chain: pivot, reciprocal root, column, next pivot.  One wave runs
// it on two halves of 16, in registers, with broadcasts inside rows of 16
// lanes (no LDS and no barrier between columns), every row of lanes on the
// same block and each with 16 more rows that take the same column steps: the
// rows below it (lanes 0-15) and those of X^T = I L^-T (the others, X = L^-1).
// Between the halves L21 L21^T and X11^T L21^T leave the second one's rows, by
// FP64 MFMA.  The loop over the halves stays rolled: a launch runs this once,
// so code is fetched cold, and size is time.  n = 896 (28 blocks): 427 us with
// four waves on groups of four columns (30 KB of code) -> 326 us (6 KB), with
// the tile fetched along with its operands; both halves written out, 658 us.
__device__ void factor_block(double (*s)[CB + 1], double (*x)[CB + 1], int nbk, int c0b, const CholArgs &arg,
                             double *Linv)
{
    const int n = arg.n;
    for (int i = threadIdx.x; i < CB * CB; i += 256) x[i / CB][i % CB] = i / CB == i % CB ? 1.0 : 0.0;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x, r = lane & 15, g = lane >> 4;
        double *er = g == 0 ? s[16 + r] : x[16 * (min(g, 2) - 1) + r];
#pragma unroll 1
        for (int h = 0; h < CB; h += 16) {
            double a[16], e[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                a[k] = s[h + r][h + k];
                e[k] = er[h + k];
            }
            factor16<0>(a, e);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                s[h + r][h + k] = a[k];
                er[h + k] = e[k];
            }
            wave_lds_sync();
            if (h == 0) {
                d4 c, f;  // rows g + 4 v, column r
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    c[v] = s[16 + g + 4 * v][16 + r];
                    f[v] = 0.0;
                }
#pragma unroll
                for (int k = 0; k < 16; k += 4) {
                    const double l = s[16 + r][k + g];
                    c = __builtin_amdgcn_mfma_f64_16x16x4f64(-l, l, c, 0, 0, 0);
                    f = __builtin_amdgcn_mfma_f64_16x16x4f64(-x[r][k + g], l, f, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[16 + g + 4 * v][16 + r] = c[v];
                    x[g + 4 * v][16 + r] = f[v];
                }
                wave_lds_sync();
            }
        }
        // the first pivot that was not positive and finite
        const unsigned long long bad = __ballot(lane < nbk && !(s[lane & (CB - 1)][lane & (CB - 1)] > 0.0));
        if (lane == 0 && bad != 0 && *arg.flag == n) *arg.flag = c0b + __builtin_ctzll(bad);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < CB * CB; i += 256) {
        const int r = i / CB, q = i % CB;
        Linv[i] = x[q][r];
        if (r < nbk && q <= r) arg.L[(long)(c0b + r) * n + c0b + q] = s[r][q];
    }
}

// the first diagonal block (the others are factored by the step before them)
__global__ void __launch_bounds__(256) chol_diag_kernel(CholArgs a)
{
    __shared__ double s[CB][CB + 1], x[CB][CB + 1];
    const int n = a.n, nbk = min(CB, n);
    for (int e = threadIdx.x; e < CB * CB; e += 256) {
        const int r = e / CB, q = e % CB;
        s[r][q] = r < nbk && q <= r ? a.A[(long)r * n + q] : (r == q ? 1.0 : 0.0);
    }
    factor_block(s, x, nbk, 0, a, a.Linv);
}

// Step b of the right-looking factorization over the trailing lower tiles
// (rb, cb), b < cb <= rb: P = A_blk L_bb^-T for block rows rb and cb, then
// A_{rb,cb} -= P_rb P_cb^T (FP64 MFMA, wave w: output block (w / 2, w % 2)).
// The tile (rb, rb) stores P_rb as the factor; the tile (b + 1, b + 1),
// complete after this update, is factored and inverted right away.  The
// inverse of block b is read from Linv[b & 1] and that of b + 1 written to
// the other half, so no workgroup of this launch reads what another writes.
__global__ void __launch_bounds__(256, 2) chol_step_kernel(CholArgs a, int b)
{
    __shared__ double li[CB][CB + 1];
    __shared__ double ar[CB][CB + 1];
    __shared__ double ac[CB][CB + 1];
    __shared__ double pr[CB][CB + 1];
    __shared__ double pc[CB][CB + 1];
    int rr, cc;
    tri_index(blockIdx.x, rr, cc);
    const int rb = b + 1 + rr, cb = b + 1 + cc;
    const int n = a.n, c0 = b * CB, R0 = rb * CB, C0 = cb * CB;
    const bool diag = rb == cb;
    const double *Li = a.Linv + (b & 1) * CB * CB;
    for (int e = threadIdx.x; e < CB * CB; e += 256) {
        const int x = e / CB, y = e % CB;
        li[x][y] = Li[e];
        // block column b is whole: b < the last block column
        ar[x][y] = R0 + x < n ? a.A[(long)(R0 + x) * n + c0 + y] : 0.0;
        if (!diag) ac[x][y] = C0 + x < n ? a.A[(long)(C0 + x) * n + c0 + y] : 0.0;
    }
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
    const int ba = 16 * (wv >> 1), bb = 16 * (wv & 1);
    double old[4];  // this wave's block of the tile, fetched with the operands
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int x = ba + lq + 4 * v, y = bb + lr;
        old[v] = R0 + x < n && C0 + y < n ? a.A[(long)(R0 + x) * n + C0 + y] : 0.0;
    }
    __syncthreads();
    d4 c1 = {0.0, 0.0, 0.0, 0.0}, c2 = c1;
#pragma unroll
    for (int kk = 0; kk < CB; kk += 4) {
        const double y = li[bb + lr][kk + lq];
        c1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[ba + lr][kk + lq], y, c1, 0, 0, 0);
        if (!diag) c2 = __builtin_amdgcn_mfma_f64_16x16x4f64(ac[ba + lr][kk + lq], y, c2, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        pr[ba + lq + 4 * v][bb + lr] = c1[v];
        if (!diag) pc[ba + lq + 4 * v][bb + lr] = c2[v];
    }
    __syncthreads();
    double(*pcc)[CB + 1] = diag ? pr : pc;
    d4 cu = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < CB; kk += 4)
        cu = __builtin_amdgcn_mfma_f64_16x16x4f64(pr[ba + lr][kk + lq], pcc[bb + lr][kk + lq], cu, 0, 0, 0);
    const bool next = diag && rb == b + 1;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int x = ba + lq + 4 * v, y = bb + lr;
        if (R0 + x < n && C0 + y < n && (!diag || y <= x)) {
            const long e = (long)(R0 + x) * n + C0 + y;
            const double nv = old[v] - cu[v];
            a.A[e] = nv;
            if (next) ar[x][y] = nv;  // ar is no longer read: the products above are done
        } else if (next) {
            ar[x][y] = x == y ? 1.0 : 0.0;
        }
    }
    if (diag) {
        for (int e = threadIdx.x; e < CB * CB; e += 256) {
            const int x = e / CB, y = e % CB;
            if (R0 + x >= n) continue;
            const long eL = (long)(R0 + x) * n + c0 + y;
            a.L[eL] = pr[x][y];
        }
    }
    if (next) factor_block(ar, li, min(CB, n - R0), R0, a, a.Linv + ((b + 1) & 1) * CB * CB);
}

void launch_cholesky(const CholArgs &a, hipStream_t s)
{
    const long N = (long)a.n * a.n;
    const int g = (int)std::min<long>((N + 255) / 256, 4096);
    hipLaunchKernelGGL(chol_init_kernel, dim3(g), dim3(256), 0, s, a);
    hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(256), 0, s, a);
    const int nb = (a.n + CB - 1) / CB;
    for (int b = 0; b + 1 < nb; ++b) {
        const int T = nb - b - 1;
        hipLaunchKernelGGL(chol_step_kernel, dim3(T * (T + 1) / 2), dim3(256), 0, s, a, b);
    }
}

// ------------------------------------------------------------------ sampling
// U = clip(nu + Z L^T) with Z (K x n normals) and L (n x n, lower) split into
// three bf16 parts each (24 bits and more; L's from double), the product as
// six bf16 partial products accumulated in FP32: 2.7 times the FP32 matrix
// rate, and closer to FP64 than with L rounded to FP32 (1.9e-7 of the result's
// norm against 3.2e-7).  What an MFMA drops (below 2^-24 of the largest of eight
// products) it drops downwards, so the odd chunks of L are negated and have
// sums of their own, which are subtracted: with one sum 2.7e-7, and all samples
// shifted by -2.3e-8 of their standard deviation (now -4e-9; 24.5 -> 24.9 us).
// Two launches instead of four (conversion of L,
// clearing of its upper triangle, normals, product): K = 1024, n = 896 39.8 ->
// 24.9 us, K = 4096, n = 1400 184 -> 99 us; what is left is the operands' way
// from the L2 (three chunks ahead; one ahead 29.9 us), not the products' 2 us.
//
// Both are laid out as MFMA 16x16x32 operands: 16 rows x 32 columns are 64
// lanes x 8 values (lane l: row l % 16, columns 8 (l / 16) ..), part after
// part, so a wave reads an operand as one contiguous kilobyte.  Rows past K or
// n and columns past n are zero; of L only the chunks up to the diagonal exist.
//
// L is scaled by 2^32 (and the sums back), so that its third parts stay normal
// down to entries of 1e-42, where single precision ends; entries past 1e28
// make a sum infinite, which is then formed again (below).
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
constexpr double LS = 4294967296.0;  // 2^32

__device__ __forceinline__ void split3(float x, unsigned short p[3])
{
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const __bf16 b = (__bf16)x;
        p[t] = __builtin_bit_cast(unsigned short, b);
        x -= (float)b;
    }
}

struct Parts8 {
    unsigned short v[3][8];
};
__device__ __forceinline__ void put_parts(unsigned short *dst, const Parts8 &q)
{
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        uint4 w;
        __builtin_memcpy(&w, q.v[t], 16);
        *reinterpret_cast<uint4 *>(dst + 512 * t) = w;  // 64 lanes x 8 to the next part
    }
}

// Operands of the product.  The first nzb workgroups write Z: a thread takes
// one sample's eight columns, the 64 lanes of a wave 64 samples of the same
// columns, so that the walk over the counters (a Philox call a quarter step,
// a Box-Muller pair every other column) is uniform; drawn a normal at a time
// as before, every value repeated both.  The others write L: a thread takes
// eight columns of a row.
__global__ void __launch_bounds__(256) sample_operands_kernel(SampleFullArgs a, int nzb)
{
    const int n = a.n, K = a.K, nc = (n + 31) >> 5;  // chunks of 32 columns
    if ((int)blockIdx.x < nzb) {
        const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
        const int oc = 4 * nc, jb = w / oc, o = w - jb * oc;  // 64 samples, 8 columns
        const int j = 64 * jb + lane;
        if (64 * jb >= K) return;
        Parts8 q = {};
        U4 rnd = {};
        float z0 = 0.f, z1 = 0.f;
        int have = -1;  // quarter step of rnd
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int p = __builtin_amdgcn_readfirstlane(8 * o + e);
            if (p < n) {
                const int k = p / NU, d = p - k * NU, quarter = 4 * k + (d >> 2);
                if (quarter != have) {
                    rnd = philox4x32_10(U4{(uint32_t)j, (uint32_t)k, (uint32_t)(d >> 2), (uint32_t)a.m}, a.key0, a.key1);
                    have = quarter;
                }
                if (e == 0 || (d & 1) == 0) {
                    const bool hi = (d & 3) >> 1;
                    box_muller(hi ? rnd.z : rnd.x, hi ? rnd.w : rnd.y, z0, z1);
                }
                unsigned short t[3];
                split3((d & 1) ? z1 : z0, t);
                q.v[0][e] = t[0]; q.v[1][e] = t[1]; q.v[2][e] = t[2];
            }
        }
        if (j >= K) q = Parts8{};
        const int c = o >> 2, l = 16 * (o & 3) + (j & 15);
        put_parts(a.Z + (((long)(j >> 4) * nc + c) * 192 + l) * 8, q);
        return;
    }
    const int nt = (n + 15) >> 4;
    const long w = (long)(blockIdx.x - nzb) * 4 + (threadIdx.x >> 6);
    const int ib = (int)(w / nc), c = (int)(w - (long)ib * nc), lane = threadIdx.x & 63;
    if (ib >= nt || 32 * c > 16 * ib + 15) return;
    const int i = 16 * ib + (lane & 15), p0 = 32 * c + 8 * (lane >> 4);
    Parts8 q = {};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int p = p0 + e;
        if (i < n && p <= i) {
            double x = (c & 1 ? -LS : LS) * a.L[(long)i * n + p];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const __bf16 b = (__bf16)(float)x;
                q.v[t][e] = __builtin_bit_cast(unsigned short, b);
                x -= (double)(float)b;
            }
        }
    }
    put_parts(a.Lp + (((long)ib * nc + c) * 192 + lane) * 8, q);
}

// Output tile: 32 samples x 64 entries; wave w owns entries i0 + 16 w .. + 15
// (two 16x16 results).  Operands go straight to registers, SD chunks ahead of
// their products: no LDS, no barrier.  Tiles of the last
// entries, whose sums are the longest, are handed out first; consecutive
// workgroups take different samples, so that with a multiple of eight sample
// tiles an XCD keeps to its own.
constexpr int SJ = 32, SI = 64, SD = 3;

__global__ void __launch_bounds__(256) sample_full_kernel(SampleFullArgs a)
{
    const int n = a.n, K = a.K, nc = (n + 31) >> 5;
    const int nj = (K + SJ - 1) / SJ, ni = (n + SI - 1) / SI;
    const int it = ni - 1 - (int)(blockIdx.x / nj), jt = blockIdx.x % nj;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int ib = 4 * it + wv, j0 = SJ * jt;
    if (16 * ib >= n) return;
    const int nch = ((16 * ib + 15) >> 5) + 1;  // chunks up to the diagonal
    const bool two = j0 + 16 < K;               // the second sample block holds a sample
    const b8 *z0 = reinterpret_cast<const b8 *>(a.Z) + (long)(2 * jt) * nc * 192 + lane;
    const b8 *z1 = z0 + (two ? (long)nc * 192 : 0);
    const b8 *lp = reinterpret_cast<const b8 *>(a.Lp) + (long)ib * nc * 192 + lane;
    f4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0, o0 = c0, o1 = c0;  // even and (negated) odd chunks
    b8 x0[SD][3], x1[SD][3], y[SD][3];
    auto load = [&](int s, int c) {
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            y[s][t] = lp[192 * c + 64 * t];
            x0[s][t] = z0[192 * c + 64 * t];
            x1[s][t] = z1[192 * c + 64 * t];
        }
    };
#pragma unroll
    for (int s = 0; s < SD; ++s) load(s, min(s, nch - 1));
    for (int cb = 0; cb < nch; cb += 2 * SD) {
#pragma unroll
        for (int u = 0; u < 2 * SD; ++u) {
            const int s = u % SD;
            if (cb + u < nch) {  // uniform over the wave
                constexpr int TX[6] = {0, 2, 1, 0, 1, 0}, TY[6] = {2, 0, 1, 1, 0, 0};  // small products first
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    f4 &d0 = u & 1 ? o0 : c0, &d1 = u & 1 ? o1 : c1;
                    d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0[s][TX[e]], y[s][TY[e]], d0, 0, 0, 0);
                    d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1[s][TX[e]], y[s][TY[e]], d1, 0, 0, 0);
                }
                load(s, min(cb + u + SD, nch - 1));
            }
        }
    }
    c0 -= o0;
    c1 -= o1;
    const int i = 16 * ib + r;
    if (i >= n) return;
    const float nui = a.nu[i], unscale = (float)(1.0 / LS);
    unsigned again = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ja = j0 + 4 * q + e;
        if (ja < K) a.U[(long)ja * n + i] = fminf(fmaxf(fmaf(unscale, c0[e], nui), -a.u_max), a.u_max);
        if (ja + 16 < K) a.U[(long)(ja + 16) * n + i] = fminf(fmaxf(fmaf(unscale, c1[e], nui), -a.u_max), a.u_max);
        again |= (isfinite(c0[e]) ? 0u : 1u << e) | (isfinite(c1[e]) ? 0u : 16u << e);
    }
    // The parts of an entry that is infinite in single precision are no sum (Inf,
    // NaN, NaN): such a row's sums are formed again from L itself, so that they
    // saturate by their sign.  From the diagonal on, for a factor that failed is
    // NaN from there.
    for (; again != 0u; again &= again - 1u) {
        const int e = __builtin_ctz(again), ja = j0 + 4 * q + (e & 3) + 4 * (e & 4);
        if (ja >= K) continue;
        double sum = 0.0;
        for (int p = i; p >= 0 && sum == sum; --p) {
            const long z = (((long)(ja >> 4) * nc + (p >> 5)) * 192 + 16 * ((p & 31) >> 3) + (ja & 15)) * 8 + (p & 7);
            float zp = 0.f;  // the parts' sum is the normal exactly
#pragma unroll
            for (int t = 0; t < 3; ++t) zp += __uint_as_float((uint32_t)a.Z[z + 512 * t] << 16);
            sum = fma((double)zp, (double)(float)a.L[(long)i * n + p], sum);
        }
        a.U[(long)ja * n + i] = fminf(fmaxf(nui + (float)sum, -a.u_max), a.u_max);
    }
}

size_t sample_z_bytes(int K, int n) { return (size_t)((K + 63) / 64) * 4 * ((n + 31) / 32) * 192 * 16; }
size_t sample_l_bytes(int n) { return (size_t)((n + 15) / 16) * ((n + 31) / 32) * 192 * 16; }

void launch_sample_full(const SampleFullArgs &a, hipStream_t s)
{
    const int nc = (a.n + 31) / 32, nt = (a.n + 15) / 16;
    const int nzb = (a.K + 63) / 64 * nc;  // four waves of (64 samples, 8 columns) a workgroup
    const int nlb = (nt * nc + 3) / 4;
    hipLaunchKernelGGL(sample_operands_kernel, dim3(nzb + nlb), dim3(256), 0, s, a, nzb);
    hipLaunchKernelGGL(sample_full_kernel, dim3(((a.n + SI - 1) / SI) * ((a.K + SJ - 1) / SJ)), dim3(256), 0, s, a);
}

__global__ void __launch_bounds__(256) diag_sigma_kernel(const float *sigma, int sps, int n, double *S)
{
    const long N = (long)n * n;
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
        const long i = e / n, l = e - i * n;
        double v = 0.0;
        if (i == l) {
            const double sg = sigma[sps ? i : i % NU];
            v = sg * sg;
        }
        S[e] = v;
    }
}

void launch_diag_sigma(const float *sigma, int sps, int n, double *S, hipStream_t s)
{
    const long N = (long)n * n;
    const int g = (int)std::min<long>((N + 255) / 256, 4096);
    hipLaunchKernelGGL(diag_sigma_kernel, dim3(g), dim3(256), 0, s, sigma, sps, n, S);
}

}  // namespace mppi
