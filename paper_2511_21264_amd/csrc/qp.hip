// QP smoothing of sampled joint-velocity sequences (Alg. 1: the projection
// of every sample after the sampling step; Eqs. proj_cost and proj_bounds
// with bounds on the joint trajectory and its first three derivatives).
//
// Each joint of each sample is a QP over the horizon in the H control-step
// velocities; the bounds are on A v with A = [I; D1; D2; L] (identity, first
// and second differences, prefix sums), all in velocity units.  The solver is
// a fixed number of over-relaxed ADMM iterations:
//     v  = P (v~ + rho A^T (z - w)),   P = (I + rho A^T A)^-1
//        (evaluated as v~ + rho P A^T (z - w - A v~))
//     a  = alpha A v + (1 - alpha) z
//     z' = clip(a + w, lo, hi);   w += a - z';   z = z'
// from z = clip(A v~), w = 0; the output is v clipped to the velocity box.
//
// Two forms, by sample count and horizon (launch_project): one wave per
// sixteen sequences (project_tile_kernel), and
// one workgroup per sample, one wave per joint (14 waves), one
// horizon step per lane for H <= 64 and two (steps k and k + 64) for
// H <= 128.  A v and A^T y are DPP whole-wave shifts and
// scans (neighbour differences, prefix and suffix sums).  The dense product
// with P, the same for every joint and sample, is one 64 x 64 by 64 x 16
// product per iteration on FP32 MFMA: the waves publish their right-hand
// sides to LDS, waves 0..4 NH - 1 each hold a 16-row block of P in registers
// for the whole kernel and multiply (16 NH steps of 16x16x4), and every wave
// reads its column of the result back.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "team.h"

namespace mppi {

namespace {

__device__ __forceinline__ float clipf(float x, float lo, float hi) { return fminf(fmaxf(x, lo), hi); }

// Wave-wide shifts and scans without an LDS trip: DPP shifts within 16-lane
// rows (lanes whose source lies outside the row read 0), then the row totals
// carried across rows (DPP row broadcasts for the prefix sum, v_readlane for
// the suffix sum).  Every lane of the wave is active wherever these run.
template <int S>
__device__ __forceinline__ float shr_row(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x110 + S, 0xF, 0xF, true));
}
template <int S>
__device__ __forceinline__ float shl_row(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x100 + S, 0xF, 0xF, true));
}
// whole-wave shifts by one lane (DPP wave_shr:1 / wave_shl:1): lane k reads
// lane k - 1 / k + 1; lane 0 / 63 reads 0
__device__ __forceinline__ float wave_shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_shl1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}
template <int L>
__device__ __forceinline__ float lane_of(float v)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), L));
}

// inclusive prefix sum over the wave: scans within the rows, then the row
// totals carried by DPP row_bcast:15 (lane 15 of each row into the next row;
// rows 1 and 3 take it) and row_bcast:31 (lane 31 into rows 2 and 3); lanes
// of the rows a broadcast leaves out add 0
__device__ __forceinline__ float prefix64(float x, int)
{
    x += shr_row<1>(x);
    x += shr_row<2>(x);
    x += shr_row<4>(x);
    x += shr_row<8>(x);
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x142, 0xA, 0xF, true));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x143, 0xC, 0xF, true));
    return x;
}
// inclusive suffix sum over the wave
__device__ __forceinline__ float suffix64(float x, int k)
{
    x += shl_row<1>(x);
    x += shl_row<2>(x);
    x += shl_row<4>(x);
    x += shl_row<8>(x);
    const float t1 = lane_of<16>(x), t2 = lane_of<32>(x), t3 = lane_of<48>(x);
    const int row = k >> 4;
    const float off = row == 3 ? 0.f : (row == 2 ? t3 : (row == 1 ? t3 + t2 : (t3 + t2) + t1));
    return x + off;
}

// A v for the sequence held one element per lane (lane k: step k); rows that
// do not exist (first difference at k = 0, second at k < 2, any k >= H) are 0
__device__ __forceinline__ void apply_A(float v, int k, bool act, float &aI, float &a1, float &a2, float &aL)
{
    const float x = act ? v : 0.f;
    const float vm1 = wave_shr1(x), vm2 = wave_shr1(vm1);  // 0 before step 0
    aI = x;
    a1 = (act && k >= 1) ? x - vm1 : 0.f;
    a2 = (act && k >= 2) ? (x - 2.f * vm1) + vm2 : 0.f;
    const float p = prefix64(x, k);
    aL = act ? p : 0.f;  // lanes past the horizon hold no row (their w must stay 0)
}

// A^T y at lane k (y of absent rows are 0): y_I + (y1_k - y1_{k+1}) +
// (y2_k - 2 y2_{k+1} + y2_{k+2}) + sum_{i >= k} yL_i
__device__ __forceinline__ float apply_At(float yI, float y1, float y2, float yL, int k)
{
    // the shifts read 0 past the end of the wave
    const float y1n = wave_shl1(y1), y2n = wave_shl1(y2), y2nn = wave_shl1(y2n);
    return yI + (y1 - y1n) + ((y2 - 2.f * y2n) + y2nn) + suffix64(yL, k);
}

// Two steps per lane (64 < H <= 128): lane k holds steps k (half 0) and
// k + 64 (half 1); the halves join at the boundary through v_readlane of
// lanes 63 and 0.
__device__ __forceinline__ void apply_A2(const float v[2], int k, const bool act[2], float aI[2], float a1[2],
                                         float a2[2], float aL[2])
{
    const float x0 = act[0] ? v[0] : 0.f, x1 = act[1] ? v[1] : 0.f;
    const float e62 = lane_of<62>(x0), e63 = lane_of<63>(x0);
    const float u0 = wave_shr1(x0), w0 = wave_shr1(u0), u1 = wave_shr1(x1), w1 = wave_shr1(u1);
    const float vm1_0 = u0, vm2_0 = w0;                                  // used for k >= 1 / k >= 2
    const float vm1_1 = k >= 1 ? u1 : e63, vm2_1 = k >= 2 ? w1 : (k == 1 ? e63 : e62);
    aI[0] = x0;
    aI[1] = x1;
    a1[0] = (act[0] && k >= 1) ? x0 - vm1_0 : 0.f;
    a2[0] = (act[0] && k >= 2) ? (x0 - 2.f * vm1_0) + vm2_0 : 0.f;
    a1[1] = act[1] ? x1 - vm1_1 : 0.f;
    a2[1] = act[1] ? (x1 - 2.f * vm1_1) + vm2_1 : 0.f;
    const float p0 = prefix64(x0, k);
    const float p1 = prefix64(x1, k) + lane_of<63>(p0);
    aL[0] = act[0] ? p0 : 0.f;
    aL[1] = act[1] ? p1 : 0.f;
}

__device__ __forceinline__ void apply_At2(const float yI[2], const float y1[2], const float y2[2], const float yL[2],
                                          int k, float out[2])
{
    const float b10 = lane_of<0>(y1[1]), b20 = lane_of<0>(y2[1]), b21 = lane_of<1>(y2[1]);
    const float s1_0 = wave_shl1(y1[0]), s2_0 = wave_shl1(y2[0]), s22_0 = wave_shl1(s2_0);
    const float s1_1 = wave_shl1(y1[1]), s2_1 = wave_shl1(y2[1]), s22_1 = wave_shl1(s2_1);
    // half 0: steps k + 1, k + 2 may lie in half 1
    const float y1n0 = k + 1 < 64 ? s1_0 : b10, y2n0 = k + 1 < 64 ? s2_0 : b20;
    const float y2nn0 = k + 2 < 64 ? s22_0 : (k == 62 ? b20 : b21);
    // half 1: nothing past step 127
    const float y1n1 = s1_1, y2n1 = s2_1, y2nn1 = s22_1;  // the shifts read 0 past lane 63
    const float q1 = suffix64(yL[1], k);
    const float q0 = suffix64(yL[0], k) + lane_of<0>(q1);
    out[0] = yI[0] + (y1[0] - y1n0) + ((y2[0] - 2.f * y2n0) + y2nn0) + q0;
    out[1] = yI[1] + (y1[1] - y1n1) + ((y2[1] - 2.f * y2n1) + y2nn1) + q1;
}

}  // namespace

// NH horizon steps per lane (1: H <= 64, 2: H <= 128); waves 0 .. 4 NH - 1
// hold the 16-row blocks of P.  FULL: H = 64 NH, so every lane holds a step
// and the masks of absent steps fold away.
template <int NH, bool FULL>
__global__ void __launch_bounds__(14 * 64) project_kernel(ProjectArgs a)
{
    constexpr int QS = 64 * NH + 4;  // LDS row stride of the right-hand sides and results (floats)
    constexpr int NST = 16 * NH;     // k-steps of the product
    __shared__ __align__(16) float R[16][QS];  // right-hand sides, one row per joint (rows 14, 15: zero)
    __shared__ __align__(16) float V[16][QS];  // P times them
    const int H = a.H, S = a.S;
    const int j = blockIdx.x;
    const int d = threadIdx.x >> 6, k = threadIdx.x & 63;
    bool act[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) act[h] = FULL || k + 64 * h < H;  // FULL: H = 64 NH, every lane holds a step
    if (d < 2) {
#pragma unroll
        for (int h = 0; h < NH; ++h) R[14 + d][k + 64 * h] = 0.f;
    }
    // waves 0 .. 4 NH - 1 keep rows 16 w .. 16 w + 15 of P as MFMA A operands:
    // pa[s] = P[16 w + l % 16][4 s + l / 16]
    const int lr = k & 15, lq = k >> 4;
    float pa[NST];
#pragma unroll
    for (int st = 0; st < NST; ++st) {
        const int row = 16 * d + lr, col = 4 * st + lq;
        pa[st] = (d < 4 * NH && row < H && col < H) ? a.P[row * S + col] : 0.f;
    }
    const float *x0 = a.x0 + (a.x0_shared ? 0 : (long)j * NX);
    const float q0 = x0[XQDES + d];
    float vt[NH], loI[NH], hiI[NH], lo1[NH], hi1[NH], lo2[NH], hi2[NH], loL[NH], hiL[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const int st = k + 64 * h;  // this lane's step in half h
        vt[h] = 0.f;
        if (act[h]) {
            if (a.U_in) {
                vt[h] = a.U_in[((long)j * H + st) * NU + d];
            } else {
                const float z = normal_joint(a.key0, a.key1, (uint32_t)j, (uint32_t)st, (uint32_t)a.m, d);
                vt[h] = fmaf(a.sigma[(a.sigma_per_step ? st * NU : 0) + d], z, a.nu[st * NU + d]);
            }
        }
        // the bounds of the four rows this lane holds (absent rows: [0, 0])
        loI[h] = act[h] ? -a.u_max : 0.f;
        hiI[h] = act[h] ? a.u_max : 0.f;
        lo1[h] = (act[h] && st >= 1) ? -a.dacc : 0.f;
        hi1[h] = (act[h] && st >= 1) ? a.dacc : 0.f;
        lo2[h] = (act[h] && st >= 2) ? -a.djerk : 0.f;
        hi2[h] = (act[h] && st >= 2) ? a.djerk : 0.f;
        loL[h] = act[h] ? (a.pos_lo[d] - q0) / a.dt : 0.f;
        hiL[h] = act[h] ? (a.pos_hi[d] - q0) / a.dt : 0.f;
    }
    // A v~ is kept: the v-update is evaluated as v~ + rho P A^T (z - w - A v~),
    // the same value as P (v~ + rho A^T (z - w)) since P (I + rho A^T A) = I,
    // but without the cancellation of two large terms (the prefix-sum rows
    // of rho A^T A v~ are hundreds of times larger than v~ at H = 64)
    float tI[NH], t1[NH], t2[NH], tL[NH];
    if constexpr (NH == 1)
        apply_A(vt[0], k, act[0], tI[0], t1[0], t2[0], tL[0]);
    else
        apply_A2(vt, k, act, tI, t1, t2, tL);
    float zI[NH], z1[NH], z2[NH], zL[NH], wI[NH], w1[NH], w2[NH], wL[NH], v[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        zI[h] = clipf(tI[h], loI[h], hiI[h]);
        z1[h] = clipf(t1[h], lo1[h], hi1[h]);
        z2[h] = clipf(t2[h], lo2[h], hi2[h]);
        zL[h] = clipf(tL[h], loL[h], hiL[h]);
        wI[h] = w1[h] = w2[h] = wL[h] = 0.f;
        v[h] = vt[h];
    }
    const float rho = a.rho, alpha = a.alpha, beta = 1.f - a.alpha;
    const int nst = (H + 3) >> 2;  // k-steps of the product that touch columns < H
    for (int it = 0; it < a.iters; ++it) {
        float yI[NH], y1[NH], y2[NH], yL[NH], rhs[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            yI[h] = (zI[h] - wI[h]) - tI[h];
            y1[h] = (z1[h] - w1[h]) - t1[h];
            y2[h] = (z2[h] - w2[h]) - t2[h];
            yL[h] = (zL[h] - wL[h]) - tL[h];
        }
        if constexpr (NH == 1)
            rhs[0] = apply_At(yI[0], y1[0], y2[0], yL[0], k);
        else
            apply_At2(yI, y1, y2, yL, k, rhs);
#pragma unroll
        for (int h = 0; h < NH; ++h) R[d][k + 64 * h] = act[h] ? rho * rhs[h] : 0.f;
        __syncthreads();
        if (d < 4 * NH) {
            // V[16 d + row][joint] = sum_i P[16 d + row][i] R[joint][i]; result
            // element e of lane l is row 4 (l / 16) + e, joint l % 16
            typedef float f4 __attribute__((ext_vector_type(4)));
            f4 acc = {0.f, 0.f, 0.f, 0.f};
            if (nst == NST) {  // full horizon: one unguarded chain
#pragma unroll
                for (int st = 0; st < NST; ++st)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[st], R[lr][4 * st + lq], acc, 0, 0, 0);
            } else {
#pragma unroll
                for (int st = 0; st < NST; ++st)
                    if (st < nst) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[st], R[lr][4 * st + lq], acc, 0, 0, 0);
            }
            *reinterpret_cast<f4 *>(&V[lr][16 * d + 4 * lq]) = acc;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < NH; ++h) v[h] = act[h] ? vt[h] + V[d][k + 64 * h] : 0.f;
        float aI[NH], a1[NH], a2[NH], aL[NH];
        if constexpr (NH == 1)
            apply_A(v[0], k, act[0], aI[0], a1[0], a2[0], aL[0]);
        else
            apply_A2(v, k, act, aI, a1, a2, aL);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            aI[h] = fmaf(alpha, aI[h], beta * zI[h]);
            a1[h] = fmaf(alpha, a1[h], beta * z1[h]);
            a2[h] = fmaf(alpha, a2[h], beta * z2[h]);
            aL[h] = fmaf(alpha, aL[h], beta * zL[h]);
            float zn = clipf(aI[h] + wI[h], loI[h], hiI[h]);
            wI[h] += aI[h] - zn;
            zI[h] = zn;
            zn = clipf(a1[h] + w1[h], lo1[h], hi1[h]);
            w1[h] += a1[h] - zn;
            z1[h] = zn;
            zn = clipf(a2[h] + w2[h], lo2[h], hi2[h]);
            w2[h] += a2[h] - zn;
            z2[h] = zn;
            zn = clipf(aL[h] + wL[h], loL[h], hiL[h]);
            wL[h] += aL[h] - zn;
            zL[h] = zn;
        }
    }
#pragma unroll
    for (int h = 0; h < NH; ++h)
        if (act[h]) a.U_out[((long)j * H + k + 64 * h) * NU + d] = clipf(v[h], -a.u_max, a.u_max);
}

// ---------------------------------------------------------------------------
// Tile form: one wave per sixteen sequences (consecutive joint sequences, the
// samples one after another), the whole iteration in its registers.  The MFMA
// 16x16x4 result puts sequence l % 16 on lane l and, of every 16-row block, the
// four rows 4 (l / 16) .. + 3.  Since the rows and columns of P may be taken
// in any order, block b, element v of lane group q is given step
// R q + 4 b + v (R = 4 NB steps a group, H <= 16 NB): a lane then holds R
// consecutive steps of one sequence, so the scans and differences of A v and
// A^T y are serial adds in registers plus a few values from the neighbouring
// groups, and the right-hand side of a column step (step i of every group) is
// already an MFMA's B operand.  Nothing passes between waves, so there is no
// barrier.
//   The product is formed in fp16 MFMAs 16x16x32 from three parts of each
// factor: whole units of 2^-9 of the largest magnitude (P's of the matrix, the
// right-hand side's of the sequence, rounded up to a power of two), then twice
// 11 bits of what is left (P's from double).  Where position bounds hold, the
// right-hand side is the suffix sums of hundreds of units that P all but
// cancels, and an MFMA drops what lies below 2^-24 of the largest of eight
// products, always downwards: an error that all steps of a sequence share and
// the iteration sums up.  The products of the whole units are free of it:
// |row of P| <= 23 of its largest entries in sum (P's norm is at most four of
// them), so they stay below 2^23 units, and they have a sum of their own.
// The other five partial products, 2^-10 and less of these, share one.  An
// FP32 MFMA and vector instructions do not overlap here, not even from two
// waves (with the product in FP32: 152 us).
//   Error over the whole iteration against FP64, of the result's norm, the
// workgroup form's in brackets: 3.2e-6 (5.5e-6) at H = 64, 4.4e-6 (7.1e-6) at
// H = 128 with the default bounds; with bounds 0.05 rad away, held by most
// sequences, 2.7e-6 (8.1e-6) and 8.7e-6 (3.1e-5) at rho = 3, 3.8e-6 (4.9e-4)
// at rho = 1, H = 128.  Three bf16 parts in one sum: 1.9e-5 and 1.7e-4 at
// rho = 3 (127 us).  The block offsets of the scans are in double (without:
// half as much again of the error, 13 % of the time).
//   Bound by vector instructions, about 56 a step and iteration, at one wave per
// SIMD (K = 1024: 896 waves).  K = 1024, H = 64, 60 iterations: 250 us (a
// workgroup per sample) -> 134 us; K = 4096: 987 -> 368 us; K = 1024, H = 24:
// 241 -> 71 us, H = 100: 583 -> 315 us, H = 128: 586 -> 392 us.  P's parts are
// in LDS in operand order, 24 KB at H = 64 and 96 KB at H = 128 for a workgroup
// of four waves.
// two floats (whole units up to 512 and what is left) as three fp16 parts each
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split3(float x0, float x1, uint32_t p[3])
{
    float y0 = rintf(x0), y1 = rintf(x1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const h2 h = __builtin_convertvector(t == 0 ? f2{y0, y1} : f2{x0, x1}, h2);
        p[t] = __builtin_bit_cast(uint32_t, h);
        x0 -= t == 0 ? y0 : (float)h.x;
        x1 -= t == 0 ? y1 : (float)h.y;
    }
}

// largest of the four lanes l, l + 16, l + 32, l + 48 (x >= 0), on all of them
__device__ __forceinline__ uint32_t groups_max(float x)
{
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const uint32_t m = max((uint32_t)h[0], (uint32_t)h[1]);
    const auto g = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    return max((uint32_t)g[0], (uint32_t)g[1]);
}

template <int NB, bool FULL>
__global__ void __launch_bounds__(256, NB <= 4 ? 2 : 1) project_tile_kernel(ProjectArgs a)
{
    constexpr int R = 4 * NB;
    constexpr int KS = (R + 7) / 8;  // product steps of eight columns a group
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) unsigned short PA[];  // [row block][product step][part][lane][8]
    const int H = a.H;
    for (int e = threadIdx.x; e < NB * KS * 512; e += 256) {
        const int c = e & 7, l = (e >> 3) & 63, w = e >> 9;
        const int rb = w / KS, i = 8 * (w % KS) + c;
        const int row = R * ((l & 15) >> 2) + 4 * rb + (l & 3), col = R * (l >> 4) + i;
        double p = (i < R && row < H && col < H) ? a.rhoP[row * H + col] / a.p_unit : 0.0;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const _Float16 b = (_Float16)(float)(t == 0 ? 64.0 * rint(p / 64.0) : p);
            PA[((w * 3 + t) * 64 + l) * 8 + c] = __builtin_bit_cast(unsigned short, b);
            p -= (double)(float)b;
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, q = lane >> 4;
    const long nseq = (long)a.K * NU;
    const long seq_raw = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + (lane & 15);
    if (seq_raw - (lane & 15) >= nseq) return;  // no barrier follows
    const bool live = seq_raw < nseq;
    const long seq = live ? seq_raw : nseq - 1;
    const int j = (int)(seq / NU), d = (int)(seq - (long)j * NU);
    const int s0 = R * q;  // this lane's first step
    // values of the neighbouring groups through the LDS crossbar (lanes l -+ 16 k)
    const int dn1 = ((lane - 16) & 63) << 2, dn2 = ((lane - 32) & 63) << 2, dn3 = ((lane - 48) & 63) << 2;
    const int up1 = ((lane + 16) & 63) << 2, up2 = dn2, up3 = dn1;
    auto from = [](int addr, float v) { return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v))); };
    const bool h1 = q >= 1, h2 = q >= 2, h3 = q >= 3;  // groups below this one
    const bool g1 = q <= 2, g2 = q <= 1, g3 = q == 0;  // groups above
    auto present = [&](int i) { return FULL || s0 + i < H; };
    float pos_lo = a.pos_lo[0], pos_hi = a.pos_hi[0];
#pragma unroll
    for (int e = 1; e < NU; ++e) {
        pos_lo = d == e ? a.pos_lo[e] : pos_lo;
        pos_hi = d == e ? a.pos_hi[e] : pos_hi;
    }
    const float q0 = a.x0[(a.x0_shared ? 0 : (long)j * NX) + XQDES + d];
    const float loL = (pos_lo - q0) / a.dt, hiL = (pos_hi - q0) / a.dt;
    const float um = a.u_max, da = a.dacc, dj = a.djerk;
    float vt[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int st = s0 + i;
        vt[i] = 0.f;
        if (present(i)) {
            if (a.U_in) {
                vt[i] = a.U_in[((long)j * H + st) * NU + d];
            } else {
                const float z = normal_joint(a.key0, a.key1, (uint32_t)j, (uint32_t)st, (uint32_t)a.m, d);
                vt[i] = fmaf(a.sigma[(a.sigma_per_step ? st * NU : 0) + d], z, a.nu[st * NU + d]);
            }
        }
    }
    // The rows of A x: x itself, its differences with the one and two steps
    // before (across the groups' edge, values m1 and m2; 0 where the row is
    // absent) and its prefix sums.  The sums run within a block of four, over
    // the blocks and over the groups, so that no rounding chain is longer than
    // a wave-wide scan's.
    auto diff1 = [&](const float (&x)[R], int i, float m1) {
        const float r = x[i] - (i >= 1 ? x[i >= 1 ? i - 1 : 0] : m1);
        return (i >= 1 || h1) && present(i) ? r : 0.f;
    };
    auto diff2 = [&](const float (&x)[R], int i, float m1, float m2) {
        const float b = i >= 1 ? x[i >= 1 ? i - 1 : 0] : m1;
        const float c = i >= 2 ? x[i >= 2 ? i - 2 : 0] : (i == 1 ? m1 : m2);
        const float r = (x[i] - 2.f * b) + c;
        return (i >= 2 || h1) && present(i) ? r : 0.f;
    };
    // Sums over the blocks before this one (in the scan's direction): of this
    // lane in double, of the groups before it likewise, handed back as a float
    // and what it lacks.  A block's elements share this offset, so its
    // rounding would move them together and the prefix-sum rows of all later
    // steps with it; every other rounding of the scans is an element's own.
    auto move = [&](int addr, double x, bool on) {
        const int2 w = __builtin_bit_cast(int2, x);
        const int2 m = {__builtin_amdgcn_ds_bpermute(addr, w.x), __builtin_amdgcn_ds_bpermute(addr, w.y)};
        return on ? __builtin_bit_cast(double, m) : 0.0;
    };
    auto below = [&](double x) { return (move(dn3, x, h3) + move(dn2, x, h2)) + move(dn1, x, h1); };
    auto above = [&](double x) { return (move(up3, x, g3) + move(up2, x, g2)) + move(up1, x, g1); };
    auto hi_lo = [](double x, float &hi, float &lo) {
        hi = (float)x;
        lo = (float)(x - (double)hi);
    };
    auto prefix4 = [](const float *x, float *o) {
        o[0] = x[0];
        o[1] = x[0] + x[1];
        o[2] = o[1] + x[2];
        o[3] = o[1] + (x[2] + x[3]);
    };
    const float blo[3] = {-um, -da, -dj}, bhi[3] = {um, da, dj};
    float tL[R];  // A v~, prefix-sum rows (the others follow from v~)
    // (every lane takes part in the crossbar moves; the selects come after)
    float tm1 = from(dn1, vt[R - 1]), tm2 = from(dn1, vt[R - 2]);
    tm1 = h1 ? tm1 : 0.f;
    tm2 = h1 ? tm2 : 0.f;
    {
        float o[R], hi[NB], lo[NB];
        double t = 0.0, off[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            prefix4(vt + 4 * b, o + 4 * b);
            off[b] = t;
            t += (double)o[4 * b + 3];
        }
        const double g = below(t);
#pragma unroll
        for (int b = 0; b < NB; ++b) hi_lo(off[b] + g, hi[b], lo[b]);
#pragma unroll
        for (int i = 0; i < R; ++i) tL[i] = present(i) ? hi[i >> 2] + (o[i] + lo[i >> 2]) : 0.f;
    }
    auto target = [&](int k, int i) { return k == 0 ? vt[i] : (k == 1 ? diff1(vt, i, tm1) : diff2(vt, i, tm1, tm2)); };
    // State of row k (0 identity, 1, 2 differences) of step i.
    // LEAN: the relaxed value s alone, of which z = clip(s) and w = s - z; else
    // what the next iteration takes of them, g = (1 - alpha) z + w and
    // y = z - w - A v~.
    constexpr bool LEAN = NB > 4;
    const float alpha = a.alpha, beta = 1.f - a.alpha;
    float G[3][R], Y[3][LEAN ? 1 : R];
    auto put = [&](int k, int i, float sv) {
        if (LEAN) {
            G[k][i] = sv;
        } else {
            const float z = __builtin_amdgcn_fmed3f(sv, blo[k], bhi[k]), w = sv - z;
            G[k][i] = fmaf(beta, z, w);
            Y[k][LEAN ? 0 : i] = (z - w) - target(k, i);
        }
    };
    auto get_y = [&](int k, int i) {
        if (!LEAN) return Y[k][LEAN ? 0 : i];
        const float z = __builtin_amdgcn_fmed3f(G[k][i], blo[k], bhi[k]), w = G[k][i] - z;
        return (z - w) - target(k, i);
    };
    auto relax = [&](int k, int i, float av) {
        if (!LEAN) return fmaf(alpha, av, G[k][i]);
        const float z = __builtin_amdgcn_fmed3f(G[k][i], blo[k], bhi[k]), w = G[k][i] - z;
        return fmaf(alpha, av, fmaf(beta, z, w));
    };
    // The prefix-sum rows run to a hundred times the others' size, so they keep
    // z and w themselves: w += a - z then carries the rounding of a + w, which
    // s - z would lose.  Absent ones stay at z = w = 0.
    float zL[R], wL[R];
    auto get_yL = [&](int i) { return (zL[i] - wL[i]) - tL[i]; };
    float v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        v[i] = vt[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) put(k, i, __builtin_amdgcn_fmed3f(target(k, i), blo[k], bhi[k]));  // z = clip(A v~), w = 0
        zL[i] = present(i) ? __builtin_amdgcn_fmed3f(tL[i], loL, hiL) : 0.f;
        wL[i] = 0.f;
    }
    int p_off = lane;
    for (int it = 0; it < a.iters; ++it) {
        // P's operands are read from LDS in every iteration (hoisted out of the
        // loop they would take up to 384 registers)
        asm volatile("" : "+v"(p_off));
        const h8 *P8 = reinterpret_cast<const h8 *>(PA) + p_off;
        // right-hand side A^T (z - w - A v~), from the last step down
        float r[R];
        {
            double t = 0.0, off[NB];
            float hi[NB], lo[NB];
#pragma unroll
            for (int b = NB - 1; b >= 0; --b) {
                const float x[4] = {get_yL(4 * b + 3), get_yL(4 * b + 2), get_yL(4 * b + 1), get_yL(4 * b)};
                float o[4];
                prefix4(x, o);
#pragma unroll
                for (int c = 0; c < 4; ++c) r[4 * b + 3 - c] = o[c];
                off[b] = t;
                t += (double)o[3];
            }
            float y1n = from(up1, get_y(1, 0)), y2n = from(up1, get_y(2, 0)), y2nn = from(up1, get_y(2, 1));
            const double g = above(t);
#pragma unroll
            for (int b = 0; b < NB; ++b) hi_lo(off[b] + g, hi[b], lo[b]);
            y1n = g1 ? y1n : 0.f;
            y2n = g1 ? y2n : 0.f;
            y2nn = g1 ? y2nn : 0.f;
#pragma unroll
            for (int i = R - 1; i >= 0; --i) {
                const float y1 = get_y(1, i), y2 = get_y(2, i);
                r[i] = get_y(0, i) + (y1 - y1n) + ((y2 - 2.f * y2n) + y2nn) + (hi[i >> 2] + (r[i] + lo[i >> 2]));
                y1n = y1;
                y2nn = y2n;
                y2n = y2;
            }
        }
        // The product, one row block after another, and the rows of A v with
        // the relaxed update, each piece of a block between the MFMAs of the
        // next block (the scheduling fences keep it there): one wave per SIMD
        // has nothing else to run under them.  What waits for the other groups
        // (the first two steps' differences, the prefix sums) comes last.
        // the parts of the right-hand side as MFMA operands, eight steps each, in
        // units of 2^-9 of the sequence's largest element rounded up to a power of 2
        float rm = 0.f;
#pragma unroll
        for (int i = 0; i < R; i += 2) rm = fmaxf(fmaxf(fabsf(r[i]), fabsf(r[i + 1])), rm);
        const uint32_t eb = max(groups_max(rm) & 0x7f800000u, 40u << 23);
        const float per_unit = __uint_as_float((262u << 23) - eb), unit = a.p_unit32 * __uint_as_float(eb - (8u << 23));
        union Op {
            uint32_t u[4];
            h8 h;
        } rp[KS][3];
#pragma unroll
        for (int i = 0; i < 8 * KS; i += 2) {
            uint32_t x[3] = {0u, 0u, 0u};
            if (i < R) split3(per_unit * r[i < R ? i : 0], per_unit * r[i < R ? i + 1 : 0], x);
#pragma unroll
            for (int t = 0; t < 3; ++t) rp[i >> 3][t].u[(i & 7) >> 1] = x[t];
        }
        f4 acc[NB];
        auto piece = [&](int p) {  // row kind p % 4 of step p / 4 (0: the step itself)
            const int i = p >> 2;
            if ((p & 3) == 0) v[i] = fmaf(unit, acc[i >> 2][i & 3], vt[i]);
            if ((p & 3) == 1) put(0, i, relax(0, i, v[i]));
            if ((p & 3) == 2 && i >= 1) put(1, i, relax(1, i, diff1(v, i, 0.f)));
            if ((p & 3) == 3 && i >= 2) put(2, i, relax(2, i, diff2(v, i, 0.f, 0.f)));
        };
        constexpr int PP = (16 + 6 * KS - 1) / (6 * KS);  // pieces between two MFMAs
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            acc[b] = f4{0.f, 0.f, 0.f, 0.f};
            f4 lo = acc[b];
            // the six leading products of the parts, the exact ones (0, 0) apart, the
            // others small ones first; at NB = 8 one product step after another,
            // with that step's parts alone in registers (428 us otherwise, 391 so)
            constexpr int TP[6] = {0, 2, 1, 0, 1, 0}, TR[6] = {2, 0, 1, 1, 0, 0};
            constexpr bool INNER = NB == 8;
            h8 pa[KS][3];
            auto fetch = [&](int k) {
#pragma unroll
                for (int t = 0; t < 3; ++t) pa[k][t] = P8[64 * ((b * KS + k) * 3 + t)];
            };
            if (!INNER) {
#pragma unroll
                for (int k = 0; k < KS; ++k) fetch(k);
            }
#pragma unroll
            for (int e = 0; e < 6 * KS; ++e) {
                const int k = INNER ? e / 6 : e % KS, n = INNER ? e % 6 : e / KS;
                if (INNER && n == 0) fetch(k);
                f4 &d = n < 5 ? lo : acc[b];
                d = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa[k][TP[n]], rp[k][TR[n]].h, d, 0, 0, 0);
                if (b > 0) {
#pragma unroll
                    for (int p = PP * e; p < PP * (e + 1); ++p)
                        if (p < 16) piece(16 * (b - 1) + p);
                    if (PP * e < 16) __builtin_amdgcn_sched_barrier(0);
                }
            }
            acc[b] += lo;
        }
#pragma unroll
        for (int n = 0; n < 16; ++n) piece(16 * (NB - 1) + n);
        float o[R], hi[NB], lo[NB];
        double t = 0.0, off[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            prefix4(v + 4 * b, o + 4 * b);
            off[b] = t;
            t += (double)o[4 * b + 3];
        }
        float m1 = from(dn1, v[R - 1]), m2 = from(dn1, v[R - 2]);
        const double g = below(t);
#pragma unroll
        for (int b = 0; b < NB; ++b) hi_lo(off[b] + g, hi[b], lo[b]);
        m1 = h1 ? m1 : 0.f;
        m2 = h1 ? m2 : 0.f;
        put(1, 0, relax(1, 0, diff1(v, 0, m1)));
        put(2, 0, relax(2, 0, diff2(v, 0, m1, m2)));
        put(2, 1, relax(2, 1, diff2(v, 1, m1, m2)));
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const float av = fmaf(alpha, hi[i >> 2] + (o[i] + lo[i >> 2]), beta * zL[i]);
            const float z = __builtin_amdgcn_fmed3f(av + wL[i], loL, hiL);
            wL[i] = present(i) ? wL[i] + (av - z) : 0.f;
            zL[i] = present(i) ? z : 0.f;
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (live && present(i)) a.U_out[((long)j * H + s0 + i) * NU + d] = clipf(v[i], -um, um);
}

template <int NB>
static void launch_tile(const ProjectArgs &a, hipStream_t s)
{
    const unsigned grid = (unsigned)(((long)a.K * NU + 63) / 64);
    const size_t lds = (size_t)NB * ((4 * NB + 7) / 8) * 3 * 64 * 16;
    if (a.H == 16 * NB)
        hipLaunchKernelGGL((project_tile_kernel<NB, true>), dim3(grid), dim3(256), lds, s, a);
    else
        hipLaunchKernelGGL((project_tile_kernel<NB, false>), dim3(grid), dim3(256), lds, s, a);
}

// The workgroup-per-sample form takes about 62 us (H <= 64) or 146 us (beyond)
// for every 256 samples, one workgroup a CU; the tile form 71, 134, 311 and
// 387 us at H = 24, 64, 100 and 128 for up to 1170 samples (a wave a SIMD) and
// as much again for the next.  So the tile form is taken from the sample count
// on at which it is the faster: 257 samples up to H = 32 (122 against 71 us),
// 513 beyond (K = 600: 188 against 133 us at H = 64, 439 against 387 at
// H = 128).  Up to H = 16 the other form stays (an earlier product of this one
// was less exact there, 2.6e-6 against 2.1e-6 of the result's norm at H = 8).
void launch_project(const ProjectArgs &a, hipStream_t s)
{
    if (a.H > 16 && a.K > (a.H <= 32 ? 256 : 512)) {
        switch ((a.H + 15) / 16) {
        case 2: return launch_tile<2>(a, s);
        case 3: return launch_tile<3>(a, s);
        case 4: return launch_tile<4>(a, s);
        case 5: return launch_tile<5>(a, s);
        case 6: return launch_tile<6>(a, s);
        case 7: return launch_tile<7>(a, s);
        default: return launch_tile<8>(a, s);
        }
    }
    if (a.H <= 64) {
        if (a.H == 64)
            hipLaunchKernelGGL((project_kernel<1, true>), dim3(a.K), dim3(14 * 64), 0, s, a);
        else
            hipLaunchKernelGGL((project_kernel<1, false>), dim3(a.K), dim3(14 * 64), 0, s, a);
    } else {
        if (a.H == 128)
            hipLaunchKernelGGL((project_kernel<2, true>), dim3(a.K), dim3(14 * 64), 0, s, a);
        else
            hipLaunchKernelGGL((project_kernel<2, false>), dim3(a.K), dim3(14 * 64), 0, s, a);
    }
}

}  // namespace mppi
