// Shared by the plain and the robust source updates and the A/C pass: the
// downweighting function, a group reduction, and the per-source tail of the
// S block (Sect. 5.1): Algorithms C1-C3 on the 5x5 normal equations, the
// diagonal of the inverse (first-order variances, Sect. 5.1.1), Q_i of
// eq:Qi, the update (alpha through d_1 / cos delta) and the per-source record
// the time-ordered pass gathers.
#pragma once

#include "model.h"

namespace agis {

// acc: the 15 upper-triangle entries of N (row-major), the 5 of b and h'Wh.
// rhs (optional, [n_src][5]) receives b; eps_i2 goes into the record.
__device__ __forceinline__ void source_finish(const double acc[21], int64_t i, double alpha, double delta,
                                              double plx, double pma, double pmd, double cd, double* __restrict__ s,
                                              SrcPrep* __restrict__ prep, double* __restrict__ ds,
                                              double* __restrict__ qsrc, int32_t* __restrict__ sdef,
                                              double* __restrict__ svar, double* __restrict__ rhs = nullptr,
                                              double eps_i2 = 0.0) {
    double U[25], x[5];
    {
        int e = 0;
#pragma unroll
        for (int rr = 0; rr < 5; ++rr)
#pragma unroll
            for (int cc = rr; cc < 5; ++cc) U[rr * 5 + cc] = acc[e++];
    }
#pragma unroll
    for (int rr = 0; rr < 5; ++rr) x[rr] = acc[15 + rr];
    if (rhs)
#pragma unroll
        for (int rr = 0; rr < 5; ++rr) rhs[5 * i + rr] = acc[15 + rr];
    const int d = small_chol_factor<5>(U);
    small_chol_subst<5>(U, x);
    // diagonal of the inverse normal matrix V V', V = U^-1 (upper triangular,
    // row by row from its last), the first-order variances of the five
    // parameters (Sect. 5.1.1)
    double V[25];
#pragma unroll
    for (int kk = 4; kk >= 0; --kk) {
        V[kk * 5 + kk] = U[kk * 5 + kk];
        double sum = V[kk * 5 + kk] * V[kk * 5 + kk];
#pragma unroll
        for (int cc = kk + 1; cc < 5; ++cc) {
            double t = 0.0;
#pragma unroll
            for (int m = kk + 1; m <= cc; ++m) t += U[kk * 5 + m] * V[m * 5 + cc];
            V[kk * 5 + cc] = -t * U[kk * 5 + kk];
            sum += V[kk * 5 + cc] * V[kk * 5 + cc];
        }
        svar[5 * i + kk] = d > 0 ? 0.0 : sum;
    }
    // Q_i = h'Wh - 2 d'b + d'N d (eq:Qi)
    double dNd = 0.0, db = 0.0;
    {
        int e = 0;
#pragma unroll
        for (int rr = 0; rr < 5; ++rr) {
#pragma unroll
            for (int cc = rr; cc < 5; ++cc, ++e) dNd += (cc == rr ? 1.0 : 2.0) * acc[e] * x[rr] * x[cc];
            db += x[rr] * acc[15 + rr];
        }
    }
    qsrc[i] = acc[20] - 2.0 * db + dNd;
    sdef[i] = d;
#pragma unroll
    for (int rr = 0; rr < 5; ++rr) ds[5 * i + rr] = x[rr];
    const double na = alpha + x[0] / cd, nd = delta + x[1];
    const double npl = plx + x[2], npa = pma + x[3], npd = pmd + x[4];
    double* si = s + 5 * i;
    si[0] = na;
    si[1] = nd;
    si[2] = npl;
    si[3] = npa;
    si[4] = npd;
    double sa2, ca2, sd2, cd2;
    sincos(na, &sa2, &ca2);
    sincos(nd, &sd2, &cd2);
    SrcPrep pr;
    const double p2[3] = {-sa2, ca2, 0.0};
    const double q2[3] = {-sd2 * ca2, -sd2 * sa2, cd2};
    pr.r[0] = cd2 * ca2;
    pr.r[1] = cd2 * sa2;
    pr.r[2] = sd2;
    for (int cc = 0; cc < 3; ++cc) pr.mu[cc] = p2[cc] * npa + q2[cc] * npd;
    pr.plx = npl;
    pr.pad = eps_i2;                      // the source's excess noise eps_i^2 (robust mode 2)
    prep[i] = pr;
}

// Downweighting function w(z) of eq:dw.
__device__ __forceinline__ double down_weight(double z) {
    const double a = fabs(z);
    if (a <= 2.0) return 1.0;
    if (a < 3.0) {
        const double t = a - 2.0;
        return 1.0 - 1.773735 * t * t + 1.141615 * t * t * t;
    }
    return exp(-a / 3.0);
}

// Value of v in another lane of the 16-lane row (DPP pattern CTRL).
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Sum over groups of G neighbouring lanes (every lane of the group gets it):
// within a 16-lane row by register moves (mirrored row, mirrored half row,
// swapped pairs, swapped lanes), across rows through LDS permutes.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
    if constexpr (G >= 64) v += __shfl_xor(v, 32, 64);
    if constexpr (G >= 32) v += __shfl_xor(v, 16, 64);
    if constexpr (G >= 16) v += row_move<0x140>(v);
    if constexpr (G >= 8) v += row_move<0x141>(v);
    if constexpr (G >= 4) v += row_move<0x4E>(v);
    if constexpr (G >= 2) v += row_move<0xB1>(v);
    return v;
}

}  // namespace agis
