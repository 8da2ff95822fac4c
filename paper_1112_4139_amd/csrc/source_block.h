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

// The source's data for source_row(); returns cos(delta).
__device__ __forceinline__ double source_dir(const DevConsts& k, double alpha, double delta, double plx, double pma,
                                             double pmd, SourceDir& o) {
    double sa, ca, sd, cd;
    sincos(alpha, &sa, &ca);
    sincos(delta, &sd, &cd);
    o.p0 = -sa;
    o.p1 = ca;
    o.q[0] = -sd * ca;
    o.q[1] = -sd * sa;
    o.q[2] = cd;
    o.r[0] = cd * ca;
    o.r[1] = cd * sa;
    o.r[2] = sd;
    o.mu[0] = o.p0 * pma + o.q[0] * pmd;
    o.mu[1] = o.p1 * pma + o.q[1] * pmd;
    o.mu[2] = o.q[2] * pmd;
    o.plx_r = plx * k.eph_r;
    return cd;
}

// A knot interval's record in the stage of the S pass: its four spline
// coefficients (16 neighbouring doubles of the attitude), then its KnotTab.
typedef double double2_t __attribute__((ext_vector_type(2)));
constexpr int AT_DOUBLES = 20;
constexpr int AT_BYTES = AT_DOUBLES * 8;

// The wavefront's stage for up to 64 of these records, six to a load
// instruction (10 lanes of 16 bytes each; the last four lanes write the rest of
// its KB), then the records' interval list.
constexpr int STAGE_LOADS = 11, STAGE_AHEAD = 5;
constexpr int STAGE_RECORDS = STAGE_LOADS * 1024;
constexpr int STAGE_LIST = 6 * STAGE_LOADS;
constexpr int STAGE_BYTES = STAGE_RECORDS + (STAGE_LIST + 2) * 4;

// One wavefront's records of the by-source store as a pipeline: lane by lane
// first, first + step, .. < end.  A record's columns load OBS_AHEAD records
// before it (2: 3 and 4 cost registers and 2%), and one record before it the
// attitude records of the knot intervals that the wavefront's 64 records lie
// in.  The observations of a transit (up to nine, 5 s apart) share an interval
// and neighbour each other, so lanes with the interval of the lane before them
// take that lane's record: only the distinct ones are loaded, each by ten
// neighbouring lanes, and go through LDS, where every lane reads its own (160
// bytes apart: no bank conflicts).  Each lane loading its own record (ten
// 16-byte loads) kept the address units busy for 83% of the S pass: with
// source_row(), 1M sources of 223 records 3.83 -> 3.54 ms (65% of it FP64 and
// integer issue at two wavefronts per SIMD; a third one spills).  (Loads
// straight to LDS made the compiler wait for each before the next list entry.
// Launching the sources of one scan together halved the traffic to HBM and
// gained nothing.)
// All lanes of the wavefront run every step; past its end a lane reads its last
// record again.  Slots are compile-time constants (the caller unrolls).
// EPS: also the excess attitude noise of the record's component and bucket.
constexpr int OBS_AHEAD = 2;

// Orders the wavefront's LDS accesses before and after it (which the hardware
// executes in order) for the compiler.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename SigT, bool EPS = false>
struct ObsStream {
    const double *ot, *oeta;
    const SigT* osig;
    const int32_t *ocell, *oell;
    const double *a, *knots;
    const KnotTab* ktab;
    const double *c, *eps_a2;
    char* stage;                         // this wavefront's STAGE_BYTES of LDS
    int64_t next;                        // record to load next, and how far the lane's last one is
    int ahead, step;
    double t[OBS_AHEAD], e[OBS_AHEAD];
    SigT s[OBS_AHEAD];
    int32_t cf[OBS_AHEAD], ell[OBS_AHEAD];
    double cal, ea;
    double2_t rec[STAGE_AHEAD];          // this lane's 16 bytes of the records on their way
    int n;                               // records (the same in all lanes)
    int at;                              // this lane's record in the stage [bytes]
    const char* from;                    // this lane's 16 bytes of interval 0's record
    int want;                            // its first entry of the interval list [bytes]

    __device__ __forceinline__ void load(int u) {
        t[u] = ot[next];
        e[u] = oeta[next];
        s[u] = osig[next];
        cf[u] = ocell[next];
        ell[u] = oell[next];
        const int go = ahead >= step ? step : 0;
        next += go;
        ahead -= go;
    }
    // past the list's n entries: older ones, intervals too
    __device__ __forceinline__ double2_t fetch(int i) const {
        const uint32_t j = *reinterpret_cast<const uint32_t*>(stage + STAGE_RECORDS + want + 24 * i);
        return *reinterpret_cast<const double2_t*>(from + 32 * (uint64_t)j);
    }
    __device__ __forceinline__ void gather(const DevConsts& k, int u) {
        const int32_t j = ell[u] - 3;
        if constexpr (EPS) ea = eps_a2[eps_slot(k, cf[u], j)];
        cal = c[cf[u] >> 1];
        // a new record where the interval differs from the lane before
        // (the first lane of a 16-lane row always has one)
        const int32_t before = __builtin_amdgcn_update_dpp(-1, j, 0x111, 0xF, 0xF, false);
        const uint64_t fresh = __ballot(j != before);
        n = __popcll(fresh);
        const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(fresh >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)fresh, 0u)) -
                      (j != before ? 0 : 1);
        if (j != before) reinterpret_cast<int32_t*>(stage + STAGE_RECORDS)[r] = j;
        at = r * AT_BYTES + ((r * 43) >> 8) * 64;                  // six to a KB
        wave_fence();
        // a year of nine-record transits needs 2 or 3 loads
        rec[0] = fetch(0);
        rec[1] = fetch(1);
        if (n > 12) {
            rec[2] = fetch(2);
            if (n > 18)
#pragma unroll
                for (int i = 3; i < STAGE_AHEAD; ++i) rec[i] = fetch(i);
        }
    }
    // the records on their way to the stage; more than 30 are loaded here
    __device__ __forceinline__ void arrive() const {
        double2_t* to = reinterpret_cast<double2_t*>(stage) + (threadIdx.x & 63);
        to[0] = rec[0];
        to[64] = rec[1];
        if (n > 12) {
            to[128] = rec[2];
            if (n > 18)
#pragma unroll
                for (int i = 3; i < STAGE_AHEAD; ++i) to[64 * i] = rec[i];
            if (n > 6 * STAGE_AHEAD) {
                double2_t more[STAGE_LOADS - STAGE_AHEAD];
#pragma unroll
                for (int i = STAGE_AHEAD; i < STAGE_LOADS; ++i) more[i - STAGE_AHEAD] = fetch(i);
#pragma unroll
                for (int i = STAGE_AHEAD; i < STAGE_LOADS; ++i) to[64 * i] = more[i - STAGE_AHEAD];
            }
        }
        wave_fence();
    }
    // end > first record of the store; a lane with first >= end reads its last
    __device__ __forceinline__ void start(int64_t first, int64_t end, int step_) {
        const int64_t last = end > 0 ? end - 1 : 0;
        step = step_;
        next = first < last ? first : last;
        ahead = (int)(last - next);
        const int lane = threadIdx.x & 63, sixth = (lane * 205) >> 11, part = lane - 10 * sixth;  // lane / 10, lane % 10
        from = part < 8 ? reinterpret_cast<const char*>(a) + 16 * part
                        : reinterpret_cast<const char*>(ktab) + 16 * (part - 8);
        want = 4 * (sixth < 5 ? sixth : 5);
        reinterpret_cast<int32_t*>(stage + STAGE_RECORDS)[lane] = 0;
        if (lane < STAGE_LIST - 64) reinterpret_cast<int32_t*>(stage + STAGE_RECORDS)[64 + lane] = 0;
        wave_fence();
#pragma unroll
        for (int u = 0; u < OBS_AHEAD; ++u) load(u);
    }
    __device__ __forceinline__ void take(const DevConsts& k, int u, double qa[4], double& sL, double& cL) const {
        arrive();
        double p[AT_DOUBLES];
        const double2_t* own = reinterpret_cast<const double2_t*>(stage + at);
#pragma unroll
        for (int i = 0; i < AT_DOUBLES / 2; ++i) {
            const double2_t v = own[i];
            p[2 * i] = v.x;
            p[2 * i + 1] = v.y;
        }
        wave_fence();
        const KnotTab kt = {p[16], p[17], p[18], p[19]};
        const double dt = t[u] - kt.tau;
        attitude_at(p, kt, dt, knots + (ell[u] - 2), t[u], qa);
        orbit_at(k, kt, dt, t[u], sL, cL);
    }
    // the record of slot u has been taken: the next one's gathers, and a new
    // record for its slot
    __device__ __forceinline__ void advance(const DevConsts& k, int u) {
        gather(k, (u + 1) % OBS_AHEAD);
        load(u);
    }
};

// Trips of the wavefront's record loop: its largest group's.
template <int G>
__device__ __forceinline__ int wave_trips(int64_t l0, int64_t l1) {
    int n = (int)((l1 - l0 + G - 1) / G);
#pragma unroll
    for (int m = 32; m >= G; m >>= 1) {
        const int o = __shfl_xor(n, m, 64);
        n = o > n ? o : n;
    }
    return __builtin_amdgcn_readfirstlane(n);
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
