// The three kernels that carry the iteration's cost.
//
//   k_source_update<G>  S block (Sect. 5.1).  G lanes per source stream the
//                       source's observations (by-source store), evaluate the
//                       model and the design row (Sect. 5.1.3) and accumulate
//                       the 15 + 5 sums of eq:normS in registers; a butterfly
//                       over the G lanes reduces them; one lane per source
//                       runs Algorithms C1-C3 on the 5x5 system and applies
//                       the update.
//   k_ac_pass           A/C accumulation (Sect. 5.2.1, 5.2.4, 5.3).  One
//                       wavefront per one to eight knot intervals streams
//                       the time-ordered store at (s^(k+1), a^(k), c^(k)) and
//                       sums, on the FP64 matrix cores, the 10 block pairs x
//                       10 unique entries of eq:normAmod, its 16
//                       right-hand-side entries and the per-fov calibration
//                       sums of eq:normC.
//   k_band_solve        A solve (Sect. 5.2.2, App. C): one wavefront per
//                       segment; right-looking modified band Cholesky
//                       (Algorithm C1 with C2 folded in) as a moving 16x16
//                       front in registers, four scalar pivots and one
//                       matrix-core update per coefficient; then C3; the
//                       segment keeps its selected coefficients.
//
// Each lane walks its item's observations with stride G and loads the next
// observation's columns while the current one is evaluated.  No global
// atomics; all sums have a fixed order.
#include <algorithm>
#include <type_traits>

#include "agis_internal.h"
#include "source_block.h"

namespace agis {

namespace {

// pair index of (n, m), 0 <= n <= m <= 3 (also the entry index of (r, c))
__host__ __device__ __forceinline__ int tri4(int n, int m) { return n * 4 - (n * (n - 1)) / 2 + (m - n); }


// ------------------------------------------------------------------ S block
// Compensated (Kahan) single-precision running sum: s + (-c) carries the sum.
__device__ __forceinline__ void kahan_add(float& s, float& c, float x) {
    const float y = x - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

// AC: the observations may include across-scan ones (cell/fov code from
// k.ac_cf0 on); the along-scan-only instance is the plain pass.  SigT: the
// type of the sigma column (float: the input; double: the frozen sigma_eff
// of the hybrid scheme).
template <int G, bool MIXED, bool AC, typename SigT, bool DEFL = false>
__global__ __launch_bounds__(256, 2) void k_source_update(DevConsts k, int64_t n_src, const int64_t* __restrict__ off,
                                                       const double* __restrict__ ot, const double* __restrict__ oeta,
                                                       const SigT* __restrict__ osig,
                                                       const int32_t* __restrict__ ocell,
                                                       const int32_t* __restrict__ oell,
                                                       const double* __restrict__ knots,
                                                       const KnotTab* __restrict__ ktab, const double* __restrict__ a,
                                                       const double* __restrict__ c, double* __restrict__ s,
                                                       SrcPrep* __restrict__ prep, double* __restrict__ ds,
                                                       double* __restrict__ qsrc, int32_t* __restrict__ sdef,
                                                       double* __restrict__ svar, const int32_t* __restrict__ order,
                                                       double* __restrict__ rhs) {
    constexpr int GPB = 256 / G;
    __shared__ double pool[GPB][23];
    const int gl = threadIdx.x % G;
    // group k takes the k-th source of the launch order
    const int64_t kg = (int64_t)blockIdx.x * GPB + threadIdx.x / G;
    const bool valid = kg < n_src;
    const int64_t i = valid ? order[kg] : 0;
    double alpha = 0.0, delta = 0.0, plx = 0.0, pma = 0.0, pmd = 0.0;
    int64_t l0 = 0, l1 = 0;
    if (valid) {
        const double* si = s + 5 * i;
        alpha = si[0];
        delta = si[1];
        plx = si[2];
        pma = si[3];
        pmd = si[4];
        l0 = off[i];
        l1 = off[i + 1];
    }
    double sa, ca, sd, cd;
    sincos(alpha, &sa, &ca);
    sincos(delta, &sd, &cd);
    const double p[3] = {-sa, ca, 0.0};
    const double q[3] = {-sd * ca, -sd * sa, cd};
    const double r[3] = {cd * ca, cd * sa, sd};
    double mu[3];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) mu[cc] = p[cc] * pma + q[cc] * pmd;

    double acc[21];
#pragma unroll
    for (int e = 0; e < 21; ++e) acc[e] = 0.0;
    // mixed precision: the 15 normal-matrix sums from single-precision
    // partials with compensation; the right-hand side and h'Wh stay FP64,
    // so the iteration's fixed point is the FP64 one (the FP32 matrix only
    // changes the path to it)
    float fs[MIXED ? 15 : 1], fc[MIXED ? 15 : 1];
#pragma unroll
    for (int e = 0; e < (MIXED ? 15 : 1); ++e) fs[e] = fc[e] = 0.0f;
    int64_t l = l0 + gl;
    // Current observation: columns, and the gathered attitude coefficients,
    // interval table entry and calibration of its cell.  The next
    // observation's columns load at the top of an iteration, its gathers
    // after the current observation has been evaluated.
    double t_c = 0.0, e_c = 0.0, cal_c = 0.0;
    SigT s_c = 1;
    int32_t ell_c = 3;
    bool ac_c = false;
    double a_c[16];
    KnotTab kt_c = {0.0, 1.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 16; ++e) a_c[e] = 0.0;
    if (l < l1) {
        t_c = ot[l];
        e_c = oeta[l];
        s_c = osig[l];
        ell_c = oell[l];
        const int32_t cf = ocell[l];
        cal_c = c[cf >> 1];
        ac_c = AC && cf >= k.ac_cf0;
        const double* a4 = a + 4 * (ell_c - 3);
#pragma unroll
        for (int e = 0; e < 16; ++e) a_c[e] = a4[e];
        kt_c = ktab[ell_c - 3];
    }
    for (; l < l1; l += G) {
        const int64_t ln = l + G;
        const bool more = ln < l1;
        double t_n = 0.0, e_n = 0.0;
        SigT s_n = 1;
        int32_t c_n = 0, ell_n = 3;
        if (more) {
            t_n = ot[ln];
            e_n = oeta[ln];
            s_n = osig[ln];
            c_n = ocell[ln];
            ell_n = oell[ln];
        }
        ObsEval o;
        observe<DEFL>(k, t_c, e_c, cal_c, r, mu, plx, a_c, knots + (ell_c - 2), kt_c, o, ac_c);
        double A[5];
        source_partials(o, p, q, r, A, ac_c);
        const double sg = (double)s_c;
        const double W = rcp_nr(sg * sg);
        if constexpr (MIXED) {
            float Af[5];
#pragma unroll
            for (int rr = 0; rr < 5; ++rr) Af[rr] = (float)A[rr];
            const float Wf = (float)W;
            int e = 0;
#pragma unroll
            for (int rr = 0; rr < 5; ++rr) {
                const float wa = Wf * Af[rr];
#pragma unroll
                for (int cc = rr; cc < 5; ++cc) {
                    kahan_add(fs[e], fc[e], wa * Af[cc]);
                    ++e;
                }
            }
#pragma unroll
            for (int rr = 0; rr < 5; ++rr) acc[15 + rr] += W * A[rr] * o.R;
            acc[20] += W * o.R * o.R;
        } else {
            int e = 0;
#pragma unroll
            for (int rr = 0; rr < 5; ++rr) {
                const double wa = W * A[rr];
#pragma unroll
                for (int cc = rr; cc < 5; ++cc) acc[e++] += wa * A[cc];
            }
#pragma unroll
            for (int rr = 0; rr < 5; ++rr) acc[15 + rr] += W * A[rr] * o.R;
            acc[20] += W * o.R * o.R;
        }
        t_c = t_n;
        e_c = e_n;
        s_c = s_n;
        ell_c = ell_n;
        if (more) {
            cal_c = c[c_n >> 1];
            ac_c = AC && c_n >= k.ac_cf0;
            const double* a4 = a + 4 * (ell_n - 3);
#pragma unroll
            for (int e2 = 0; e2 < 16; ++e2) a_c[e2] = a4[e2];
            kt_c = ktab[ell_n - 3];
        }
    }
    if constexpr (MIXED) {
#pragma unroll
        for (int e = 0; e < 15; ++e) acc[e] = (double)fs[e] - (double)fc[e];
    }
#pragma unroll
    for (int e = 0; e < 21; ++e) acc[e] = group_sum<G>(acc[e]);
    // the block's sources finish in the first lanes of its first wavefront: by
    // the group leaders, one lane in G, every wavefront would run the solves
    // (20,000 sources 44 -> 36 us, 1M sources of 223 records 4.24 -> 4.16 ms)
    if (gl == 0) {
#pragma unroll
        for (int e = 0; e < 21; ++e) pool[threadIdx.x / G][e] = acc[e];
        pool[threadIdx.x / G][21] = cd;
    }
    __syncthreads();
    if (threadIdx.x >= GPB) return;
    const int64_t kf = (int64_t)blockIdx.x * GPB + threadIdx.x;
    if (kf >= n_src) return;
    const int64_t fi = order[kf];
    double sum[21];
#pragma unroll
    for (int e = 0; e < 21; ++e) sum[e] = pool[threadIdx.x][e];
    const double* si = s + 5 * fi;
    source_finish(sum, fi, si[0], si[1], si[2], si[3], si[4], pool[threadIdx.x][21], s, prep, ds, qsrc, sdef, svar, rhs);
}

// ------------------------------------------------------------- A/C pass
typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// A row of the transposition buffer.  FP64: B_0..B_3, 1, [fov +1], [fov -1],
// then b; the reading lanes form a's products, so that three wavefronts' buffers
// per SIMD fit a compute unit's LDS (160 KB in granules of 1,280 bytes: two
// doubles more a row leave room for 11 blocks instead of 12, and cost 1.5% to 3%,
// 111M records 2.78 ms instead of 2.71).  Mixed precision: a, then b.  (Odd
// strides, in doubles: no bank conflicts between the rows' writes.)
constexpr int AC_ROW = 23, AC_B = 7;
constexpr int AC_ROW_MIXED = 33;

// Slots of an interval of n records, and how many of a chunk's 64 lie before
// slot `end`.  Unsigned: a range may hold every record of a survey, up to 2^31 -
// 1, and its slots, and the chunk after them, reach past 2^31.
__host__ __device__ constexpr uint32_t ac_slots(uint32_t n) { return (n + 3) & ~3u; }
__host__ __device__ constexpr int ac_left(uint32_t end, uint32_t base) {
    return end - base < 64 ? (int)(end - base) : 64;
}
constexpr uint32_t AC_MOST = ac_slots(0x7FFFFFFFu) + 4 * 8;
static_assert(ac_slots(0x7FFFFFFFu) == 0x80000000u && ac_left(AC_MOST, 0) == 64 && ac_left(AC_MOST, AC_MOST - 4) == 4 &&
              AC_MOST + 128 > AC_MOST, "the slots of the largest survey");

// The A/C pass's gathers, one chunk of 64 records ahead.
struct AcRecord {
    double t, e, cal, ea;
    int32_t cf;
    int iv;                                // knot interval within the wavefront's range
    int32_t pos;                           // place in the geometric calibration's group order, or -1
    bool mine;                             // the lane's slot holds an observation
    SrcPrep sp;
};

// A/C accumulation as a matrix product on the FP64 matrix cores.  Every
// observation of knot interval j gives two 16-vectors
//   a = (B_n B_m for the 10 pairs n <= m, B_0..B_3, [fov +1], [fov -1])
//   b = (10 unique entries of W (g g' + 4 lambda^2 q q'),
//        -W (g R - 2 lambda^2 q D) (4), W, W R)
// and the interval's sums are blocks of C = sum over observations of a b'
// (16 x 16): pairs x entries (eq:normAmod), B_n x right-hand side, and
// fov x (W, W R) for eq:normC.  One wavefront takes `range` (at most RANGE)
// neighbouring knot intervals, 64 observations at a time (one per lane), writes b and the factors
// of a to LDS and feeds them to v_mfma_f64_16x16x4 steps of four observations
// of one interval each, in an order that does not depend on the range (nor do
// the sums).
//
// An interval of 15 to 300 observations by itself leaves 29% to 88% of the
// lanes' slots filled and starts the loads anew each time; over eight they
// follow on (97%; 4 and 16 intervals: 4% and 2% slower at 1.6 million intervals).
// Fewer intervals with more records each are shared out more evenly in shorter
// ranges: agis_ac_pass_range below.
//
// A SIMD's FP64 products and FP64 arithmetic share a pipe within a wavefront but
// not between them.  Counters at 223M observations: vector issue 57% of the
// SIMDs' cycles, matrix unit 32%, no bank conflicts, 2.9 wavefronts per SIMD
// that wait for 47% of their time: latencies bound it, at three wavefronts per
// SIMD (168 registers and 12 bytes of scratch a lane, robust 100; 12.4 KB).  1M
// sources, 223M observations: 7.65 -> 5.17 ms (27 bytes of columns and, by
// source, a seventh of a 64-byte record per observation; variants, against 5.29
// before the shorter rows: two wavefronts 5.9; the next columns asked for before
// the rows are written 5.37; 12 of 16 blocks by v_mfma_f64_4x4x4, whose operands
// take two more reads, 5.49).
//
// Mixed precision (MIXED): the model stays FP64; a and b are formed in FP32
// from single-precision partials, each 64-observation chunk is summed by
// v_mfma_f32_16x16x4 and the chunk sums enter compensated (Kahan) FP32
// running sums, converted to FP64 for the band solve.
// AC: across-scan observations present (cell/fov code from k.ac_cf0 on):
// their rows carry the AC attitude partials and no calibration entries.
template <bool MIXED, bool AC, typename SigT, bool DEFL, bool ROBUST, int RANGE>
__global__ __launch_bounds__(64, MIXED ? 2 : 3) void k_ac_pass(DevConsts k, int64_t K, const int64_t* __restrict__ iv_off,
                                                   const double* __restrict__ ot, const double* __restrict__ oeta,
                                                   const SigT* __restrict__ osig,
                                                   const int32_t* __restrict__ ocellfov,
                                                   const int32_t* __restrict__ osrc,
                                                   const SrcPrep* __restrict__ prep,
                                                   const double* __restrict__ knots,
                                                   const KnotTab* __restrict__ ktab, const double* __restrict__ a,
                                                   const double* __restrict__ c, const double* __restrict__ eps_a2,
                                                   int robust, int range, double* __restrict__ iv_sums,
                                                   double* __restrict__ iv_cal, double* __restrict__ wr_out,
                                                   const int32_t* __restrict__ wr_pos) {
    static_assert(!MIXED || RANGE == 1, "the FP64 sums of mixed precision belong to one interval");
    using XT = typename std::conditional<MIXED, float, double>::type;
    constexpr int ROW = MIXED ? AC_ROW_MIXED : AC_ROW;
    __shared__ __align__(16) XT xw[64][ROW];
    __shared__ __align__(16) double sh_a[4 * (RANGE + 3)];
    __shared__ __align__(16) double sh_k[4 * RANGE];
    static_assert(MIXED || 12 * ((sizeof(xw) + sizeof(sh_a) + sizeof(sh_k) + 1279) / 1280) <= 128,
                  "twelve wavefronts in a compute unit's LDS");
    const int lane = threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.x * range;
    const int count = (int)(K - j0 < range ? K - j0 : range);
    const int64_t first = iv_off[j0];
    // Slots for the range's observations, each interval's from a multiple of
    // four on: no step of four observations spans two intervals.  Lane i holds
    // the end of interval i's slots, what turns its slots into observations
    // counted from the range's first, and the end of these.
    uint32_t ends, shift, stop;
    {
        const int64_t jl = j0 + (lane < count ? lane : count - 1);
        const uint32_t start = (uint32_t)(iv_off[jl] - first);
        stop = (uint32_t)(iv_off[jl + 1] - first);
        const uint32_t slots = lane < count ? ac_slots(stop - start) : 0;
        ends = slots;
#pragma unroll
        for (int m = 1; m < RANGE; m <<= 1) {
            const uint32_t below = __shfl_up(ends, m, 64);
            ends += lane >= m ? below : 0;
        }
        shift = start - (ends - slots);
    }
    if (lane < 4 * (count + 3)) sh_a[lane] = a[4 * j0 + lane];
    if (lane < 4 * count) sh_k[lane] = reinterpret_cast<const double*>(ktab + j0)[lane];
    auto lane_of = [](uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    const uint32_t n = lane_of(ends, count - 1);
    const double lam2x4 = 4.0 * k.lam2;
    const int ri = lane & 15, rk = lane >> 4;
    // this lane's operands of step kk, 4 kk rows on (FP64: a is a product of two
    // entries)
    const XT *at, *at2 = nullptr, *atb;
    if constexpr (MIXED) {
        at = &xw[rk][ri];
        atb = &xw[rk][16 + ri];
    } else {
        const int f1 = ri < 4 ? 0 : ri < 7 ? 1 : ri < 9 ? 2 : ri < 10 ? 3 : ri < 14 ? ri - 10 : ri - 9;
        const int f2 = ri < 4 ? ri : ri < 7 ? ri - 3 : ri < 9 ? ri - 5 : ri < 10 ? 3 : 4;
        at = &xw[rk][f1];
        at2 = &xw[rk][f2];
        atb = &xw[rk][AC_B + ri];
    }
    double4_t C = {0.0, 0.0, 0.0, 0.0};
    float4_t Cs = {0.0f, 0.0f, 0.0f, 0.0f}, Cc = {0.0f, 0.0f, 0.0f, 0.0f};
    // mixed precision: the right-hand sides (B_n times the 4 attitude
    // right-hand sides, and W, WR per field of view) are summed per lane in
    // FP64 and reduced over the wavefront at the end, so the fixed point of
    // the iteration is the FP64 one
    double rb[MIXED ? 16 : 1], cb[MIXED ? 4 : 1];
#pragma unroll
    for (int e = 0; e < (MIXED ? 16 : 1); ++e) rb[e] = 0.0;
#pragma unroll
    for (int e = 0; e < (MIXED ? 4 : 1); ++e) cb[e] = 0.0;

    // Where this lane's sums of the first interval go, and how far the next
    // one's are.  Lane l holds C[4 v + l / 16][l % 16] (FP64 product) or
    // C[4 (l / 16) + v][l % 16] (FP32 product), v = 0..3.  FP64: v = 0, 1 are
    // pairs, the lower half of v = 2 too, the upper half and the lower one of v
    // = 3 right-hand sides, the rest calibration sums.
    double* out = iv_sums + j0 * IV_SUMS + rk * 10 + ri;
    double* out2 = iv_sums + j0 * IV_SUMS + (rk < 2 ? 80 + rk * 10 + ri : 92 + (rk - 2) * 4 + (ri - 2));
    double* out3 = rk < 2 ? iv_sums + j0 * IV_SUMS + 98 + rk * 4 + ri
                          : iv_cal + j0 * IV_CAL + (rk - 2) * 2 + (ri - 14);
    const int step3 = rk < 2 ? IV_SUMS : IV_CAL;
    const bool mid = ri >= 10 && ri < 14;
    const bool has2 = rk < 2 ? ri < 10 : mid, has3 = rk < 2 ? mid : ri >= 14;
    // the sums of interval `now` go out
    int now = 0;
    auto flush = [&]() {
        if constexpr (MIXED) {
            const int64_t j = j0 + now;
            double* to = iv_sums + j * IV_SUMS;
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
#pragma unroll
                for (int e = 0; e < 16; ++e) rb[e] += __shfl_xor(rb[e], m, 64);
#pragma unroll
                for (int e = 0; e < 4; ++e) cb[e] += __shfl_xor(cb[e], m, 64);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 4 * rk + v;
                if (i < 10 && ri < 10) to[i * 10 + ri] = (double)Cs[v] - (double)Cc[v];
            }
            // every lane holds the reduced FP64 sums; lane e writes entry e
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (lane == e) to[100 + e] = rb[e];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (lane == 16 + e) iv_cal[j * IV_CAL + e] = cb[e];
        } else {
            if (ri < 10) {
                out[0] = C[0];
                out[40] = C[1];
            }
            if (has2) *out2 = C[2];
            if (has3) *out3 = C[3];
            out += IV_SUMS;
            out2 += IV_SUMS;
            out3 += step3;
            C = double4_t{0.0, 0.0, 0.0, 0.0};
        }
        ++now;
    };

    // columns two chunks ahead, gathers one; a slot without an observation
    // takes its interval's last again, with weight zero
    double t_n = 0.0, e_n = 0.0;
    SigT s_n = 1, s_g = 1;
    int32_t cf_n = 0, src_n = 0, pos_n = -1, iv_n = 0;
    bool mine_n = false;
    AcRecord g = {};
    int iv_load = 0;                       // interval of the first slot to load
    auto load = [&](uint32_t base) {
        const uint32_t slot = base + lane < n ? base + lane : n - 1;
        iv_n = iv_load;
        uint32_t by = lane_of(shift, iv_load), past = lane_of(stop, iv_load);
        while (iv_load + 1 < count) {
            const uint32_t end = lane_of(ends, iv_load);
            if (end > base + 64) break;
            ++iv_load;
            const bool on = slot >= end;
            iv_n = on ? iv_load : iv_n;
            by = on ? lane_of(shift, iv_load) : by;
            past = on ? lane_of(stop, iv_load) : past;
        }
        const uint32_t at = slot + by;
        mine_n = at < past && base + lane < n;
        // from a base that the wavefront shares: a slot is at most 3 RANGE
        // further on than its observation
        constexpr int BACK = 4 * RANGE;
        const int64_t from = first + base - BACK;
        const uint32_t l = (at < past ? at : past - 1) - base + BACK;
        auto column = [&](auto* p) {
            return *reinterpret_cast<decltype(p)>(reinterpret_cast<const char*>(p + from) + (uint32_t)(l * sizeof(*p)));
        };
        t_n = column(ot);
        e_n = column(oeta);
        s_n = column(osig);
        cf_n = column(ocellfov);
        src_n = column(osrc);
        if (wr_out) pos_n = column(wr_pos);
    };
    auto gather = [&]() {
        g.t = t_n;
        g.e = e_n;
        g.cf = cf_n;
        g.pos = mine_n ? pos_n : -1;
        g.iv = iv_n;
        g.mine = mine_n;
        s_g = s_n;
        g.sp = prep[src_n];
        g.cal = c[cf_n >> 1];
        if constexpr (ROBUST) g.ea = eps_a2[eps_slot(k, cf_n, j0 + iv_n)];
    };
    __syncthreads();
    if (n > 0) {
        load(0);
        gather();
        if (n > 64) load(64);
    }
    for (uint32_t base = 0; base < n; base += 64) {
        const bool ac = AC && g.cf >= k.ac_cf0;
        TimeRow o;
        {
            double p[16];
            const double2_t* own = reinterpret_cast<const double2_t*>(sh_a + 4 * g.iv);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double2_t v = own[i];
                p[2 * i] = v.x;
                p[2 * i + 1] = v.y;
            }
            const double2_t* own_k = reinterpret_cast<const double2_t*>(sh_k + 4 * g.iv);
            const double2_t k0 = own_k[0], k1 = own_k[1];
            const KnotTab kt = {k0.x, k0.y, k1.x, k1.y};
            time_row<AC, DEFL>(k, g.sp, p, kt, knots + (j0 + g.iv + 1), g.t, g.e + g.cal, ac, o);
        }
        const double sg = (double)s_g;
        double W;
        if constexpr (ROBUST) {
            // sigma~^2 = sigma^2 + eps_a^2 of the record's component in the
            // interval's bucket; robust mode 2: plus the source's excess noise
            // eps_i^2 (eq:W)
            const double s2 = sg * sg + g.ea + (robust == 2 ? g.sp.pad : 0.0);
            W = down_weight(o.R * rsqrt_nr(s2)) * rcp_nr(s2);
        } else {
            W = rcp_nr(sg * sg);
        }
        W = g.mine ? W : 0.0;
        // geometric calibration: each along-scan record's W and W R for its C
        // block, at its place in the group order
        if (g.pos >= 0) reinterpret_cast<double2_t*>(wr_out)[g.pos] = double2_t{W, W * o.R};
        const int f = g.cf & 1;
        // the next chunk's gathers, and the columns of the one after it
        if (base + 64 < n) {
            gather();
        }
        XT* row = xw[lane];
        if constexpr (MIXED) {
            float B[4], gf[4], qf[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                B[m] = (float)o.B[m];
                gf[m] = (float)o.g[m];
                qf[m] = (float)o.q[m];
            }
            const float Wf = (float)W, Rf = (float)o.R, Df = (float)o.D, l2 = (float)k.lam2;
            int e = 0;
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int mm = m; mm < 4; ++mm) row[e++] = B[m] * B[mm];
#pragma unroll
            for (int m = 0; m < 4; ++m) row[e++] = B[m];
            row[e++] = (f == 0 && !ac) ? 1.0f : 0.0f;
            row[e++] = (f == 1 && !ac) ? 1.0f : 0.0f;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int cc = rr; cc < 4; ++cc) row[e++] = Wf * (gf[rr] * gf[cc] + 4.0f * l2 * qf[rr] * qf[cc]);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) row[e++] = -Wf * (gf[rr] * Rf - 2.0f * l2 * qf[rr] * Df);
            row[e++] = Wf;
            row[e] = Wf * Rf;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const double rhs = -W * (o.g[rr] * o.R - 0.5 * lam2x4 * o.q[rr] * o.D);
#pragma unroll
                for (int m = 0; m < 4; ++m) rb[4 * m + rr] += o.B[m] * rhs;
            }
            if (!ac) {
                cb[2 * f] += W;
                cb[2 * f + 1] += W * o.R;
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4; ++m) row[m] = o.B[m];
            row[4] = 1.0;
            row[5] = (f == 0 && !ac) ? 1.0 : 0.0;
            row[6] = (f == 1 && !ac) ? 1.0 : 0.0;
            double wg[4], wq[4];
            const double wl = W * lam2x4;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                wg[m] = W * o.g[m];
                wq[m] = wl * o.q[m];
            }
            XT* b = row + AC_B;
            int e = 0;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int cc = rr; cc < 4; ++cc) b[e++] = wg[rr] * o.g[cc] + wq[rr] * o.q[cc];
            const double hd = 0.5 * o.D;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) b[10 + rr] = wq[rr] * hd - wg[rr] * o.R;
            b[14] = W;
            b[15] = W * o.R;
        }
        wave_fence();
        if constexpr (MIXED) {
            if (base + 128 < n) load(base + 128);
            // groups of four observations past the interval's end hold padding
            // rows of weight zero: their matrix-core steps would add zeros
            const int steps = (ac_left(n, base) + 3) >> 2;
            float4_t Ck = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) {
                if (kk >= steps) break;
                const int d = 4 * kk * ROW;
                Ck = __builtin_amdgcn_mfma_f32_16x16x4f32(at[d], atb[d], Ck, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float sv = Cs[v], cv = Cc[v];
                kahan_add(sv, cv, Ck[v]);
                Cs[v] = sv;
                Cc[v] = cv;
            }
        } else {
            // operands of four steps in registers while the next four load (their
            // latency, up to 300 clocks, is longer than a step's product, 64)
            double av[4], zv[4], bv[4], an[4], zn[4], bn[4];
            int end = ac_left(lane_of(ends, now), base);
            auto fetch = [&](int q, double x[4], double z[4], double y[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    x[u] = at[(16 * q + 4 * u) * ROW];
                    z[u] = at2[(16 * q + 4 * u) * ROW];
                    y[u] = atb[(16 * q + 4 * u) * ROW];
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto steps = [&](int row, double x[4], const double z[4], const double y[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] *= z[u];
                if (end - row >= 16) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) C = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u], y[u], C, 0, 0, 0);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        // the interval's sums are complete (and empty ones')
                        while (row + 4 * u >= end && now + 1 < count) {
                            flush();
                            end = ac_left(lane_of(ends, now), base);
                        }
                        if (row + 4 * u < end) C = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u], y[u], C, 0, 0, 0);
                    }
                }
            };
            fetch(0, av, zv, bv);
            if (base + 128 < n) load(base + 128);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
            for (int q = 0; q < 4; q += 2) {
                fetch(q + 1, an, zn, bn);
                steps(16 * q, av, zv, bv);
                if (q < 2) fetch(q + 2, av, zv, bv);
                steps(16 * q + 16, an, zn, bn);
            }
        }
        wave_fence();
    }
    // the last interval, and the empty ones before and after the observations
    while (now < count) flush();
}

// ------------------------------------------------------------ band solve
// Value of v in another lane of the 16-lane row (DPP).  CTRL 0x150 + n
// broadcasts lane n of the row, 0x100 + n reads lane + n, 0x110 + n reads
// lane - n, 0x120 + n rotates by n; lanes with no source read 0.
template <int CTRL>
__device__ __forceinline__ double row_dpp(double v) {
    if constexpr (CTRL >= 0x150) {
        return __builtin_amdgcn_update_dpp(0.0, v, CTRL, 0xF, 0xF, true);   // one 64-bit move
    } else {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
        return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
    }
}

// old, with the quads (four-lane banks of each 16-lane row) of BANKS taken
// from v moved by CTRL.
template <int CTRL, int BANKS>
__device__ __forceinline__ double quad_dpp(double old, double v) {
    const uint64_t o = __builtin_bit_cast(uint64_t, old), b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)b, CTRL, 0xF, BANKS, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(b >> 32), CTRL, 0xF, BANKS,
                                               false);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// The four 16-lane rows of v, each in all four rows: r[p](lane 16 q + d) =
// v(lane 16 p + d), by row swaps (no LDS).
__device__ __forceinline__ void gather_rows(double v, double (&r)[4]) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    uint32_t h[2][4];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const uint32_t x = w ? (uint32_t)(b >> 32) : (uint32_t)b;
        const auto y = __builtin_amdgcn_permlane32_swap(x, x, false, false);      // rows 0 1 0 1, rows 2 3 2 3
        const auto lo = __builtin_amdgcn_permlane16_swap(y[0], y[0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(y[1], y[1], false, false);
        h[w][0] = lo[0];
        h[w][1] = lo[1];
        h[w][2] = hi[0];
        h[w][3] = hi[1];
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) r[p] = __builtin_bit_cast(double, ((uint64_t)h[1][p] << 32) | h[0][p]);
}

constexpr int BAND_AHEAD = 4;           // intervals in flight before their use
constexpr int BAND_BACK = 8;            // factor blocks in flight on the way back

// Modified band Cholesky of the attitude segments (Algorithms C1-C3 with
// half bandwidth 15, Sect. 5.2.2), one wavefront per segment.  The system is
// eliminated as a moving 16x16 front: interval k couples coefficients
// k .. k+3, so its sums are added to the front just before the four rows of
// coefficient k are eliminated.  Lane 16 q + d holds, of front rows 4i + q (i
// = 0..3), the entry at column offset d from the diagonal block: W[i] =
// entry (4(k+i) + q, 4(k+i) + d); a zero or negative pivot gives a zero
// factor row and counts one defect.
//  * The four pivot rows are copied to all four 16-lane rows and eliminated
//    there by row broadcasts (scalar pivots in their order, as C1 asks), with
//    the right-hand side (R: lane d holds row 4k + d).
//  * With the factor rows back in place (row q in 16-lane row q), lane
//    c + 4b + 16q holds element (q, c) of the 4x4 block U(k, k+b): the operand
//    layout of v_mfma_f64_4x4x4 with its four blocks b.  The update
//    W[i](block b) -= U(k, k+i)' U(k, k+i+b) is then one matrix instruction
//    per i, whose operands are U shifted by i blocks and block i repeated.
// C3 runs back up the segment: each 16-lane row forms the product of its
// factor row with the known unknowns, the 4x4 triangle is solved by all lanes.
//
// Bound by the instruction issue of the serial chain (about 170 instructions
// per coefficient forward, 110 back): a segment's time is its length, whatever
// else runs, until there are several segments per SIMD.  Before, one 16-lane
// row per segment, per scalar pivot 15 shifted and 15 broadcast rank-1 columns
// and the entering row summed from an LDS ring took 1340 us for 110 segments
// of 264 intervals, 1726 us for 12,138 of 154; this form takes 184 and 920 us.
__global__ __launch_bounds__(64) void k_band_solve(const SegDesc* __restrict__ segs,
                                                   const double* __restrict__ iv_sums, double* __restrict__ ufac,
                                                   double* __restrict__ yfac, double* __restrict__ da,
                                                   int32_t* __restrict__ seg_def) {
    const int lane = threadIdx.x;
    const int d = lane & 15, q = lane >> 4, c = d & 3, g = d >> 2;
    const SegDesc sd = segs[blockIdx.x];
    const int nb = (int)(sd.n_hi - sd.n_lo + 1);       // coefficients; intervals: nb - 3
    const int n_iv = nb - 3;
    const double* sums = iv_sums + sd.n_lo * IV_SUMS;
    double* U = ufac + sd.u_off * 16 + lane;
    double* Y = yfac + sd.u_off + q;
    // the lane's entries of an interval: front block (n, n + g), entry (q, c),
    // for n + g <= 3 (others are read from block (n, 3) and taken zero times)
    const int e = q < c ? tri4(q, c) : tri4(c, q);
    int at[4];
    double use[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int m = n + g < 3 ? n + g : 3;
        at[n] = tri4(n, m) * 10 + e;
        use[n] = n + g <= 3 ? 1.0 : 0.0;
    }
    double nw[BAND_AHEAD][4], nr[BAND_AHEAD];
    auto fetch = [&](int k, int slot) {
        const double* iv = sums + (int64_t)(k < n_iv ? k : n_iv - 1) * IV_SUMS;
#pragma unroll
        for (int n = 0; n < 4; ++n) nw[slot][n] = iv[at[n]];
        nr[slot] = iv[100 + d];
    };
#pragma unroll
    for (int u = 0; u < BAND_AHEAD; ++u) fetch(u, u);
    double W[4] = {0.0, 0.0, 0.0, 0.0};
    double R = 0.0;
    int defect = 0;
    for (int k0 = 0; k0 < nb; k0 += BAND_AHEAD) {
#pragma unroll
        for (int u = 0; u < BAND_AHEAD; ++u) {
            const int k = k0 + u;
            if (k >= nb) break;
            if (k < n_iv) {
#pragma unroll
                for (int n = 0; n < 4; ++n) W[n] = __builtin_fma(nw[u][n], use[n], W[n]);
                R += nr[u];
            }
            fetch(k + BAND_AHEAD, u);
            double P[4], y[4];
            gather_rows(W[0], P);
            auto pivot = [&](auto pc) {
                constexpr int p = decltype(pc)::value;
                const double piv = row_dpp<0x150 + p>(P[p]);
                const double inv = rsqrt_pivot(piv);
                defect += piv > 0.0 ? 0 : 1;
                P[p] *= inv;
                y[p] = row_dpp<0x150 + p>(R) * inv;
                if constexpr (p < 1) P[1] -= row_dpp<0x151>(P[p]) * P[p];
                if constexpr (p < 2) P[2] -= row_dpp<0x152>(P[p]) * P[p];
                if constexpr (p < 3) P[3] -= row_dpp<0x153>(P[p]) * P[p];
                R -= P[p] * y[p];
            };
            pivot(std::integral_constant<int, 0>{});
            pivot(std::integral_constant<int, 1>{});
            pivot(std::integral_constant<int, 2>{});
            pivot(std::integral_constant<int, 3>{});
            R = row_dpp<0x104>(R);
            const double X = q < 2 ? (q == 0 ? P[0] : P[1]) : (q == 2 ? P[2] : P[3]);
            const double yq = q < 2 ? (q == 0 ? y[0] : y[1]) : (q == 2 ? y[2] : y[3]);
            U[(int64_t)k * 64] = X;
            if (d == 0) Y[4 * (int64_t)k] = yq;
            // blocks i, i+1, .. in places 0, 1, ..; and block i in each place
            // that front row i has
            const double b1 = row_dpp<0x104>(X), b2 = row_dpp<0x108>(X), b3 = row_dpp<0x10C>(X);
            const double a1 = quad_dpp<0x114, 0x4>(quad_dpp<0x104, 0x1>(X, X), X);
            const double a2 = quad_dpp<0x104, 0x2>(b2, X);
            W[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(-a1, b1, W[1], 0, 0, 0);
            W[1] = __builtin_amdgcn_mfma_f64_4x4x4f64(-a2, b2, W[2], 0, 0, 0);
            W[2] = __builtin_amdgcn_mfma_f64_4x4x4f64(-b3, b3, W[3], 0, 0, 0);
            W[3] = 0.0;
        }
    }
    __syncthreads();   // forward-substituted y visible to all lanes
    // Algorithm C3 from the last coefficient up: x in lane d is the unknown
    // 4k + d, d >= 4, when coefficient k is solved (0 in lanes 0..3)
    double fX[BAND_BACK], fY[BAND_BACK];
    auto fetch_back = [&](int k, int slot) {
        const int64_t kk = k > 0 ? k : 0;
        fX[slot] = U[kk * 64];
        fY[slot] = Y[4 * kk];
    };
#pragma unroll
    for (int u = 0; u < BAND_BACK; ++u) fetch_back(nb - 1 - u, u);
    double x = 0.0;
    for (int k0 = nb - 1; k0 >= 0; k0 -= BAND_BACK) {
#pragma unroll
        for (int u = 0; u < BAND_BACK; ++u) {
            const int k = k0 - u;
            if (k < 0) break;
            const double X = fX[u], yq = fY[u];
            fetch_back(k - BAND_BACK, u);
            // reciprocal pivots (0 where the factor row is zero) on the diagonal
            const double iv = X > 0.0 ? rcp_nr(X) : 0.0;
            double T[4], S[4];
            gather_rows(d == q ? iv : X, T);
            double t = X * x;
            t += row_dpp<0x128>(t);
            t += row_dpp<0x124>(t);
            t += row_dpp<0x122>(t);
            t += row_dpp<0x121>(t);
            gather_rows(yq - t, S);
            const double x3 = S[3] * row_dpp<0x153>(T[3]);
            const double x2 = (S[2] - row_dpp<0x153>(T[2]) * x3) * row_dpp<0x152>(T[2]);
            const double x1 = (S[1] - row_dpp<0x153>(T[1]) * x3 - row_dpp<0x152>(T[1]) * x2) * row_dpp<0x151>(T[1]);
            const double x0 = (S[0] - row_dpp<0x153>(T[0]) * x3 - row_dpp<0x152>(T[0]) * x2 -
                               row_dpp<0x151>(T[0]) * x1) * row_dpp<0x150>(T[0]);
            const double xs = c < 2 ? (c == 0 ? x0 : x1) : (c == 2 ? x2 : x3);
            const int64_t n = sd.n_lo + k;
            if (n >= sd.keep_lo && n <= sd.keep_hi && lane < 4) da[4 * n + lane] = xs;
            x = row_dpp<0x114>(d < 4 ? xs : x);
        }
    }
    if (lane == 0) seg_def[blockIdx.x] = defect;
}

inline int groups_grid(int64_t n_items, int items_per_block) {
    return (int)((n_items + items_per_block - 1) / items_per_block);
}

}  // namespace

#define AGIS_S_KERNEL(G, T)                                                                                    \
    (ctx->cfg.precision == AGIS_MIXED                                                                          \
         ? (ctx->has_ac ? k_source_update<G, true, true, T> : k_source_update<G, true, false, T>)               \
         : (ctx->has_ac ? k_source_update<G, false, true, T> : k_source_update<G, false, false, T>))
#define AGIS_S_ARGS(SIG)                                                                                       \
    ctx->k, ctx->n_src, ctx->src_off, ctx->s_t, ctx->s_eta, SIG, ctx->s_cell, ctx->s_ell, ctx->knots, ctx->ktab,   \
        ctx->a, ctx->c, ctx->s, ctx->prep, ctx->ds, ctx->qsrc, ctx->sdef, ctx->svar, ctx->src_order, ctx->rhs_s_out
#define AGIS_S_LAUNCH(G)                                                                                       \
    if (ctx->k.defl > 0.0)                                                                                     \
        (ctx->has_ac ? k_source_update<G, false, true, float, true> : k_source_update<G, false, false, float, true>) \
            <<<groups_grid(ctx->n_src, 256 / G), 256, 0, ctx->stream>>>(AGIS_S_ARGS(ctx->s_sig));            \
    else if (ctx->frozen)                                                                                      \
        AGIS_S_KERNEL(G, double)<<<groups_grid(ctx->n_src, 256 / G), 256, 0, ctx->stream>>>(                  \
            AGIS_S_ARGS(ctx->s_sig_eff));                                                                      \
    else                                                                                                       \
        AGIS_S_KERNEL(G, float)<<<groups_grid(ctx->n_src, 256 / G), 256, 0, ctx->stream>>>(AGIS_S_ARGS(ctx->s_sig))

void launch_source_update(agis_ctx* ctx) {
    if (ctx->n_src == 0) return;
    switch (ctx->s_group) {
        case 8: AGIS_S_LAUNCH(8); break;
        case 16: AGIS_S_LAUNCH(16); break;
        case 32: AGIS_S_LAUNCH(32); break;
        default: AGIS_S_LAUNCH(64); break;
    }
}

// Knot intervals per wavefront of the A/C pass, at most.
constexpr int AC_RANGE = 8;

template <typename KERN, typename T>
static void ac_launch(agis_ctx* ctx, KERN kern, int range, const T* sig) {
    kern<<<(unsigned)((ctx->K + range - 1) / range), 64, 0, ctx->stream>>>(
        ctx->k, ctx->K, ctx->iv_off, ctx->t_t, ctx->t_eta, sig, ctx->t_cellfov, ctx->t_src, ctx->prep, ctx->knots,
        ctx->ktab, ctx->a, ctx->c, ctx->eps_a2, robust_now(ctx), range, ctx->iv_sums, ctx->iv_cal,
        ctx->geo_ccds > 0 ? ctx->geo_wr : nullptr, ctx->geo_pos);
}

template <bool ROBUST, typename T>
static void ac_pass_with(agis_ctx* ctx, const T* sig) {
    if (ctx->cfg.precision == AGIS_MIXED) {
        ac_launch(ctx, ctx->has_ac ? k_ac_pass<true, true, T, false, ROBUST, 1>
                                   : k_ac_pass<true, false, T, false, ROBUST, 1>, 1, sig);
        return;
    }
    auto kern = ctx->has_ac ? k_ac_pass<false, true, T, false, ROBUST, AC_RANGE>
                            : k_ac_pass<false, false, T, false, ROBUST, AC_RANGE>;
    if constexpr (std::is_same<T, float>::value) {
        // the model with the Sun's light deflection (FP64 only, as the
        // global block requires)
        if (ctx->k.defl > 0.0)
            kern = ctx->has_ac ? k_ac_pass<false, true, T, true, ROBUST, AC_RANGE>
                               : k_ac_pass<false, false, T, true, ROBUST, AC_RANGE>;
    }
    ac_launch(ctx, kern, ctx->ac_range, sig);
}

void launch_ac_pass(agis_ctx* ctx) {
    if (ctx->K == 0) return;
    if (ctx->frozen)
        ac_pass_with<false>(ctx, ctx->t_sig_eff);
    else if (robust_now(ctx))
        ac_pass_with<true>(ctx, ctx->t_sig);
    else
        ac_pass_with<false>(ctx, ctx->t_sig);
}

void launch_band_solve(agis_ctx* ctx) {
    const int64_t nseg = (int64_t)ctx->h_segs.size();
    if (nseg == 0) return;
    k_band_solve<<<(unsigned)nseg, 64, 0, ctx->stream>>>(ctx->segs, ctx->iv_sums, ctx->ufac, ctx->yfac, ctx->da,
                                                         ctx->seg_def);
}

}  // namespace agis

// Knot intervals per wavefront of the FP64 A/C pass: 1, 2, 4 or 8, whichever
// takes least by this count.  A wavefront takes the chunks of 64 slots that its
// intervals' observations fill, and about two more to start and end; the device
// holds 3 x 1,024 wavefronts, and the longest runs on while it empties, nine
// tenths of its time.  Long ranges win where intervals are many and short, by
// fewer and fuller chunks; short ones where they are few and long, by sharing
// out evenly.  Measured (ms for ranges of 1, 2, 4, 8; the choice in brackets):
//   4,383 intervals of 6,099 records   [0.737] 0.863  1.197  1.634
//   17,532 of 1,525                    [0.615] 0.627  0.715  0.841
//   39,447 of 678                       0.632 [0.603] 0.624  0.706
//   39,447 of 113                       0.153  0.134 [0.130] 0.138
//   473,364 of 141                      2.039  1.749  1.652 [1.625]
//   17,532 of 17                        0.042  0.027  0.028 [0.025]
// Eleven other shapes: at most 1.2% more than the best.
extern "C" int32_t agis_ac_pass_range(int64_t n_intervals, const int64_t* off) {
    int32_t best = 1;
    double least = 0.0;
    for (int32_t r = 1; r <= agis::AC_RANGE; r *= 2) {
        int64_t total = 0, longest = 0;
        for (int64_t j0 = 0; j0 < n_intervals; j0 += r) {
            int64_t slots = 0;
            for (int64_t j = j0; j < std::min(j0 + r, n_intervals); ++j) slots += (off[j + 1] - off[j] + 3) & ~int64_t(3);
            const int64_t chunks = (slots + 63) / 64 + 2;
            total += chunks;
            longest = std::max(longest, chunks);
        }
        const double time = (double)total / 3072.0 + 0.9 * (double)longest;
        if (r == 1 || time < least) {
            best = r;
            least = time;
        }
    }
    return best;
}
