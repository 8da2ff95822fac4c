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
//                       wavefront per knot interval streams the time-ordered
//                       store at (s^(k+1), a^(k), c^(k)) and sums, on the FP64
//                       matrix cores, the 10 block pairs x 10 unique entries
//                       of eq:normAmod, its 16 right-hand-side entries and the
//                       per-fov calibration sums of eq:normC.
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
                                                       const double* __restrict__ knots, const KnotTab* __restrict__ ktab,
                                                       const double* __restrict__ a,
                                                       const double* __restrict__ c, double* __restrict__ s,
                                                       SrcPrep* __restrict__ prep, double* __restrict__ ds,
                                                       double* __restrict__ qsrc, int32_t* __restrict__ sdef,
                                                       double* __restrict__ svar, const int32_t* __restrict__ order,
                                                       double* __restrict__ rhs) {
    constexpr int GPB = 256 / G;
    __shared__ double pool[GPB][23];
    __shared__ __align__(16) char stage[4][STAGE_BYTES];
    const int gl = threadIdx.x % G;
    // group k takes the k-th source of the launch order
    const int64_t kb = (int64_t)blockIdx.x * GPB;
    const int64_t kg = kb + threadIdx.x / G;
    const bool valid = kg < n_src;
    SourceDir sd;
    int64_t l0 = 0, l1 = 0;
    double cd;
    ObsStream<SigT> st{ot, oeta, osig, ocell, oell, a, knots, ktab, c, nullptr, stage[threadIdx.x >> 6]};
    int trips, mine;                     // the wavefront's and this lane's records
    {
        double alpha = 0.0, delta = 0.0, plx = 0.0, pma = 0.0, pmd = 0.0;
        if (valid) {
            const int64_t i = order[kg];
            l0 = off[i];
            l1 = off[i + 1];
            const double* si = s + 5 * i;
            alpha = si[0];
            delta = si[1];
            plx = si[2];
            pma = si[3];
            pmd = si[4];
        }
        trips = wave_trips<G>(l0, l1);
        mine = (int)(l1 - l0 - gl + G - 1) / G;
        if (trips > 0) st.start(l0 + gl, l1, G);
        cd = source_dir(k, alpha, delta, plx, pma, pmd, sd);
        if (trips > 0) st.gather(k, 0);
    }
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
    auto record = [&](int u, int at) {
        double qa[4], sL, cL;
        st.take(k, u, qa, sL, cL);
        const double t = st.t[u], obs = st.e[u] + st.cal;
        const bool ac = AC && st.cf[u] >= k.ac_cf0;
        const double sg = (double)st.s[u];
        st.advance(k, u);
        if (at >= mine) return;
        double A[5], R, tau;
        source_row<AC, DEFL>(k, sd, qa, sL, cL, t - k.t_ep, obs, ac, A, R, tau);
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
        }
        int e = 0;
#pragma unroll
        for (int rr = 0; rr < 5; ++rr) {
            const double wa = W * A[rr];
            if constexpr (!MIXED) {
#pragma unroll
                for (int cc = rr; cc < 5; ++cc) acc[e++] += wa * A[cc];
            }
            acc[15 + rr] += wa * R;
        }
        acc[20] += W * R * R;
    };
    for (int it = 0; it < trips; it += OBS_AHEAD) {
#pragma unroll
        for (int u = 0; u < OBS_AHEAD; ++u) {
            if (it + u >= trips) break;
            record(u, it + u);
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
    // (with division-free solves: 20,000 sources 44 -> 27 us, 1M sources of
    // 223 records 4.25 -> 3.83 ms)
    if (gl == 0) {
#pragma unroll
        for (int e = 0; e < 21; ++e) pool[threadIdx.x / G][e] = acc[e];
        pool[threadIdx.x / G][21] = cd;
    }
    __syncthreads();
    if (threadIdx.x >= GPB) return;
    const int64_t kf = kb + threadIdx.x;
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

constexpr int AC_WAVES = 1;             // wavefronts per block, one knot interval each (2 and 4 measured 4% and 7% slower)
constexpr int AC_XS = 33;               // LDS row stride (doubles) of the transposition buffer

// A/C accumulation as a matrix product on the FP64 matrix cores.  Every
// observation of knot interval j gives two 16-vectors
//   a = (B_n B_m for the 10 pairs n <= m, B_0..B_3, [fov +1], [fov -1])
//   b = (10 unique entries of W (g g' + 4 lambda^2 q q'),
//        -W (g R - 2 lambda^2 q D) (4), W, W R)
// and the interval's sums are blocks of C = sum over observations of a b'
// (16 x 16): pairs x entries (eq:normAmod), B_n x right-hand side, and
// fov x (W, W R) for eq:normC.  One wavefront takes 64 observations at a
// time (one per lane), writes (a, b) to LDS and feeds them to 16
// v_mfma_f64_16x16x4 steps, four observations each.
//
// Mixed precision (MIXED): the model stays FP64; a and b are formed in FP32
// from single-precision partials, each 64-observation chunk is summed by
// v_mfma_f32_16x16x4 and the chunk sums enter compensated (Kahan) FP32
// running sums, converted to FP64 for the band solve.
// AC: across-scan observations present (cell/fov code from k.ac_cf0 on):
// their rows carry the AC attitude partials and no calibration entries.
template <bool MIXED, bool AC, typename SigT, bool DEFL = false>
__global__ __launch_bounds__(64 * AC_WAVES) void k_ac_pass(DevConsts k, int64_t K, const int64_t* __restrict__ iv_off,
                                                           const double* __restrict__ ot,
                                                           const double* __restrict__ oeta,
                                                           const SigT* __restrict__ osig,
                                                           const int32_t* __restrict__ ocellfov,
                                                           const int32_t* __restrict__ osrc,
                                                           const SrcPrep* __restrict__ prep,
                                                           const double* __restrict__ knots,
                                                           const KnotTab* __restrict__ ktab,
                                                           const double* __restrict__ a,
                                                           const double* __restrict__ c,
                                                           const double* __restrict__ eps_a2, int eps_bucket,
                                                           int robust, double* __restrict__ iv_sums,
                                                           double* __restrict__ iv_cal, double* __restrict__ wr_out,
                                                           const int32_t* __restrict__ wr_pos) {
    using XT = typename std::conditional<MIXED, float, double>::type;
    __shared__ XT xb[AC_WAVES][64][AC_XS];
    __shared__ double sh_a[AC_WAVES][16];
    __shared__ double sh_k[AC_WAVES][6];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.x * AC_WAVES + wv;
    const bool valid = j < K;
    if (lane < 22) {
        double v = 0.0;
        if (valid) v = lane < 16 ? a[4 * j + lane] : knots[j + 1 + (lane - 16)];
        if (lane < 16) sh_a[wv][lane] = v;
        else sh_k[wv][lane - 16] = v;
    }
    __syncthreads();
    const double lam2 = k.lam2;
    const int64_t l0 = valid ? iv_off[j] : 0, l1 = valid ? iv_off[j + 1] : 0;
    const KnotTab kt = valid ? ktab[j] : KnotTab{0.0, 1.0, 0.0, 0.0};
    // robust: sigma~^2 = sigma^2 + eps_a^2 of the record's component in the
    // interval's bucket (eq:W)
    XT (*xw)[AC_XS] = xb[wv];
    const int ri = lane & 15, rk = lane >> 4;
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
    // lanes past the end evaluate the interval's last observation again with
    // weight zero
    int64_t base = l0;
    double t_c = 0.0, e_c = 0.0;
    SigT s_c = 1;
    int32_t cf_c = 0;
    bool h_c = false;
    SrcPrep sp_c = {};
    if (base < l1) {
        h_c = base + lane < l1;
        const int64_t le = h_c ? base + lane : l1 - 1;
        t_c = ot[le];
        e_c = oeta[le];
        s_c = osig[le];
        cf_c = ocellfov[le];
        sp_c = prep[osrc[le]];
    }
    for (; base < l1; base += 64) {
        const int64_t bn = base + 64;
        double t_n = 0.0, e_n = 0.0;
        SigT s_n = 1;
        int32_t cf_n = 0, src_n = 0;
        bool h_n = false;
        if (bn < l1) {
            h_n = bn + lane < l1;
            const int64_t le = h_n ? bn + lane : l1 - 1;
            t_n = ot[le];
            e_n = oeta[le];
            s_n = osig[le];
            cf_n = ocellfov[le];
            src_n = osrc[le];
        }
        {
            const bool ac = AC && cf_c >= k.ac_cf0;
            ObsEval o;
            observe<DEFL>(k, t_c, e_c, c[cf_c >> 1], sp_c.r, sp_c.mu, sp_c.plx, sh_a[wv], sh_k[wv], kt, o, ac);
            double g[4];
            attitude_partial(o, g, ac);
            const double sg = (double)s_c;
            double W;
            if (robust) {
                // robust mode 2: plus the source's excess noise eps_i^2 (eq:W)
                const double s2 = sg * sg + eps_a2[eps_slot(k, cf_c, j)] + (robust == 2 ? sp_c.pad : 0.0);
                W = h_c ? down_weight(o.R / sqrt(s2)) / s2 : 0.0;
            } else {
                W = h_c ? rcp_nr(sg * sg) : 0.0;
            }
            // geometric calibration: each along-scan record's W and W R for
            // its C block, at its place in the group order
            if (wr_out && h_c) {
                const int32_t p = wr_pos[base + lane];
                if (p >= 0) {
                    wr_out[2 * (int64_t)p] = W;
                    wr_out[2 * (int64_t)p + 1] = W * o.R;
                }
            }
            XT* row = xw[lane];
            const int f = cf_c & 1;
            if constexpr (MIXED) {
                float B[4], gf[4], qf[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    B[n] = (float)o.B[n];
                    gf[n] = (float)g[n];
                    qf[n] = (float)o.qraw[n];
                }
                const float Wf = (float)W, Rf = (float)o.R, Df = (float)o.D, l2 = (float)lam2;
                int e = 0;
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int m = n; m < 4; ++m) row[e++] = B[n] * B[m];
#pragma unroll
                for (int n = 0; n < 4; ++n) row[10 + n] = B[n];
                row[14] = (f == 0 && !ac) ? 1.0f : 0.0f;
                row[15] = (f == 1 && !ac) ? 1.0f : 0.0f;
                e = 0;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                    for (int cc = rr; cc < 4; ++cc) row[16 + e++] = Wf * (gf[rr] * gf[cc] + 4.0f * l2 * qf[rr] * qf[cc]);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) row[26 + rr] = -Wf * (gf[rr] * Rf - 2.0f * l2 * qf[rr] * Df);
                row[30] = Wf;
                row[31] = Wf * Rf;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const double rhs = -W * (g[rr] * o.R - 2.0 * lam2 * o.qraw[rr] * o.D);
#pragma unroll
                    for (int n = 0; n < 4; ++n) rb[4 * n + rr] += o.B[n] * rhs;
                }
                if (!ac) {
                    cb[2 * f] += W;
                    cb[2 * f + 1] += W * o.R;
                }
            } else {
                int e = 0;
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int m = n; m < 4; ++m) row[e++] = o.B[n] * o.B[m];
#pragma unroll
                for (int n = 0; n < 4; ++n) row[10 + n] = o.B[n];
                row[14] = (f == 0 && !ac) ? 1.0 : 0.0;
                row[15] = (f == 1 && !ac) ? 1.0 : 0.0;
                e = 0;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                    for (int cc = rr; cc < 4; ++cc)
                        row[16 + e++] = W * (g[rr] * g[cc] + 4.0 * lam2 * o.qraw[rr] * o.qraw[cc]);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) row[26 + rr] = -W * (g[rr] * o.R - 2.0 * lam2 * o.qraw[rr] * o.D);
                row[30] = W;
                row[31] = W * o.R;
            }
        }
        SrcPrep sp_n = {};
        if (bn < l1) sp_n = prep[src_n];
        // the rows just written are read back below by other lanes: a
        // workgroup barrier (the block is one wavefront, so it reduces to
        // waiting for the LDS stores) orders the stores before the reads
        __syncthreads();
        // groups of four observations past the interval's end hold padding
        // rows of weight zero: their matrix-core steps would add zeros
        const int64_t n_here = l1 - base < 64 ? l1 - base : 64;
        const int steps = (int)((n_here + 3) >> 2);
        if constexpr (MIXED) {
            float4_t Ck = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) {
                if (kk >= steps) break;
                const float av = xw[4 * kk + rk][ri];
                const float bv = xw[4 * kk + rk][16 + ri];
                Ck = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, Ck, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float sv = Cs[v], cv = Cc[v];
                kahan_add(sv, cv, Ck[v]);
                Cs[v] = sv;
                Cc[v] = cv;
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) {
                if (kk >= steps) break;
                const double av = xw[4 * kk + rk][ri];
                const double bv = xw[4 * kk + rk][16 + ri];
                C = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, C, 0, 0, 0);
            }
        }
        // the next chunk's stores overwrite these rows: every lane's reads
        // above come first
        __syncthreads();
        t_c = t_n;
        e_c = e_n;
        s_c = s_n;
        cf_c = cf_n;
        h_c = h_n;
        sp_c = sp_n;
    }
    if (!valid) return;
    if constexpr (MIXED) {
#pragma unroll
        for (int v = 0; v < 4; ++v) C[v] = (double)Cs[v] - (double)Cc[v];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
#pragma unroll
            for (int e = 0; e < 16; ++e) rb[e] += __shfl_xor(rb[e], m, 64);
#pragma unroll
            for (int e = 0; e < 4; ++e) cb[e] += __shfl_xor(cb[e], m, 64);
        }
    }
    // lane l holds C[4 v + l / 16][l % 16] (FP64 product) or
    // C[4 (l / 16) + v][l % 16] (FP32 product), v = 0..3
    double* out = iv_sums + j * IV_SUMS;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = MIXED ? 4 * rk + v : 4 * v + rk, jj = ri;
        if (i < 10 && jj < 10) out[i * 10 + jj] = C[v];
        else if (!MIXED && i >= 10 && i < 14 && jj >= 10 && jj < 14) out[100 + (i - 10) * 4 + (jj - 10)] = C[v];
        else if (!MIXED && i >= 14 && jj >= 14) iv_cal[j * IV_CAL + (i - 14) * 2 + (jj - 14)] = C[v];
    }
    if constexpr (MIXED) {
        // every lane holds the reduced FP64 sums; lane e writes entry e
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (lane == e) out[100 + e] = rb[e];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (lane == 16 + e) iv_cal[j * IV_CAL + e] = cb[e];
    }
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
// Bound by the instruction issue of the serial chain (about 150 instructions
// per coefficient forward, 110 back): a segment's time is its length, whatever
// else runs, until there are several segments per SIMD.  Before, one 16-lane
// row per segment, per scalar pivot 15 shifted and 15 broadcast rank-1 columns
// and the entering row summed from an LDS ring took 1340 us for 110 segments
// of 264 intervals, 1726 us for 12,138 of 154; this form takes 184 and 920 us.
__global__ __launch_bounds__(64) void k_band_solve(int64_t nseg, const SegDesc* __restrict__ segs,
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

template <typename T>
static void ac_pass_with(agis_ctx* ctx, const T* sig) {
    auto kern = ctx->cfg.precision == AGIS_MIXED
                    ? (ctx->has_ac ? k_ac_pass<true, true, T> : k_ac_pass<true, false, T>)
                    : (ctx->has_ac ? k_ac_pass<false, true, T> : k_ac_pass<false, false, T>);
    if constexpr (std::is_same<T, float>::value) {
        // the model with the Sun's light deflection (FP64 only, as the
        // global block requires)
        if (ctx->k.defl > 0.0) kern = ctx->has_ac ? k_ac_pass<false, true, float, true> : k_ac_pass<false, false, float, true>;
    }
    kern<<<(unsigned)((ctx->K + AC_WAVES - 1) / AC_WAVES), 64 * AC_WAVES, 0, ctx->stream>>>(
        ctx->k, ctx->K, ctx->iv_off, ctx->t_t, ctx->t_eta, sig, ctx->t_cellfov, ctx->t_src, ctx->prep, ctx->knots,
        ctx->ktab, ctx->a, ctx->c, ctx->eps_a2, ctx->cfg.eps_bucket, robust_now(ctx), ctx->iv_sums, ctx->iv_cal,
        ctx->geo_ccds > 0 ? ctx->geo_wr : nullptr, ctx->geo_pos);
}

void launch_ac_pass(agis_ctx* ctx) {
    if (ctx->K == 0) return;
    if (ctx->frozen)
        ac_pass_with(ctx, ctx->t_sig_eff);
    else
        ac_pass_with(ctx, ctx->t_sig);
}

void launch_band_solve(agis_ctx* ctx) {
    const int64_t nseg = (int64_t)ctx->h_segs.size();
    if (nseg == 0) return;
    k_band_solve<<<(unsigned)nseg, 64, 0, ctx->stream>>>(nseg, ctx->segs, ctx->iv_sums, ctx->ufac, ctx->yfac, ctx->da,
                                                         ctx->seg_def);
}

}  // namespace agis
