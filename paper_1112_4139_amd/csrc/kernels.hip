// Kernels of the C block, the frame rotator, residuals and statistics (the
// source update, the A/C accumulation pass and the band solve are in hot.hip).
//
//   k_calib_solve    per constraint pair: eq:normC solve and eq:calCon
//   frame rotator    eq:cond-mu3 normal equations (two-stage reduction),
//                    6x6 solve, rigorous source transform, eq:fr-q4
//
// No global atomics: every reduction has a fixed order, so results are
// bitwise reproducible run to run.
#include <algorithm>

#include "agis_internal.h"

namespace agis {

namespace {

constexpr int WAVE = 64;

// pair index of (n, m), 0 <= n <= m <= 3, and entry index of (r, c), r <= c
__device__ __forceinline__ int tri4(int n, int m) { return n * 4 - (n * (n - 1)) / 2 + (m - n); }

// ---------------------------------------------------------------- sources
// pad carries the source's excess noise eps_i^2 (robust mode 2; else 0)
__global__ __launch_bounds__(256) void k_prep_sources(int64_t n_src, const double* __restrict__ s,
                                                      const double* __restrict__ src_eps2,
                                                      SrcPrep* __restrict__ prep) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_src;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double* si = s + 5 * i;
        double sa, ca, sd, cd;
        sincos(si[0], &sa, &ca);
        sincos(si[1], &sd, &cd);
        SrcPrep o;
        const double p[3] = {-sa, ca, 0.0};
        const double q[3] = {-sd * ca, -sd * sa, cd};
        o.r[0] = cd * ca;
        o.r[1] = cd * sa;
        o.r[2] = sd;
        for (int c = 0; c < 3; ++c) o.mu[c] = p[c] * si[3] + q[c] * si[4];
        o.plx = si[2];
        o.pad = src_eps2 ? src_eps2[i] : 0.0;
        prep[i] = o;
    }
}

// x += dx and, in the same launch, y += dy
__global__ void k_apply_add(int64_t n, double* __restrict__ x, const double* __restrict__ dx, int64_t m,
                            double* __restrict__ y, const double* __restrict__ dy) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n + m; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < n) x[i] += dx[i];
        else y[i - n] += dy[i - n];
    }
}

// ------------------------------------------------------ calibration solve
// One block per constraint pair (cells 2j, 2j+1): eq:normC with Phi = 1
// (a 1x1 system per cell, Algorithms C1-C3), then eq:calCon.  rc
// (optional) receives each cell's right-hand side -sum W R.
__global__ __launch_bounds__(256) void k_calib_solve(int64_t n_cells, const int32_t* __restrict__ cell_iv,
                                                     const int32_t* __restrict__ iv_cell,
                                                     const double* __restrict__ iv_cal, double* __restrict__ c,
                                                     double* __restrict__ dc, double* __restrict__ rc) {
    __shared__ double red[256][2];
    __shared__ double dt[2];
    const int64_t pair = blockIdx.x;
    for (int h = 0; h < 2; ++h) {
        const int64_t cell = 2 * pair + h;
        double sw = 0.0, swr = 0.0;
        if (cell < n_cells) {
            const int32_t lo = cell_iv[2 * cell], hi = cell_iv[2 * cell + 1];
            for (int32_t j = lo + threadIdx.x; j < hi; j += blockDim.x) {
                for (int f = 0; f < 2; ++f) {
                    if (iv_cell[2 * j + f] == (int32_t)cell) {
                        sw += iv_cal[(int64_t)j * IV_CAL + 2 * f];
                        swr += iv_cal[(int64_t)j * IV_CAL + 2 * f + 1];
                    }
                }
            }
        }
        red[threadIdx.x][0] = sw;
        red[threadIdx.x][1] = swr;
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) {
                red[threadIdx.x][0] += red[threadIdx.x + s][0];
                red[threadIdx.x][1] += red[threadIdx.x + s][1];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            double U = red[0][0];
            double x = -red[0][1];
            if (rc && cell < n_cells) rc[cell] = x;
            double Um[1] = {U}, xm[1] = {x};
            small_chol_solve<1>(Um, xm);
            dt[h] = (cell < n_cells) ? xm[0] : 0.0;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int64_t c0 = 2 * pair, c1 = 2 * pair + 1;
        if (c1 < n_cells) {
            const double z = (dt[0] + dt[1]) / 2.0;
            const double d0 = dt[0] - z, d1 = dt[1] - z;
            dc[c0] = d0;
            dc[c1] = d1;
        } else if (c0 < n_cells) {
            dc[c0] = dt[0];
        }
    }
}

// Sums of NV values over the 256 threads of a block, in a fixed order: first
// over each wavefront (all NV exchanges of a step are independent), then over
// the four wavefronts; thread e receives sum e (e < NV).  A tree over LDS
// with a barrier per step took ten times as long as the data it summed.
template <int NV, bool MAX5 = false>
__device__ __forceinline__ double block_sums(double (&v)[NV], double (*red)[NV]) {
    // MAX5: values 5..9 are maxima
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            const double o = __shfl_xor(v[e], m, 64);
            v[e] = MAX5 && e >= 5 && e < 10 ? fmax(v[e], o) : v[e] + o;
        }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int e = 0; e < NV; ++e) red[threadIdx.x >> 6][e] = v[e];
    __syncthreads();
    const int e = threadIdx.x < NV ? threadIdx.x : 0;
    double s = red[0][e];
    for (int w = 1; w < 4; ++w) s = MAX5 && e >= 5 && e < 10 ? fmax(s, red[w][e]) : s + red[w][e];
    return s;
}

// ---------------------------------------------------------- frame rotator
constexpr int FR_BLOCKS = 512;
// Sums per block.  With rows (0, q), (0, -p), (q, tau q), (-p, -tau p) for
// mu_a*, mu_d, alpha*, delta (eq:cond-mu3, tau the same for every source) the
// 6x6 matrix is (E, tau E; tau E, F + tau^2 E), E = sum w_a q q' + w_d p p'
// and F the same with the weights of the proper motions, the right-hand side
// (u, v + tau u): 6 + 6 + 3 + 3 sums instead of 21 + 6.
constexpr int FR_VALS = 18;

// Weighted by the inverse variances of the last S update (eq:cond-mu3 rows
// for mu_a*, mu_d, alpha*, delta); zero or non-finite variance: zero weight.
// part: [FR_VALS][blocks].  Bound by the reduction for small catalogues
// (20,000 sources: 34 -> 9 us with the final sum below 53 -> 6 us).
__global__ __launch_bounds__(256) void k_frame_fit_partial(int64_t n_src, const double* __restrict__ s,
                                                           const double* __restrict__ sref,
                                                           const double* __restrict__ svar,
                                                           double* __restrict__ part) {
    __shared__ double red[4][FR_VALS];
    double acc[FR_VALS];
#pragma unroll
    for (int e = 0; e < FR_VALS; ++e) acc[e] = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_src;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double* x = s + 5 * i;
        const double* h = sref + 5 * i;
        const double* vi = svar + 5 * i;
        double sa, ca, sd, cd, sah, cah, sdh, cdh;
        sincos(x[0], &sa, &ca);
        sincos(x[1], &sd, &cd);
        sincos(h[0], &sah, &cah);
        sincos(h[1], &sdh, &cdh);
        const double p[3] = {-sa, ca, 0.0};
        const double q[3] = {-sd * ca, -sd * sa, cd};
        const double dr[3] = {cd * ca - cdh * cah, cd * sa - cdh * sah, sd - sdh};
        auto weight = [](double v) { return (v > 0.0 && isfinite(v)) ? 1.0 / v : 0.0; };
        const double wa = weight(vi[0]), wd = weight(vi[1]), wma = weight(vi[3]), wmd = weight(vi[4]);
        const double ra = wa * dot3(p, dr), rd = wd * dot3(q, dr);
        const double rma = wma * (x[3] - h[3]), rmd = wmd * (x[4] - h[4]);
        int e = 0;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
            for (int c = r; c < 3; ++c, ++e) {
                acc[e] += wa * q[r] * q[c] + wd * p[r] * p[c];
                acc[6 + e] += wma * q[r] * q[c] + wmd * p[r] * p[c];
            }
            acc[12 + r] += ra * q[r] - rd * p[r];
            acc[15 + r] += rma * q[r] - rmd * p[r];
        }
    }
    const double v = block_sums<FR_VALS>(acc, red);
    if (threadIdx.x < FR_VALS) part[threadIdx.x * FR_BLOCKS + blockIdx.x] = v;
}

// One wavefront per sum; its lanes take FR_BLOCKS / 64 partials each.
__global__ __launch_bounds__(1024) void k_frame_fit_final(DevConsts k, const double* __restrict__ part,
                                                          double* __restrict__ eo) {
    __shared__ double tot[FR_VALS];
    const int lane = threadIdx.x & 63;
    for (int e = threadIdx.x >> 6; e < FR_VALS; e += 16) {
        double v = 0.0;
#pragma unroll
        for (int b = 0; b < FR_BLOCKS / 64; ++b) v += part[e * FR_BLOCKS + 64 * b + lane];
        v = wave_sum(v);
        if (lane == 0) tot[e] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double tau = (k.t_ep - k.t_fr) / k.year_s;
    double U[36], x[6];
    int e = 0;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int c = r; c < 3; ++c, ++e) {
            U[r * 6 + c] = tot[e];
            U[r * 6 + 3 + c] = U[c * 6 + 3 + r] = tau * tot[e];
            U[(3 + r) * 6 + 3 + c] = tot[6 + e] + tau * tau * tot[e];
        }
        x[r] = tot[12 + r];
        x[3 + r] = tot[15 + r] + tau * tot[12 + r];
    }
    small_chol_solve<6>(U, x);
#pragma unroll
    for (int r = 0; r < 6; ++r) eo[r] = x[r];
}

// f(t) = Q[(t - t_fr) omega] Q(eps) (eq:fr1)
__device__ __forceinline__ void frame_quat(const DevConsts& k, const double* eo, double t, double f[4]) {
    const double dt = (t - k.t_fr) / k.year_s;
    const double wv[3] = {dt * eo[3], dt * eo[4], dt * eo[5]};
    double qw[4], qe[4];
    qrot(wv, qw);
    qrot(eo, qe);
    qmul(qw, qe, f);
}

// Rigorous transformation of the astrometric parameters (Sect. 6.1.2,
// steps 1-5) and of the source data used by the time-ordered pass.
__device__ __forceinline__ void frame_apply_sources(const DevConsts& k, int64_t first, int64_t stride, int64_t n_src,
                                                    const double* __restrict__ eo, double* __restrict__ s,
                                                    SrcPrep* __restrict__ prep) {
    double f[4], A[9];
    frame_quat(k, eo, k.t_ep, f);
    quat2mat(f, A);
    for (int64_t i = first; i < n_src; i += stride) {
        double* x = s + 5 * i;
        double sa, ca, sd, cd;
        sincos(x[0], &sa, &ca);
        sincos(x[1], &sd, &cd);
        const double pt[3] = {-sa, ca, 0.0};
        const double qt[3] = {-sd * ca, -sd * sa, cd};
        const double rt[3] = {cd * ca, cd * sa, sd};
        const double wxr[3] = {eo[4] * rt[2] - eo[5] * rt[1], eo[5] * rt[0] - eo[3] * rt[2],
                               eo[3] * rt[1] - eo[4] * rt[0]};
        double mut[3];
        for (int m = 0; m < 3; ++m) mut[m] = pt[m] * x[3] + qt[m] * x[4] - wxr[m];
        double rC[3], muC[3];
        for (int m = 0; m < 3; ++m) {
            rC[m] = A[3 * m] * rt[0] + A[3 * m + 1] * rt[1] + A[3 * m + 2] * rt[2];
            muC[m] = A[3 * m] * mut[0] + A[3 * m + 1] * mut[1] + A[3 * m + 2] * mut[2];
        }
        const double alpha = atan2(rC[1], rC[0]);
        const double delta = atan2(rC[2], sqrt(rC[0] * rC[0] + rC[1] * rC[1]));
        double sa2, ca2, sd2, cd2;
        sincos(alpha, &sa2, &ca2);
        sincos(delta, &sd2, &cd2);
        const double p[3] = {-sa2, ca2, 0.0};
        const double q[3] = {-sd2 * ca2, -sd2 * sa2, cd2};
        const double pma = dot3(p, muC), pmd = dot3(q, muC);
        x[0] = alpha;
        x[1] = delta;
        x[3] = pma;
        x[4] = pmd;
        SrcPrep o;
        o.r[0] = cd2 * ca2;
        o.r[1] = cd2 * sa2;
        o.r[2] = sd2;
        for (int m = 0; m < 3; ++m) o.mu[m] = p[m] * pma + q[m] * pmd;
        o.plx = x[2];
        o.pad = prep[i].pad;                  // the source's eps_i^2 stays
        prep[i] = o;
    }
}

// eq:fr-q4 with the support mid-time eq:RF4.
__device__ __forceinline__ void frame_apply_attitude(const DevConsts& k, int64_t first, int64_t stride, int64_t N,
                                                     const double* __restrict__ eo, const double* __restrict__ knots,
                                                     double* __restrict__ a) {
    for (int64_t n = first; n < N; n += stride) {
        const double tbar = 0.5 * (knots[n] + knots[n + 4]);
        double f[4];
        frame_quat(k, eo, tbar, f);
        const double fi[4] = {-f[0], -f[1], -f[2], f[3]};
        double* an = a + 4 * n;
        const double cur[4] = {an[0], an[1], an[2], an[3]};
        double r[4];
        qmul(fi, cur, r);
        an[0] = r[0];
        an[1] = r[1];
        an[2] = r[2];
        an[3] = r[3];
    }
}

// Both in one launch: the first src_blocks blocks take the sources.
__global__ __launch_bounds__(256) void k_frame_apply(DevConsts k, int src_blocks, int64_t n_src, int64_t N,
                                                     const double* __restrict__ eo, double* __restrict__ s,
                                                     SrcPrep* __restrict__ prep, const double* __restrict__ knots,
                                                     double* __restrict__ a) {
    const int64_t b = blockIdx.x;
    if (b < src_blocks)
        frame_apply_sources(k, b * 256 + threadIdx.x, (int64_t)src_blocks * 256, n_src, eo, s, prep);
    else
        frame_apply_attitude(k, (b - src_blocks) * 256 + threadIdx.x, (int64_t)(gridDim.x - src_blocks) * 256, N, eo,
                             knots, a);
}

// ------------------------------------------------------------ residuals
template <bool DEFL>
__global__ __launch_bounds__(256) void k_residuals(DevConsts k, int64_t K, const int64_t* __restrict__ iv_off,
                                                   const double* __restrict__ ot, const double* __restrict__ oeta,
                                                   const int32_t* __restrict__ ocellfov,
                                                   const int32_t* __restrict__ osrc,
                                                   const int32_t* __restrict__ operm, const SrcPrep* __restrict__ prep,
                                                   const double* __restrict__ knots,
                                                   const KnotTab* __restrict__ ktab, const double* __restrict__ a,
                                                   const double* __restrict__ c, double* __restrict__ R) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t j = (int64_t)blockIdx.x * (blockDim.x / WAVE) + (threadIdx.x / WAVE);
    if (j >= K) return;
    double a4[16], kn[6];
    for (int e = 0; e < 16; ++e) a4[e] = a[4 * j + e];
    for (int e = 0; e < 6; ++e) kn[e] = knots[j + 1 + e];
    const KnotTab kt = ktab[j];
    for (int64_t l = iv_off[j] + lane; l < iv_off[j + 1]; l += WAVE) {
        const SrcPrep sp = prep[osrc[l]];
        const int32_t cf = ocellfov[l];
        ObsEval o;
        observe<DEFL>(k, ot[l], oeta[l], c[cf >> 1], sp.r, sp.mu, sp.plx, a4, kn, kt, o, cf >= k.ac_cf0);
        R[operm[l]] = o.R;
    }
}

// ----------------------------------------------------------- statistics
// Per job (blockIdx.y): sums of squares and maxima per column of x [n][w],
// the sums of extra [n] and of iextra [n_i].  part: [job][12][blocks].
constexpr int ST_BLOCKS = 1024;

__global__ __launch_bounds__(256) void k_stats_partial(StatJobs jobs, double* __restrict__ part) {
    __shared__ double red[4][12];
    const StatJob jb = jobs.job[blockIdx.y];
    double v[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = first; i < jb.n; i += stride) {
#pragma unroll
        for (int cc = 0; cc < 5; ++cc)
            if (cc < jb.w) {
                const double x = jb.x[i * jb.w + cc];
                v[cc] += x * x;
                v[5 + cc] = fmax(v[5 + cc], fabs(x));
            }
        if (jb.extra) v[10] += jb.extra[i];
    }
    for (int64_t i = first; i < jb.n_i; i += stride) v[11] += (double)jb.iextra[i];
    const double s = block_sums<12, true>(v, red);
    if (threadIdx.x < 12) part[((int64_t)blockIdx.y * 12 + threadIdx.x) * gridDim.x + blockIdx.x] = s;
}

// One block per job, one wavefront per value (in turn).  out: [job][12].
__global__ __launch_bounds__(256) void k_stats_final(StatJobs jobs, int blocks, const double* __restrict__ part,
                                                     double* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t n = jobs.job[blockIdx.x].n;
    for (int e = threadIdx.x >> 6; e < 12; e += 4) {
        const double* p = part + ((int64_t)blockIdx.x * 12 + e) * blocks;
        const bool mx = e >= 5 && e < 10;
        double v = 0.0;
        for (int b = lane; b < blocks; b += 64) v = mx ? fmax(v, p[b]) : v + p[b];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            const double o = __shfl_xor(v, m, 64);
            v = mx ? fmax(v, o) : v + o;
        }
        if (lane == 0) out[blockIdx.x * 12 + e] = e < 5 ? (n > 0 ? sqrt(v / (double)n) : 0.0) : v;
    }
}

inline int grid_for(int64_t n, int threads = 256, int cap = 65536) {
    int64_t b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

inline int waves_grid(int64_t n_items, int waves_per_block) {
    return (int)((n_items + waves_per_block - 1) / waves_per_block);
}

}  // namespace

void launch_prep_sources(agis_ctx* ctx) {
    k_prep_sources<<<grid_for(ctx->n_src), 256, 0, ctx->stream>>>(ctx->n_src, ctx->s, ctx->src_eps2, ctx->prep);
}




void launch_apply_add(agis_ctx* ctx, int64_t n, double* x, const double* dx, int64_t m, double* y, const double* dy) {
    if (n + m > 0) k_apply_add<<<grid_for(n + m), 256, 0, ctx->stream>>>(n, x, dx, m, y, dy);
}

void launch_calib_solve(agis_ctx* ctx, double* rc) {
    const int64_t pairs = (ctx->n_cells + 1) / 2;
    if (pairs == 0) return;
    k_calib_solve<<<(unsigned)pairs, 256, 0, ctx->stream>>>(ctx->n_cells, ctx->cell_iv, ctx->iv_cell, ctx->iv_cal,
                                                           ctx->c, ctx->dc, rc);
}

void launch_frame_fit(agis_ctx* ctx) {
    k_frame_fit_partial<<<FR_BLOCKS, 256, 0, ctx->stream>>>(ctx->n_src, ctx->s, ctx->s_ref, ctx->svar, ctx->red);
    k_frame_fit_final<<<1, 1024, 0, ctx->stream>>>(ctx->k, ctx->red, ctx->eo);
}

void launch_frame_apply(agis_ctx* ctx) {
    const int src_blocks = grid_for(ctx->n_src);
    k_frame_apply<<<src_blocks + grid_for(ctx->N), 256, 0, ctx->stream>>>(
        ctx->k, src_blocks, ctx->n_src, ctx->N, ctx->eo, ctx->s, ctx->prep, ctx->knots, ctx->a);
}

void launch_residuals(agis_ctx* ctx, double* R) {
    if (ctx->K == 0) return;
    (ctx->k.defl > 0.0 ? k_residuals<true> : k_residuals<false>)<<<waves_grid(ctx->K, 4), 256, 0, ctx->stream>>>(
                                                                 ctx->k, ctx->K, ctx->iv_off, ctx->t_t, ctx->t_eta,
                                                                 ctx->t_cellfov, ctx->t_src, ctx->t_perm, ctx->prep,
                                                                 ctx->knots, ctx->ktab, ctx->a, ctx->c, R);
}

void launch_stats(agis_ctx* ctx, const StatJobs& jobs, int n_jobs, double* out) {
    int64_t n = 1;
    for (int j = 0; j < n_jobs; ++j) n = std::max(n, std::max(jobs.job[j].n, jobs.job[j].n_i));
    const int blocks = grid_for(n, 256, ST_BLOCKS);
    k_stats_partial<<<dim3(blocks, n_jobs), 256, 0, ctx->stream>>>(jobs, ctx->red);
    k_stats_final<<<n_jobs, 256, 0, ctx->stream>>>(jobs, blocks, ctx->red, out);
}

}  // namespace agis
