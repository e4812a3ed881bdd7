// Kernel fit: basis tables, fused basis convolution + normal-equation
// accumulation on MFMA and FP64 reduction of the partial sums (the solve is
// in k_solve.hip).
//
// Model (Alard & Lupton 1998; Alard 2000): the design row of pixel p is
//   X_p = [P_m(p) C_k(p)]_{k<nb, m<nP} ++ [P_m(p)]_{m<nPbg},
// with C_k = ref (x) B_k.  Every entry of A = sum w X X^T is a moment
//   G_{ab}[k][l] = sum_p w_p xt^a yt^b c_k(p) c_l(p),   a+b <= 2D,
// of the 32-vector c = (C_0..C_{nb-1}, 1, 0...) (the 1 carries the
// background), and b = sum w X S needs R_{ab}[k] = sum w xt^a yt^b c_k S,
// a+b <= D.  Along one image row yt is constant, so a workgroup accumulates
// only the xt-moments of the row on MFMA (FP32, 64 pixels) and then adds
// yt^b times them into FP64 running sums: 2D+1 Gram blocks per pixel instead
// of (2D+1)(2D+2)/2.
#include "fit_accum.h"

using argus_fit::FitArgs;
using argus_fit::FitShape;
using argus_fit::SW;

namespace {

// ---------------------------------------------------------------------------
// Basis tables, computed on the device in FP64 from the spec.
// B_k(u,v) = exp(-(u^2+v^2)/2s^2) u^i v^j; B_0 -> unit sum; k>=1 with i, j
// even -> B_k - (sum B_k) B_0; k >= 1 -> unit L2 norm.  In separable form
// B'_k = alpha_k f_{g,i}(u) f_{g,j}(v) + beta_k B_0raw.
//
// One workgroup of 16 waves, a wave per basis function for the sums over the
// grid, from the 1-D factors in LDS; part of the first fit of a spec (one
// thread per basis function with two exponentials and two powers a sample took
// 325 us at h = 7, 740 us at h = 10; now 13 and 17 us).
constexpr int BT_THREADS = 1024;
constexpr int BT_PMAX = 7;                 // powers 0..6

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__global__ __launch_bounds__(BT_THREADS) void basis_tables_kernel(argus_kernel_spec s, BasisTables *T) {
    __shared__ int kg[32], ki[32], kj[32], kp[32], s_nb;
    __shared__ double f[4][BT_PMAX][32];   // exp(-u^2/2s^2) u^i, index u + h
    __shared__ double alpha[32], beta[32];
    const int h = s.half_width, K = 2 * h + 1;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) {
        int k = 0, p = 0;
        for (int g = 0; g < s.n_gauss; ++g)
            for (int i = 0; i <= s.degree[g]; ++i, ++p) {
                for (int j = 0; j <= s.degree[g] - i; ++j, ++k) {
                    kg[k] = g; ki[k] = i; kj[k] = j; kp[k] = p;
                }
                T->ipow[p] = i;
            }
        s_nb = k;
        T->nb = k;
        T->nplanes = p;
        T->h = h;
    }
    if (tid < 4 * 32) {
        const int g = tid >> 5, u = (tid & 31) - h;
        if (g < s.n_gauss && u <= h) {
            const double is2 = 1.0 / (2.0 * s.sigma[g] * s.sigma[g]);
            const double e = exp(-(double)(u * u) * is2);
            double pw = 1.0;                   // u^i, exact
            for (int i = 0; i < BT_PMAX; ++i, pw *= (double)u) f[g][i][u + h] = e * pw;
        }
    }
    __syncthreads();
    const int nb = s_nb;
    // every wave forms B_0's sum itself
    double S0 = 0.0;
    for (int t = lane; t < K * K; t += 64) S0 += f[0][0][t % K] * f[0][0][t / K];
    S0 = wave_sum(S0);
    for (int k = wv; k < nb; k += BT_THREADS / 64) {
        const double *fu = f[kg[k]][ki[k]], *fv = f[kg[k]][kj[k]];
        double raw_sum = 0.0;
        for (int t = lane; t < K * K; t += 64) raw_sum += fu[t % K] * fv[t / K];
        raw_sum = wave_sum(raw_sum);
        const bool even = (ki[k] % 2 == 0) && (kj[k] % 2 == 0);
        const double c0 = (k >= 1 && even) ? raw_sum / S0 : 0.0;   // subtract c0 * B_0raw
        double nrm = 0.0;
        for (int t = lane; t < K * K; t += 64) {
            const double b = fu[t % K] * fv[t / K] - c0 * (f[0][0][t % K] * f[0][0][t / K]);
            nrm += b * b;
        }
        nrm = wave_sum(nrm);
        const double a = k == 0 ? 1.0 / S0 : 1.0 / sqrt(nrm), be = k == 0 ? 0.0 : -c0 * a;
        if (lane == 0) {
            alpha[k] = a;
            beta[k] = be;
            T->gam[k] = (float)(be * S0);     // C'_k = alpha_k conv_k + (beta_k / alpha_0) C'_0
            T->kpl[k] = kp[k];
        }
        if (lane < K) {
            T->colf[k][lane] = (float)(a * fv[lane]);
            if (kj[k] == 0) T->rowf[kp[k]][lane] = (float)fu[lane];      // one j = 0 per plane
        }
    }
    __syncthreads();
    // 2-D normalised basis for the kernel expansion
    for (int idx = tid; idx < nb * K * K; idx += BT_THREADS) {
        const int k = idx / (K * K), t = idx % (K * K);
        const int v = t / K, u = t % K;
        T->b2d[k][t] = alpha[k] * (f[kg[k]][ki[k]][u] * f[kg[k]][kj[k]][v]) +
                       beta[k] * (f[0][0][u] * f[0][0][v]);
    }
}

// Sum consecutive groups of partial vectors in a fixed order (deterministic);
// 8 loads in flight per thread (the adds stay in order).
__global__ void sum_parts_kernel(const double *in, int stride, int n_in, int group, double *out) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    int set = blockIdx.y;
    if (e >= stride) return;
    const int j0 = set * group, j1 = min(j0 + group, n_in);
    const double *p = in + e;
    double s = 0.0;
    int j = j0;
    for (; j + 8 <= j1; j += 8) {
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = p[(size_t)(j + i) * stride];
#pragma unroll
        for (int i = 0; i < 8; ++i) s += v[i];
    }
    for (; j < j1; ++j) s += p[(size_t)j * stride];
    out[(size_t)set * stride + e] = s;
}

// K_m = sum_k a_{k nP + m} B_k (FP64), bg_m = a_{nb nP + m}: a workgroup per
// 64 samples of a stamp, the basis values of 31 functions in flight (the sum
// over k stays in order; with a workgroup per stamp and one load at a time
// the launch took 27 us at 21 x 21, now 5 us)
__global__ __launch_bounds__(64) void expand_kernel(const BasisTables *T, const double *coeffs,
                                                    int n, int nP, int nPb, int K, int nb,
                                                    float *stamps, float *bg) {
    const int s = blockIdx.x / nP, m = blockIdx.x % nP;
    const double *a = coeffs + (size_t)s * n;
    const int t = blockIdx.y * 64 + threadIdx.x;
    if (t < K * K) {
        double b[ARGUS_MAX_NB], c[ARGUS_MAX_NB], acc = 0.0;
#pragma unroll
        for (int k = 0; k < ARGUS_MAX_NB; ++k) {
            const int kc = min(k, nb - 1);
            b[k] = T->b2d[kc][t];
            c[k] = a[kc * nP + m];
        }
#pragma unroll
        for (int k = 0; k < ARGUS_MAX_NB; ++k)
            if (k < nb) acc += c[k] * b[k];
        stamps[((size_t)s * nP + m) * K * K + t] = (float)acc;
    }
    if (t == 0 && m < nPb) bg[(size_t)s * nPb + m] = (float)a[nb * nP + m];
}

template <int D>
int fit_launch_d(argus_ctx *ctx, argus_dims d, const argus_kernel_spec *spec, FitArgs &fa,
                 int n_regions, int parts_per_region, double **sums_out) {
    using S = FitShape<D>;
    fa.stride = S::NQ * 768 + S::NR * 32 + 1;
    fa.stride = (fa.stride + 1) & ~1;
    const int n_parts = n_regions * parts_per_region;
    const int group = 64;
    const int n_g1 = spec->mode == ARGUS_FIT_GLOBAL ? (n_parts + group - 1) / group : 0;
    size_t need = ((size_t)n_parts + n_g1 + n_regions) * fa.stride * sizeof(double);
    int rc = argus_ws_reserve(ctx, need + 256);
    if (rc) return rc;
    double *base = (double *)ctx->ws;
    fa.partials = base;
    double *stage1 = base + (size_t)n_parts * fa.stride;
    double *sums = stage1 + (size_t)n_g1 * fa.stride;
    dim3 grid(fa.RX * fa.spt, fa.RY * fa.rchunks);
    argus_time_begin(ctx);
    switch (spec->precision) {
        case ARGUS_FP64: rc = fit_accum_launch_fp64(ctx, fa, D, grid); break;
        case ARGUS_BF16X3: rc = fit_accum_launch_bf16x3(ctx, fa, D, grid); break;
        default:
            if (D >= 1 && d.width >= FIT_WIDE_MIN)
                rc = fit_accum_launch_wide(ctx, fa, D, grid);
            else
                rc = fit_accum_launch_fp32(ctx, fa, D, grid);
            break;
    }
    if (rc) return rc;
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    argus_time_end(ctx, "fit_accum");
    argus_time_begin(ctx);
    dim3 rb((fa.stride + 255) / 256);
    if (spec->mode == ARGUS_FIT_GLOBAL) {
        hipLaunchKernelGGL(sum_parts_kernel, dim3(rb.x, n_g1), dim3(256), 0, ctx->stream,
                           (const double *)fa.partials, fa.stride, n_parts, group, stage1);
        hipLaunchKernelGGL(sum_parts_kernel, dim3(rb.x, 1), dim3(256), 0, ctx->stream,
                           (const double *)stage1, fa.stride, n_g1, n_g1, sums);
    } else {
        hipLaunchKernelGGL(sum_parts_kernel, dim3(rb.x, n_regions), dim3(256), 0, ctx->stream,
                           (const double *)fa.partials, fa.stride, n_parts, parts_per_region, sums);
    }
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    argus_time_end(ctx, "fit_reduce");
    *sums_out = sums;
    return ARGUS_OK;
}

}  // namespace

int launch_basis_tables_to(argus_ctx *ctx, const argus_kernel_spec *spec, BasisTables *dst) {
    hipLaunchKernelGGL(basis_tables_kernel, dim3(1), dim3(BT_THREADS), 0, ctx->stream, *spec, dst);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}

int launch_basis_tables(argus_ctx *ctx, const argus_kernel_spec *spec) {
    const argus_kernel_spec &o = ctx->tables_spec;
    bool same = ctx->tables_valid && o.n_gauss == spec->n_gauss && o.half_width == spec->half_width;
    for (int g = 0; same && g < spec->n_gauss; ++g)
        same = o.sigma[g] == spec->sigma[g] && o.degree[g] == spec->degree[g];
    if (same) return ARGUS_OK;
    hipLaunchKernelGGL(basis_tables_kernel, dim3(1), dim3(BT_THREADS), 0, ctx->stream, *spec, ctx->tables);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    ctx->tables_spec = *spec;
    ctx->tables_valid = true;
    return ARGUS_OK;
}

int launch_fit(argus_ctx *ctx, argus_dims d, const argus_kernel_spec *spec, const float *ref,
               const float *ref_var, const uint8_t *ref_mask, const float *sci,
               const float *sci_var, const uint8_t *sci_mask, double *coeffs, int64_t *n_fit,
               int32_t *status) {
    FitArgs fa;
    fa.ref = ref; fa.rvar = ref_var; fa.sci = sci; fa.svar = sci_var;
    fa.rmask = ref_mask; fa.smask = sci_mask;
    fa.tab = ctx->tables;
    fa.pitch = d.pitch; fa.W = d.width; fa.H = d.height;
    fa.h = spec->half_width;
    fa.nb = argus_nbasis(spec);
    fa.nplanes = argus_nplanes(spec);
    // planes to the convolution waves, longest first onto the least loaded
    // wave: 8 waves (wave 0 at most 1 plane, the others at most 2) or 4 waves
    // (at most 4 each); at most 13 planes fit the basis limit.  Cost of a plane in VALU operations per pixel
    // row with paired symmetric taps: its row filter (h + 1), the paired
    // window of its column (2h, or h when it feeds one even filter) and h + 2
    // per column filter it feeds; wave 0 also stages the fit-set weights.
    {
        const int h = spec->half_width;
        int cost[ARGUS_MAX_PLANES];
        int p = 0;
        for (int g = 0; g < spec->n_gauss; ++g)
            for (int i = 0; i <= spec->degree[g]; ++i, ++p) {
                const int nk = spec->degree[g] - i + 1;
                cost[p] = (h + 1) + (nk > 1 ? 2 * h : h) + nk * (h + 2);
            }
        // 4 convolution waves (FP64 form), up to 4 planes each
        int load[4] = {3 * h, 0, 0, 0}, nin[4] = {};
        bool used[ARGUS_MAX_PLANES] = {};
        for (int w = 0; w < 4; ++w)
            for (int j = 0; j < 4; ++j) fa.plist[w][j] = -1;
        for (int n = 0; n < fa.nplanes; ++n) {
            int best = -1;
            for (int q = 0; q < fa.nplanes; ++q)
                if (!used[q] && (best < 0 || cost[q] > cost[best])) best = q;
            int w = -1;
            for (int c = 0; c < 4; ++c)
                if (nin[c] < 4 && (w < 0 || load[c] < load[w])) w = c;
            used[best] = true;
            fa.plist[w][nin[w]++] = (int8_t)best;
            load[w] += cost[best];
        }
        // 8 convolution waves (FP32 and BF16x3 forms)
        int load8[8] = {}, nin8[8] = {};
        load8[0] = 3 * h;
        bool used8[ARGUS_MAX_PLANES] = {};
        for (int w = 0; w < 8; ++w)
            for (int j = 0; j < 2; ++j) fa.plist8[w][j] = -1;
        for (int n = 0; n < fa.nplanes; ++n) {
            int best = -1;
            for (int q = 0; q < fa.nplanes; ++q)
                if (!used8[q] && (best < 0 || cost[q] > cost[best])) best = q;
            int w = -1;
            for (int c = 0; c < 8; ++c)
                if (nin8[c] < (c == 0 ? 1 : 2) && (w < 0 || load8[c] < load8[w])) w = c;
            used8[best] = true;
            fa.plist8[w][nin8[w]++] = (int8_t)best;
            load8[w] += cost[best];
        }
    }
    const bool global = spec->mode == ARGUS_FIT_GLOBAL;
    fa.RX = global ? 1 : spec->tiles_x;
    fa.RY = global ? 1 : spec->tiles_y;
    int maxw = (d.width + fa.RX - 1) / fa.RX;
    int maxh = (d.height + fa.RY - 1) / fa.RY;
    fa.spt = (maxw + SW - 1) / SW;
    // Row chunks: one workgroup runs per CU at a time, so the accumulation
    // takes ceil(workgroups / CUs) rounds of (rows per chunk + 2h halo rows)
    // steps of about 1 us + 0.4 us per degree (FP64 moments: twice that), and
    // every chunk's partial moments are written and read again (at about 3 TB/s
    // together).  Take the chunk count, chunks of 4 rows and up, with the
    // smallest sum: large frames get a last round that leaves few CUs idle,
    // small ones many short chunks (256 x 224, degree 1: 94 -> 27 us against
    // chunks no shorter than 8h rows).
    {
        const int base = fa.RX * fa.RY * fa.spt;
        const int maxc = maxh / 4 > 1 ? maxh / 4 : 1;
        const int ncu = ctx->n_cu > 0 ? ctx->n_cu : 256;
        const int D = spec->spatial_degree;
        const double step_us = (1.0 + 0.4 * D) * (spec->precision == ARGUS_FP64 ? 2.0 : 1.0);
        const double part_us = 2.0 * 8.0 * 768.0 * argus_npoly(2 * D) / 3e6;
        double best = -1.0;
        fa.rchunks = 1;
        for (int c = 1; c <= maxc; ++c) {
            const int64_t wg = (int64_t)base * c, rounds = (wg + ncu - 1) / ncu;
            // (halo rows and partials only grow with c)
            const double least = (double)(rounds * 2 * fa.h) * step_us + (double)wg * part_us;
            if (best >= 0.0 && least >= best) break;
            const double t = least + (double)(rounds * ((maxh + c - 1) / c)) * step_us;
            if (best < 0.0 || t < best) {
                best = t;
                fa.rchunks = c;
            }
        }
    }
    fa.sx = d.width > 1 ? 2.0 / (d.width - 1) : 0.0;
    fa.sy = d.height > 1 ? 2.0 / (d.height - 1) : 0.0;
    const int n_regions = fa.RX * fa.RY;
    const int parts_per_region = fa.rchunks * fa.spt;
    double *sums = nullptr;
    int rc;
    switch (spec->spatial_degree) {
        case 0: rc = fit_launch_d<0>(ctx, d, spec, fa, n_regions, parts_per_region, &sums); break;
        case 1: rc = fit_launch_d<1>(ctx, d, spec, fa, n_regions, parts_per_region, &sums); break;
        default: rc = fit_launch_d<2>(ctx, d, spec, fa, n_regions, parts_per_region, &sums); break;
    }
    if (rc) return rc;
    return launch_solve(ctx, spec, sums, fa.stride, n_regions, coeffs, n_fit, status);
}

namespace {
__global__ void chi2_failed_kernel(double *chi2, const int32_t *status, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && status[i] != ARGUS_OK) chi2[i] = __builtin_nan("");
}
}  // namespace

int launch_chi2_failed(argus_ctx *ctx, double *chi2, const int32_t *status, int n) {
    hipLaunchKernelGGL(chi2_failed_kernel, dim3((n + 255) / 256), dim3(256), 0, ctx->stream, chi2,
                       status, n);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}

int launch_expand(argus_ctx *ctx, const argus_kernel_spec *spec, const double *coeffs,
                  float *stamps, float *bg) {
    int n, ns;
    argus_kernel_dims(spec, &n, &ns);
    int nP = argus_npoly(spec->spatial_degree), nPb = argus_npoly(spec->bg_degree);
    const int K = 2 * spec->half_width + 1;
    hipLaunchKernelGGL(expand_kernel, dim3(ns * nP, (K * K + 63) / 64), dim3(64), 0, ctx->stream,
                       (const BasisTables *)ctx->tables, coeffs, n, nP, nPb, K, argus_nbasis(spec),
                       stamps, bg);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}
