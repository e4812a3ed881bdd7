// Jacobi-scaled FP64 Cholesky solve of the kernel fit's normal equations, one
// workgroup per solve.
//
// The system (n <= 192 unknowns) is a chain of n pivots; what bounds it is
// the latency of that chain, not its 2.4 MFLOP.  So the matrix lives in
// registers as 16 x 16 blocks in the accumulator layout of
// v_mfma_f64_16x16x4f64, dealt column-major over the waves (the blocks still
// alive at any step are a contiguous run, so the waves stay balanced), and a
// step takes 16 columns:
//   - the owners put the step's block column in LDS;
//   - waves 0..3 factor it, a lane per row: every wave holds the 16 rows of
//     the diagonal block in lanes 0..15 (redundantly, so no exchange) and 48
//     panel rows in the others; pivot row values are broadcast by readlane,
//     so a column costs one reciprocal square root and one FMA per later
//     column, and the panel is solved by the same instructions;
//   - every wave applies the step to its trailing blocks, 4 MFMAs a block.
// The right-hand side rides along as row n of the matrix (its factor is the
// forward substitution's result); the back substitution runs over the same
// blocks, 16 unknowns a step.  Measured: 192 unknowns 458 -> 90 us, 96
// unknowns 162 -> 44 us, 16 solves of 32 unknowns 47 -> 17 us (before: the
// packed triangle in LDS, a column pair per barrier).
#include "fit_accum.h"

using argus_fit::qidx;

namespace {

struct SolveArgs {
    const double *sums;        // [n_solves][stride] moments, rhs, pixel count
    int stride;
    int nb, D, Dbg, n;
    double *coeffs;
    int64_t *n_fit;
    int32_t *status;
};

constexpr int SB = 16;         // block side
constexpr int ST = SB + 1;     // LDS row stride in doubles (bank spread)

__device__ __forceinline__ void unpack_row(int r, int nb, int D, int Dbg, int &k, int &p, int &q) {
    const int nP = (D + 1) * (D + 2) / 2;
    int m, Dm;
    if (r < nb * nP) { k = r / nP; m = r % nP; Dm = D; }
    else { k = nb; m = r - nb * nP; Dm = Dbg; }
    // monomial m of degree <= Dm: p outer, q inner
    int pp = 0;
    while (m > Dm - pp) { m -= Dm - pp + 1; ++pp; }
    p = pp;
    q = m;
}

__device__ __forceinline__ double gram_at(const double *G, int q, int k, int l) {
    // G[q][bp][16][16], blocks (0,0), (0,1), (1,1) of the symmetric 32x32 moment
    if (k > l) { const int t = k; k = l; l = t; }
    const double *g = G + (size_t)q * 768;
    if (l < 16) return g[k * 16 + l];
    if (k < 16) return g[256 + k * 16 + (l - 16)];
    return g[512 + (k - 16) * 16 + (l - 16)];
}

__device__ __forceinline__ double bcast(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// 1 / sqrt(p) for a positive normal p: the hardware estimate and two Newton
// steps (y <- y + y (1/2 - (p y) (y/2))), full FP64 accuracy to about an ulp.
__device__ __forceinline__ double rsqrt_newton(double p) {
    double y = __builtin_amdgcn_rsq(p);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(y, fma(-(p * y), 0.5 * y, 0.5), y);
    return y;
}

// LDS of the solve: two block columns (as assembled / as factored), the
// factored diagonal blocks, and the vectors.
__host__ __device__ constexpr int solve_blocks(int n) { return (n + SB) / SB; }   // rows 0..n
__host__ __device__ constexpr size_t solve_lds(int n) {
    return ((size_t)2 * solve_blocks(n) * SB * ST + (size_t)((n + SB - 1) / SB) * SB * ST +
            3 * (size_t)solve_blocks(n) * SB) * sizeof(double);
}

template <int NW, int NS>
__global__ __launch_bounds__(NW * 64) void fit_solve_kernel(SolveArgs a) {
    constexpr int NT = NW * 64;
    extern __shared__ double sl[];
    __shared__ short rk[256];             // basis, x-power and y-power of row r
    __shared__ unsigned char rp[256], rq[256];
    __shared__ double red[NW];
    __shared__ int bad;
    const int n = a.n, tid = threadIdx.x, sol = blockIdx.x;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, lg = lane >> 4;
    const int nblk = solve_blocks(n), kb = (n + SB - 1) / SB, nr = nblk * SB;
    double *P = sl;                       // block column before the factorisation
    double *Lp = P + nr * ST;             // and after it
    double *Dg = Lp + nr * ST;            // [kb] factored diagonal blocks
    double *yv = Dg + kb * SB * ST;       // L^-1 b, then the back substitution
    double *dd = yv + nr;                 // Jacobi scale
    double *rd = dd + nr;                 // 1 / L_jj
    const double *sums = a.sums + (size_t)sol * a.stride;
    const int D = a.D, NQ = (2 * D + 1) * (2 * D + 2) / 2;
    const double cnt = sums[(size_t)NQ * 768 + (D + 1) * (D + 2) / 2 * 32];
    double *co = a.coeffs + (size_t)sol * n;
    if (tid == 0) {
        bad = 0;
        if (a.n_fit) a.n_fit[sol] = (int64_t)cnt;
    }
    if (cnt < (double)n) {
        for (int i = tid; i < n; i += NT) co[i] = __builtin_nan("");
        if (tid == 0) a.status[sol] = ARGUS_ETOOFEW;
        return;
    }
    __syncthreads();
    double mx = 0.0;
    for (int r = tid; r < nr; r += NT) {
        double d = 0.0;
        if (r < n) {
            int k, p, q;
            unpack_row(r, a.nb, D, a.Dbg, k, p, q);
            rk[r] = (short)k;
            rp[r] = (unsigned char)p;
            rq[r] = (unsigned char)q;
            const double dg = gram_at(sums, qidx(2 * p, 2 * q, 2 * D), k, k);
            if (!(dg > 0.0)) bad = 1;
            d = dg > 0.0 ? 1.0 / sqrt(dg) : 0.0;
            mx = fmax(mx, dg * (d * d));
        }
        dd[r] = d;
        yv[r] = 0.0;
    }
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if (lane == 0) red[wv] = mx;
    __syncthreads();
    if (bad) {
        for (int i = tid; i < n; i += NT) co[i] = __builtin_nan("");
        if (tid == 0) a.status[sol] = ARGUS_ESINGULAR;
        return;
    }
    double maxdiag = 0.0;
    for (int i = 0; i < NW; ++i) maxdiag = fmax(maxdiag, red[i]);
    const double tol = (double)n * 0x1p-52 * maxdiag;
    // this wave's blocks (bi, bj), bi >= bj < kb, column-major, t = s NW + wave
    int bi[NS], bj[NS];
    doublex4 acc[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        int t = s * NW + wv, j = 0;
        while (j < kb && t >= nblk - j) { t -= nblk - j; ++j; }
        bj[s] = j < kb ? j : -1;
        bi[s] = j < kb ? j + t : -1;
        acc[s] = doublex4{0.0, 0.0, 0.0, 0.0};
        if (bj[s] >= 0) {
            const int c = SB * bj[s] + col;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = SB * bi[s] + 4 * r + lg;
                double v = 0.0;
                if (c < n && row < n)
                    v = gram_at(sums, qidx(rp[row] + rp[c], rq[row] + rq[c], 2 * D), rk[row],
                                rk[c]) * (dd[row] * dd[c]);
                else if (c < n && row == n)
                    v = sums[(size_t)NQ * 768 + qidx(rp[c], rq[c], D) * 32 + rk[c]] * dd[c];
                acc[s][r] = v;
            }
        }
    }
    for (int k = 0; k < kb; ++k) {
        // the block column, as updated by every earlier step
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (bj[s] == k)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    P[(SB * (bi[s] - k) + 4 * r + lg) * ST + col] = acc[s][r];
        __syncthreads();
        const int rows = SB * (nblk - k);              // diagonal block and panel
        const int jm = min(SB, n - SB * k);            // columns with a pivot
        if (wv == 0 || SB + 48 * wv < rows) {
            const int row = lane < SB ? lane : 48 * wv + lane;
            const bool have = row < rows;
            double x[SB];
#pragma unroll
            for (int m = 0; m < SB; ++m) x[m] = have ? P[row * ST + m] : 0.0;
            double rs_mine = 0.0;
            bool fail = false;
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                if (j < jm) {
                    const double piv = bcast(x[j], j);
                    fail |= !(piv > tol);
                    const double rs = rsqrt_newton(piv);
                    const double l = x[j] * rs;
                    x[j] = l;
                    if (lane == j) rs_mine = rs;
#pragma unroll
                    for (int m = j + 1; m < SB; ++m) x[m] = fma(-l, bcast(l, m), x[m]);
                }
            }
            if (lane >= SB && have) {
#pragma unroll
                for (int m = 0; m < SB; ++m) Lp[row * ST + m] = x[m];
            }
            if (lane < SB && wv == 0) {
#pragma unroll
                for (int m = 0; m < SB; ++m) Dg[(k * SB + lane) * ST + m] = x[m];
                rd[SB * k + lane] = rs_mine;
            }
            if (SB * k + row == n && (lane >= SB || wv == 0)) {
#pragma unroll
                for (int m = 0; m < SB; ++m)
                    if (m < jm) yv[SB * k + m] = x[m];
            }
            if (fail && lane == 0 && wv == 0) bad = 1;
        }
        __syncthreads();
        if (bad) break;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (bj[s] > k) {
                const double *pa = Lp + (SB * (bi[s] - k) + col) * ST + lg;
                const double *pb = Lp + (SB * (bj[s] - k) + col) * ST + lg;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(-pa[4 * q], pb[4 * q], acc[s], 0, 0, 0);
            } else if (bj[s] == k && bi[s] > k) {
                // kept for the back substitution
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[s][r] = Lp[(SB * (bi[s] - k) + 4 * r + lg) * ST + col];
            }
        }
    }
    if (bad) {
        for (int i = tid; i < n; i += NT) co[i] = __builtin_nan("");
        if (tid == 0) a.status[sol] = ARGUS_ESINGULAR;
        return;
    }
    // L^T x = y, 16 unknowns a step: every wave solves the diagonal block
    // itself, then takes its own blocks of that block row off the earlier y
    // (each block column has one owner, so the updates need no atomics)
    for (int k = kb - 1; k >= 0; --k) {
        const int jm = min(SB, n - SB * k);
        double y = col < jm ? yv[SB * k + col] : 0.0;
        const double rdc = col < jm ? rd[SB * k + col] : 0.0;
#pragma unroll
        for (int r = SB - 1; r > 0; --r) {
            if (r < jm) {
                const double xr = bcast(y * rdc, r);
                const double lr = Dg[(k * SB + r) * ST + col];
                if (col < r) y = fma(-lr, xr, y);
            }
        }
        const double x = y * rdc;
        if (wv == 0 && lane < jm) co[SB * k + lane] = dd[SB * k + lane] * x;
        double xv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) xv[r] = __shfl(x, 4 * r + lg);
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (bi[s] == k && bj[s] < k) {
                double p = 0.0;
#pragma unroll
                for (int r = 0; r < 4; ++r) p = fma(acc[s][r], xv[r], p);
                p += __shfl_xor(p, 16);
                p += __shfl_xor(p, 32);
                if (lane < SB) yv[SB * bj[s] + col] -= p;
            }
        __syncthreads();
    }
    if (tid == 0) a.status[sol] = ARGUS_OK;
}

template <int NW, int NS>
int solve_launch(argus_ctx *ctx, const SolveArgs &sa, int n_solves) {
    const size_t lds = solve_lds(sa.n);
    ARGUS_HIP_CHECK(ctx, hipFuncSetAttribute((const void *)fit_solve_kernel<NW, NS>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    argus_time_begin(ctx);
    hipLaunchKernelGGL((fit_solve_kernel<NW, NS>), dim3(n_solves), dim3(NW * 64), lds, ctx->stream, sa);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    argus_time_end(ctx, "fit_solve");
    return ARGUS_OK;
}

}  // namespace

int launch_solve(argus_ctx *ctx, const argus_kernel_spec *spec, const double *sums, int stride,
                 int n_solves, double *coeffs, int64_t *n_fit, int32_t *status) {
    SolveArgs sa;
    sa.sums = sums;
    sa.stride = stride;
    sa.nb = argus_nbasis(spec);
    sa.D = spec->spatial_degree;
    sa.Dbg = spec->bg_degree;
    sa.n = sa.nb * argus_npoly(sa.D) + argus_npoly(sa.Dbg);
    sa.coeffs = coeffs;
    sa.n_fit = n_fit;
    sa.status = status;
    // waves x blocks per wave that hold the sum_{j<kb} (nblk - j) blocks of
    // the system: 4 x 3 up to 48 unknowns (9 blocks; small groups let many
    // per-tile solves share a CU), 8 x 5 up to 112 (35), 16 x 6 up to 192 (90)
    if (sa.n <= 48) return solve_launch<4, 3>(ctx, sa, n_solves);
    if (sa.n <= 112) return solve_launch<8, 5>(ctx, sa, n_solves);
    return solve_launch<16, 6>(ctx, sa, n_solves);
}
