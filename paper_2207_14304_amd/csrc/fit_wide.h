// Moment accumulation of the FP32 fit on wide frames (D >= 1), with the
// matrix products on BF16 instructions.
//
// On gfx950 FP32 MFMA and VALU cycles add up (they do not overlap), and the
// FP32 form of the fit (fit_accum8.h) spends half its time on FP32 MFMAs: 2D+1
// x-powers of every 64-pixel row segment.  Two things shrink that here.
//
// 1. Powers about the strip's centre.  With xt = x0 + d the moments are taken
//    in powers of d, |d| <= 31.5 * 2/(W-1), which the end of the kernel
//    combines into powers of xt (binomially, in FP64).  A solve may cover a
//    single strip (a narrow tile, or a frame whose other columns are masked):
//    about that strip's centre every power of d is a diagonal of the system, so
//    each is held to FP32 accuracy relative to itself, however small |d| is.
// 2. Split operands.  With s = sqrt(w) c', u = d s and v = d^2 s the moments of
//    powers 0..4 are s s^T, s u^T, u u^T, u v^T and v v^T.  Each vector is split
//    into h + m + l in bf16 (residual 2^-27) and a product takes h h, h m, m h,
//    h l, l h and m m (dropped terms 2^-26: below the 2^-24 of an FP32 product).
//    Products are exact in FP32 and summed in FP32 over 64 pixels, as before.
//
// The right-hand side is summed from the same s, about the strip's centre too:
// FP32 products over 4 pixels, then FP64 per lane across rows.
//
// Waves and pipeline: 8 convolution waves (fit_conv8) write row y's c at step
// n; the 8 MFMA waves split it (4 basis rows each, a lane per row and 4
// pixels) into bf16 tables at step n + 1 and multiply them at step n + 2, one
// barrier per step.  Of the two MFMA waves of a SIMD one multiplies first and
// the other splits first, so that matrix and vector work meet.
//
// What bounds it: VALU issue (filters, splits, FP64 sums) and, beside it, the
// products.  Full frame, 21 x 21: degree 2 7.42 -> 6.26 ms against the FP32 form,
// degree 1 6.16 -> 4.57; the difference image as far from the 64-bit one as
// before (9.1e-6 relative).  Tiles of 64 to 409 columns at the centre of a 6144
// x 140 frame: difference 1.2e-5 to 1.1e-4 sigma RMS from the 64-bit solution's,
// 7.3e-5 to 2.7e-2 with the FP32 form (its powers are those of the frame's
// coordinate).  Three products for powers 1 to 4 (5.35 ms) leave such tiles'
// systems indefinite.
#pragma once
#include "fit_accum8.h"

namespace argus_fit {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

template <int D, int HH>
struct FitWideLds {
    using Base = FitLds8<D, HH, false>;
    static constexpr int CKB = SW + 8;                   // row stride of a table (16-byte rows)
    // tables of one buffer: h, m, l of s, of d s and, for D = 2, of d^2 s
    static constexpr int NTAB = 3 * (D + 1);
    static constexpr int TAB = 32 * CKB;                 // bf16 values of a table
    static constexpr int NF = FitShape<D>::NQ;           // (power of d, power of yt) moments
    static constexpr size_t base = (Base::bytes(8) + 15) & ~(size_t)15;
    static constexpr size_t bytes() {
        constexpr size_t t = base + (size_t)2 * NTAB * TAB * 2;
        constexpr size_t f = (size_t)NF * 768 * 8;       // end-of-kernel reuse
        return t > f ? t : f;
    }
    __device__ static __bf16 *tab(float *lds, int b, int t) {
        return (__bf16 *)(lds + base / 4) + (b * NTAB + t) * TAB;
    }
};

// Tasks (power of d, block pair) of MFMA wave MW: at most two, of 12 products
// each, or 8 for a diagonal block of an even power (waves MW and MW + 4 share a
// SIMD: 40, 40, 40 and 36 of D = 2's 156 products, 24, 20, 24 and 24 of D = 1's
// 92).  A high power, with few sums, goes with a low one.
struct WideTask { int a, bp; };
template <int D>
__host__ __device__ constexpr WideTask wide_task(int mw, int i) {
    constexpr WideTask t2[8][2] = {{{0, 0}, {4, 0}}, {{0, 2}, {4, 2}}, {{0, 1}, {4, 1}},
                                   {{1, 0}, {3, 0}}, {{1, 1}, {3, 1}}, {{1, 2}, {3, 2}},
                                   {{2, 0}, {2, 2}}, {{2, 1}, {-1, 0}}};
    constexpr WideTask t1[8][2] = {{{0, 0}, {-1, 0}}, {{0, 2}, {-1, 0}}, {{0, 1}, {-1, 0}},
                                   {{1, 0}, {-1, 0}}, {{2, 0}, {2, 2}}, {{1, 1}, {-1, 0}},
                                   {{1, 2}, {-1, 0}}, {{2, 1}, {-1, 0}}};
    return D == 1 ? t1[mw][i] : t2[mw][i];
}

// xt at the centre of the strip whose first column is sx0
__device__ __forceinline__ double wide_centre(const FitArgs &a, int sx0) {
    return ((double)sx0 + 31.5) * a.sx - 1.0;
}

__device__ __forceinline__ bf16x4 to_bf16(const float (&v)[4]) {
    return bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
}

// v <- v - b
__device__ __forceinline__ void less(float (&v)[4], bf16x4 b) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] -= (float)b[i];
}

template <int D, int HH, int MW>
__device__ void fit_wide_mfma(const FitArgs &a, float *lds, int sx0, int ry0, int ry1, bool active,
                              double *part) {
    using S = FitShape<D>;
    using L = FitWideLds<D, HH>;
    constexpr int CKM = FitLds8<D, HH, false>::CKM, CKB = L::CKB;
    constexpr int NB = 2 * D + 1;
    constexpr WideTask T0 = wide_task<D>(MW, 0), T1 = wide_task<D>(MW, 1);
    constexpr bool SPLIT_FIRST = MW >= 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int col = lane & 15, pk = lane >> 4;
    FitLds8<D, HH, false> l(lds);
    // split side: basis row and 4 pixels of this lane
    const int k = 4 * MW + pk, p4 = 4 * col;
    const float gam = k < a.nb ? a.tab->gam[k] : 0.f;
    float dl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) dl[i] = (float)(((double)(p4 + i) - 31.5) * a.sx);
    double RF[S::NR];
#pragma unroll
    for (int i = 0; i < S::NR; ++i) RF[i] = 0.0;
    double F0[NB][4], F1[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) F0[b][r] = F1[b][r] = 0.0;

    auto ypowers = [&](int yv, double *ypw) {
        const double yt = (double)yv * a.sy - (a.sy != 0.0 ? 1.0 : 0.0);
        double yp = 1.0;
#pragma unroll
        for (int b = 0; b <= 2 * D; ++b) { ypw[b] = yp; yp *= yt; }
    };
    auto frag = [&](int buf, int t, int half, int s) {
        return *(const bf16x8 *)(L::tab(lds, buf, t) + (16 * half + col) * CKB + 32 * s + 8 * pk);
    };
    // one task: the moments over a row's 64 pixels, h h in acc, the smaller
    // products in cross (in one sum, the roundings of equal pixels add up), and
    // their yt powers into the FP64 sums
    auto task = [&](auto ta, auto tb, double (&F)[NB][4], int buf, const double *ypw) {
        constexpr int A = decltype(ta)::value, BP = decltype(tb)::value;
        constexpr int ra = BP == 2 ? 1 : 0, rb = BP == 0 ? 0 : 1;
        constexpr int va = 3 * (A / 2), vb = 3 * (A - A / 2);     // first tables of the two vectors
        constexpr bool SAME = ra == rb && va == vb;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f}, cross = acc;
#define ARGUS_MM(X, Y, C) C = __builtin_amdgcn_mfma_f32_16x16x32_bf16(X, Y, C, 0, 0, 0);
        if constexpr (SAME) {
            // m h and l h are the transposes of h m and h l (the block is
            // symmetrised at the end): cross is half their sum with m m
            bf16x8 h[SW / 32], m[SW / 32], l[SW / 32];
#pragma unroll
            for (int s = 0; s < SW / 32; ++s) {
                h[s] = frag(buf, va, ra, s);
                m[s] = frag(buf, va + 1, ra, s);
                l[s] = frag(buf, va + 2, ra, s);
                ARGUS_MM(m[s], m[s], cross)
                ARGUS_MM(h[s], h[s], acc)
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) cross[r] *= 0.5f;
#pragma unroll
            for (int s = 0; s < SW / 32; ++s) {
                ARGUS_MM(h[s], l[s], cross)
                ARGUS_MM(h[s], m[s], cross)
            }
        } else {
#pragma unroll
            for (int s = 0; s < SW / 32; ++s) {
                const bf16x8 h0 = frag(buf, va, ra, s), m0 = frag(buf, va + 1, ra, s), l0 = frag(buf, va + 2, ra, s);
                const bf16x8 h1 = frag(buf, vb, rb, s), m1 = frag(buf, vb + 1, rb, s), l1 = frag(buf, vb + 2, rb, s);
                ARGUS_MM(h0, h1, acc)
                ARGUS_MM(h0, l1, cross)
                ARGUS_MM(l0, h1, cross)
                ARGUS_MM(m0, m1, cross)
                ARGUS_MM(h0, m1, cross)
                ARGUS_MM(m0, h1, cross)
            }
        }
#undef ARGUS_MM
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double v = (double)acc[r] + (SAME ? 2.0 : 1.0) * (double)cross[r];
#pragma unroll
            for (int b = 0; b <= 2 * D - A; ++b) F[b][r] += ypw[b] * v;
        }
    };
    auto multiply = [&](int y, int buf) {
        double ypw[NB];
        ypowers(y, ypw);
        task(std::integral_constant<int, T0.a>{}, std::integral_constant<int, T0.bp>{}, F0, buf, ypw);
        if constexpr (T1.a >= 0)
            task(std::integral_constant<int, T1.a>{}, std::integral_constant<int, T1.bp>{}, F1, buf, ypw);
    };
    // s = sqrt(w) c' of this lane's row and pixels, its tables, and the
    // right-hand side's products
    auto split = [&](int y, int cb, int tb) {
        const float *cv = l.cvec(cb);
        const float4 c4 = *(const float4 *)(cv + k * CKM + p4), z4 = *(const float4 *)(cv + p4);
        const float4 q4 = *(const float4 *)(l.wx(cb) + p4);
        float s[4] = {(c4.x + gam * z4.x) * q4.x, (c4.y + gam * z4.y) * q4.y,
                      (c4.z + gam * z4.z) * q4.z, (c4.w + gam * z4.w) * q4.w};
        double ypw[NB];
        ypowers(y, ypw);
#pragma unroll
        for (int e = 0; e < S::NRA; ++e) {
            const float4 t = *(const float4 *)(l.wsx(cb) + e * SW + p4);
            const double r = (double)(t.x * s[0] + t.y * s[1] + t.z * s[2] + t.w * s[3]);
#pragma unroll
            for (int b = 0; b <= D; ++b)
                if (e + b <= D) RF[qidx(e, b, D)] += ypw[b] * r;
        }
        auto put = [&](int t, bf16x4 v) { *(bf16x4 *)(L::tab(lds, tb, t) + k * CKB + p4) = v; };
#pragma unroll
        for (int j = 0; j <= D; ++j) {                   // s, d s, d^2 s
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = s[i];
            const bf16x4 h = to_bf16(v);
            put(3 * j, h);
            less(v, h);
            const bf16x4 m = to_bf16(v);
            put(3 * j + 1, m);
            less(v, m);
            put(3 * j + 2, to_bf16(v));
            if (j < D)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] *= dl[i];
        }
    };

    const int ystart = ry0 - HH, yend = active ? ry1 + HH : ystart;
    const int ys0 = ystart & ~1;
    const int ylast = ys0 + fit8_strip_steps<true>(yend - ys0) - 1;
    __syncthreads();
    for (int yy = ys0; yy <= ylast; ++yy) {
        // the row convolved in step yy - 1 is split into buffer yy & 1, the one
        // split in step yy - 1 multiplied
        const int buf = yy & 1;
        const bool sp = yy - 1 >= ry0 + HH && yy - 1 < yend;
        const bool mu = yy - 2 >= ry0 + HH && yy - 2 < yend;
        if (SPLIT_FIRST && sp) split(yy - 1 - HH, buf ^ 1, buf);
        if (mu) multiply(yy - 2 - HH, buf ^ 1);
        if (!SPLIT_FIRST && sp) split(yy - 1 - HH, buf ^ 1, buf);
        __syncthreads();
    }
    // right-hand side: the 16 lanes of a basis row; powers of xt as below
#pragma unroll
    for (int i = 0; i < S::NR; ++i)
        for (int off = 8; off > 0; off >>= 1) RF[i] += __shfl_xor(RF[i], off);
    const double x0 = wide_centre(a, sx0);
#pragma unroll
    for (int p = 0; p <= D; ++p)
#pragma unroll
        for (int b = 0; b <= D - p; ++b) {
            double v = RF[qidx(p, b, D)];
            if (p >= 1) v += p * x0 * RF[qidx(p - 1, b, D)];
            if (p == 2) v += x0 * x0 * RF[qidx(0, b, D)];
            if (col == 0) part[(size_t)S::NQ * 768 + qidx(p, b, D) * 32 + k] = v;
        }
    // the moments in powers of d, for the whole workgroup to combine
    double *fb = (double *)lds;
    auto out = [&](WideTask t, const double (&F)[NB][4]) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (b <= 2 * D - t.a)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    fb[(size_t)qidx(t.a, b, 2 * D) * 768 + t.bp * 256 + (4 * pk + r) * 16 + col] = F[b][r];
    };
    out(T0, F0);
    if constexpr (T1.a >= 0) out(T1, F1);
}

template <int D, int HH, int MW>
__device__ __forceinline__ void fit_wide_dispatch(int w, const FitArgs &a, float *lds, int sx0, int ry0,
                                                  int ry1, bool active, double *part) {
    if constexpr (MW < 8) {
        if (w == 8 + MW) fit_wide_mfma<D, HH, MW>(a, lds, sx0, ry0, ry1, active, part);
        else fit_wide_dispatch<D, HH, MW + 1>(w, a, lds, sx0, ry0, ry1, active, part);
    }
}

// One workgroup: a 64-column strip, rows [ry0, ry1) (fit_accum8_kernel's grid).
template <int D, int HH>
__global__ __launch_bounds__(1024) void fit_wide_kernel(FitArgs a) {
    extern __shared__ __align__(16) float lds[];
    using S = FitShape<D>;
    using L = FitWideLds<D, HH>;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = blockIdx.x % a.spt, rx = blockIdx.x / a.spt;
    const int rc = blockIdx.y % a.rchunks, ry = blockIdx.y / a.rchunks;
    const int rx0 = (int)((int64_t)rx * a.W / a.RX), rx1 = (int)((int64_t)(rx + 1) * a.W / a.RX);
    const int ry0g = (int)((int64_t)ry * a.H / a.RY), ry1g = (int)((int64_t)(ry + 1) * a.H / a.RY);
    const int ix0 = max(rx0, HH), ix1 = min(rx1, a.W - HH);
    const int iy0 = max(ry0g, HH), iy1 = min(ry1g, a.H - HH);
    const int sx0 = ix0 + s * SW, sx1 = min(sx0 + SW, ix1);
    const int rows = max(iy1 - iy0, 0);
    const int rh = (rows + a.rchunks - 1) / a.rchunks;
    const int ry0 = iy0 + rc * rh, ry1 = min(ry0 + rh, iy1);
    const bool active = sx0 < sx1 && ry0 < ry1;    // otherwise the partial is all zeros
    const int pid = ((ry * a.RX + rx) * a.rchunks + rc) * a.spt + s;
    double *part = a.partials + (size_t)pid * a.stride;
    // constant tail of c: 1 at index nb (background), zeros after, both buffers
    using LB = FitLds8<D, HH, false>;
    LB lb(lds);
    for (int i = tid; i < 2 * 32 * LB::CKM; i += 1024) {
        const int k = (i / LB::CKM) % 32;
        if (k >= a.nb) lb.cvec0[i] = (k == a.nb) ? 1.f : 0.f;
    }
    int count = 0;
    if (w == 0)
        count = fit_conv8<D, HH, ARGUS_FP32, 8, 1, true, true>(a, lds, sx0, sx1, ry0, ry1, active, 0);
    else if (w < 8)
        fit_conv8<D, HH, ARGUS_FP32, 8, 2, false, true>(a, lds, sx0, sx1, ry0, ry1, active, w);
    else
        fit_wide_dispatch<D, HH, 0>(w, a, lds, sx0, ry0, ry1, active, part);
    if (w == 0) {
        const int lane = tid & 63;
        double c = (double)count;
        for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
        if (lane == 0) part[(size_t)S::NQ * 768 + S::NR * 32] = c;
    }
    __syncthreads();
    // powers of xt = x0 + d: xt^p = sum_j C(p, j) x0^(p - j) d^j; diagonal
    // blocks symmetrised
    const double *fb = (const double *)lds;
    const double x0 = wide_centre(a, sx0);
    constexpr double bin[5][5] = {{1, 0, 0, 0, 0}, {1, 1, 0, 0, 0}, {1, 2, 1, 0, 0}, {1, 3, 3, 1, 0}, {1, 4, 6, 4, 1}};
    for (int i = tid; i < 768; i += 1024) {
        const int bp = i >> 8, r = (i >> 4) & 15, c = i & 15;
        const int it = bp == 1 ? i : (bp << 8) + c * 16 + r;
        double F[2 * D + 1][2 * D + 1];
#pragma unroll
        for (int j = 0; j <= 2 * D; ++j)
#pragma unroll
            for (int b = 0; b <= 2 * D - j; ++b) {
                const double *f = fb + (size_t)qidx(j, b, 2 * D) * 768;
                F[j][b] = 0.5 * (f[i] + f[it]);
            }
#pragma unroll
        for (int p = 0; p <= 2 * D; ++p)
#pragma unroll
            for (int b = 0; b <= 2 * D - p; ++b) {
                double v = 0.0, xp = 1.0;      // x0^(p - j) from j = p down
#pragma unroll
                for (int j = p; j >= 0; --j) {
                    v += bin[p][j] * xp * F[j][b];
                    xp *= x0;
                }
                part[(size_t)qidx(p, b, 2 * D) * 768 + i] = v;
            }
    }
}

}  // namespace argus_fit
