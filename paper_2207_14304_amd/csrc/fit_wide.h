// Moment accumulation of the FP32 fit on wide frames (D >= 1), with the
// matrix products on BF16 instructions.
//
// On gfx950 FP32 MFMA and VALU cycles add up (they do not overlap), and the
// FP32 form of the fit (fit_accum8.h) spends half its time on FP32 MFMAs: 2D+1
// x-powers of every 64-pixel row segment.  Two things shrink that here.
//
// 1. Powers about the strip's centre.  With xt = x0 + d the moments are taken
//    in powers of d, |d| <= 31.5 * 2/(W-1), which the end of the kernel
//    combines into powers of xt (binomially, in FP64).  |d| is small on a wide
//    frame, so the higher powers need few bits to add nothing above FP32
//    rounding: at the narrowest frame taken (FIT_WIDE_MIN columns) |d| <=
//    2^-6.6, d^2 <= 2^-13, d^3 <= 2^-19, and d^4 is replaced by m^2 d^2 - m^4/8
//    (m the largest |d|; error m^4/8 <= 2^-29).
// 2. Split operands.  With s = sqrt(w) c' a power's moment is sum d^a s s^T.
//    s = h + m + l in bf16 (residual 2^-27 s); power 0 takes the six products
//    h h, h m, m h, h l, l h, m m (dropped terms 2^-26: below the 2^-24 of an
//    FP32 product); powers 1 and 2 take d^a s = h_a + m_a and h h_a + h m_a +
//    m h_a (2^-17 of a term that is 2^-6.6 and 2^-13 of power 0); power 3
//    takes h h_3.  Products are exact in FP32 and summed in FP32 over 64 pixels, as
//    before.  A diagonal block's m h and l h are the transposes of h m and h l
//    (one product each, doubled; the block is symmetrised at the end).
//
// The right-hand side is summed from the same s: FP32 products over 4 pixels,
// then FP64 per lane across rows.
//
// Waves and pipeline: 8 convolution waves (fit_conv8) write row y's c at step
// n; the 8 MFMA waves split it (4 basis rows each, a lane per row and 4
// pixels) into bf16 tables at step n + 1 and multiply them at step n + 2, one
// barrier per step.  Of the two MFMA waves of a SIMD one multiplies first and
// the other splits first, so that matrix and vector work meet.
//
// Full frame, D = 2, h = 10: 7.46 -> 4.95 ms against the FP32 form, the
// difference image as far from the 64-bit one as before (9.0e-6 and 9.2e-6
// relative).  Narrower frames keep the FP32 form: their |d| would need more
// products, and the frame's 2 D + 1 powers cost them less than the solve.
#pragma once
#include "fit_accum8.h"

namespace argus_fit {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

template <int D, int HH>
struct FitWideLds {
    using Base = FitLds8<D, HH, false>;
    static constexpr int CKB = SW + 8;                   // row stride of a table (16-byte rows)
    static constexpr int NJ = D == 1 ? 3 : 4;            // powers of d
    // tables of one buffer: h, m, l; h1, m1; h2, m2; h3
    static constexpr int NTAB = D == 1 ? 7 : 8;
    static constexpr int TAB = 32 * CKB;                 // bf16 values of a table
    static constexpr int NF = D == 1 ? 6 : 14;           // (power of d, power of yt) moments
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

// Tasks (power of d, block pair) of MFMA wave MW: at most two.  The loads are
// within 14..20 products per SIMD (waves MW and MW + 4 share one).
struct WideTask { int a, bp; };
template <int D>
__host__ __device__ constexpr WideTask wide_task(int mw, int i) {
    constexpr WideTask t2[8][2] = {{{0, 1}, {-1, 0}}, {{0, 0}, {-1, 0}}, {{0, 2}, {-1, 0}},
                                   {{1, 0}, {3, 0}},  {{1, 2}, {3, 2}},  {{1, 1}, {3, 1}},
                                   {{2, 0}, {2, 1}},  {{2, 2}, {-1, 0}}};
    constexpr WideTask t1[8][2] = {{{0, 1}, {-1, 0}}, {{0, 0}, {-1, 0}}, {{0, 2}, {-1, 0}},
                                   {{1, 0}, {-1, 0}}, {{1, 2}, {-1, 0}}, {{1, 1}, {-1, 0}},
                                   {{2, 0}, {2, 2}},  {{2, 1}, {-1, 0}}};
    return D == 1 ? t1[mw][i] : t2[mw][i];
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
    // the moments of one task over a row's 64 pixels; power 0: h h in acc, the
    // smaller products in cross
    auto task = [&](auto ta, auto tb, int buf, floatx4 &acc, floatx4 &cross) {
        constexpr int A = decltype(ta)::value, BP = decltype(tb)::value;
        constexpr int ra = BP == 2 ? 1 : 0, rb = BP == 0 ? 0 : 1;
        acc = cross = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (A == 0) {
#pragma unroll
            for (int s = 0; s < SW / 32; ++s) {
                const bf16x8 h0 = frag(buf, 0, ra, s), m0 = frag(buf, 1, ra, s), l0 = frag(buf, 2, ra, s);
                const bf16x8 h1 = ra == rb ? h0 : frag(buf, 0, rb, s);
                const bf16x8 m1 = ra == rb ? m0 : frag(buf, 1, rb, s);
                const bf16x8 l1 = ra == rb ? l0 : frag(buf, 2, rb, s);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, h1, acc, 0, 0, 0);
                cross = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, l1, cross, 0, 0, 0);
                cross = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l0, h1, cross, 0, 0, 0);
                cross = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m0, m1, cross, 0, 0, 0);
                cross = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h0, m1, cross, 0, 0, 0);
                cross = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m0, h1, cross, 0, 0, 0);
            }
        } else if constexpr (A == 3) {
#pragma unroll
            for (int s = 0; s < SW / 32; ++s)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(buf, 0, ra, s), frag(buf, 7, rb, s),
                                                              acc, 0, 0, 0);
        } else {
#pragma unroll
            for (int s = 0; s < SW / 32; ++s) {
                const bf16x8 h = frag(buf, 0, ra, s), m = frag(buf, 1, ra, s);
                const bf16x8 ha = frag(buf, 1 + 2 * A, rb, s), ma = frag(buf, 2 + 2 * A, rb, s);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, ma, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m, ha, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, ha, acc, 0, 0, 0);
            }
        }
    };
    auto flush = [&](auto ta, double (&F)[NB][4], floatx4 acc, floatx4 cross, const double *ypw) {
        constexpr int A = decltype(ta)::value;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double v = A == 0 ? (double)acc[r] + (double)cross[r] : (double)acc[r];
#pragma unroll
            for (int b = 0; b <= 2 * D - A; ++b) F[b][r] += ypw[b] * v;
        }
    };
    auto multiply = [&](int y, int buf) {
        double ypw[NB];
        ypowers(y, ypw);
        using A0 = std::integral_constant<int, T0.a>;
        floatx4 c0, x0, c1, x1;
        task(A0{}, std::integral_constant<int, T0.bp>{}, buf, c0, x0);
        if constexpr (T1.a >= 0) {
            using A1 = std::integral_constant<int, T1.a>;
            task(A1{}, std::integral_constant<int, T1.bp>{}, buf, c1, x1);
            flush(A0{}, F0, c0, x0, ypw);
            flush(A1{}, F1, c1, x1, ypw);
        } else {
            flush(A0{}, F0, c0, x0, ypw);
        }
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
        float u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = s[i] * dl[i];
        auto put = [&](int t, bf16x4 v) { *(bf16x4 *)(L::tab(lds, tb, t) + k * CKB + p4) = v; };
        const bf16x4 h = to_bf16(s);
        put(0, h);
        less(s, h);
        const bf16x4 m = to_bf16(s);
        put(1, m);
        less(s, m);
        put(2, to_bf16(s));
#pragma unroll
        for (int j = 1; j < 3; ++j) {
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = u[i];
            const bf16x4 hj = to_bf16(v);
            put(1 + 2 * j, hj);
            less(v, hj);
            put(2 + 2 * j, to_bf16(v));
            if (j == 1 || D == 2)
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] *= dl[i];
        }
        if constexpr (D == 2) put(7, to_bf16(u));
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
    // right-hand side: the 16 lanes of a basis row
#pragma unroll
    for (int i = 0; i < S::NR; ++i) {
        double r = RF[i];
        for (int off = 8; off > 0; off >>= 1) r += __shfl_xor(r, off);
        if (col == 0) part[(size_t)S::NQ * 768 + i * 32 + k] = r;
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
    // powers of xt = x0 + d: xt^p = sum_j C(p, j) x0^(p - j) d^j, with d^4 by
    // m^2 d^2 - m^4 / 8; diagonal blocks symmetrised
    const double *fb = (const double *)lds;
    const double x0 = ((double)sx0 + 31.5) * a.sx - 1.0;
    const double mm = (31.5 * a.sx) * (31.5 * a.sx);
    constexpr double bin[5][4] = {{1, 0, 0, 0}, {1, 1, 0, 0}, {1, 2, 1, 0}, {1, 3, 3, 1}, {1, 4, 6, 4}};
    for (int i = tid; i < 768; i += 1024) {
        const int bp = i >> 8, r = (i >> 4) & 15, c = i & 15;
        const int it = bp == 1 ? i : (bp << 8) + c * 16 + r;
        double F[L::NJ][2 * D + 1];
#pragma unroll
        for (int j = 0; j < L::NJ; ++j)
#pragma unroll
            for (int b = 0; b <= 2 * D; ++b)
                if (b <= 2 * D - j) {
                    const double *f = fb + (size_t)qidx(j, b, 2 * D) * 768;
                    F[j][b] = 0.5 * (f[i] + f[it]);
                }
#pragma unroll
        for (int p = 0; p <= 2 * D; ++p)
#pragma unroll
            for (int b = 0; b <= 2 * D; ++b)
                if (p + b <= 2 * D) {
                    double v = 0.0, xp = 1.0;      // x0^(p - j) from j = p down
#pragma unroll
                    for (int j = p; j >= 0; --j) {
                        if (j < L::NJ) v += bin[p][j] * xp * F[j][b];
                        xp *= x0;
                    }
                    if (p == 4) v += mm * F[2][b] - (mm * mm / 8.0) * F[0][b];
                    part[(size_t)qidx(p, b, 2 * D) * 768 + i] = v;
                }
    }
}

}  // namespace argus_fit
