// ZOGY subtraction (Zackay, Ofek & Gal-Yam 2016) on square tiles of a frame
// pair, in FP64 on the GPU.
//
// Per tile of side L (a power of two, 64..1024) at origin (x0, y0):
//   N^, R^ = 2-D FFTs of the new and reference tiles (masked or off-frame
//   pixels 0); with the PSF transforms P_n^, P_r^ (stamps centred on the
//   periodic tile's origin) shared by all tiles,
//     den = sqrt(s_n^2 F_r^2 |P_r^|^2 + s_r^2 F_n^2 |P_n^|^2)
//     D^ = (F_r P_r^ N^ - F_n P_n^ R^) / den,  P_D^ = F_r F_n P_r^ P_n^ / (F_D den)
//     S^ = D^ conj(P_D^),  F_D = F_n F_r / sqrt(s_n^2 F_r^2 + s_r^2 F_n^2);
//   D and S by inverse FFTs; SNR = S / sqrt(sum P_D^2) (Parseval over P_D^),
//   flux = S / (F_D sum P_D^2).  Outputs within r of the tile border are
//   EDGE, within 2r of a masked or off-frame pixel FOOT, and 0 there.
//
// The transforms move far more bytes than they compute, so the work is three
// passes over one 16-byte plane per tile (58 B read and 48 B written per
// tile pixel with the inputs and outputs):
//   rows     N + i g R (two real images, one complex transform) row by row; the
//            spectra go out transposed, [k_x][y];
//   columns  k_x and -k_x together in one workgroup: forward, N^ and R^ from
//            the symmetric and antisymmetric parts, D^ + i S^ (D and S are
//            real, so one inverse transform returns both), inverse, in place;
//            a workgroup keeps its columns' filter values in registers and
//            takes many tiles;
//   output   inverse rows, scaling, masks.
// Two images in one transform share its rounding, so they are brought to one
// scale by powers of two first: R by g = 2^k next to F_n / F_r (the images may
// be in any units), the reference's PSF by the one next to the ratio of the two
// maxima, S by the one next to 1 / sqrt(sum P_D^2) (the PSFs may have any sums).
// A length-L transform is L / 8 threads with 8 values each in registers and
// radix-8 steps (one radix-4 or -2 step where 3 does not divide log2 L)
// exchanged through LDS.  280 tiles of 512^2: 10.9 -> 1.69 ms, against two
// radix-2 transforms per direction with separate load, transpose, pointwise
// and dilation passes.
#include <math.h>

#include "internal.h"

namespace {

typedef double2 cplx;

__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return make_double2(a.x - b.x, a.y - b.y); }

// exp(-2 pi i k / L), k < L
__global__ void twiddle_kernel(cplx *tw, int L) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= L) return;
    double s, c;
    sincospi(2.0 * k / L, &s, &c);
    tw[k] = make_double2(c, -s);
}

// ---- length-L transforms over T = L / 8 threads ------------------------------
template <int LG>
struct Fft {
    static constexpr int L = 1 << LG, T = L / 8;
    static constexpr int NF = 4096 / L;        // rows of a 512-thread workgroup
    static constexpr int NP = 128 / T;         // column pairs of a 256-thread workgroup
    // LDS row in values: one pad per 8 (the radix-8 writes of consecutive
    // threads are 8 apart), and rows 2 mod 16 apart (the transposing reads
    // take 8 rows at a time)
    static constexpr int S = L + L / 8 + 2;
    static constexpr bool WAVE = T <= 64;      // a transform stays in one wave
    __device__ static int at(int i) { return i + (i >> 3); }
    __device__ static void sync() {
        if constexpr (WAVE) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    }
};

// multiply by -i (forward) or i (inverse)
template <bool INV>
__device__ __forceinline__ cplx rot(cplx a) {
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

template <bool INV>
__device__ __forceinline__ void dft4(cplx a, cplx b, cplx c, cplx d, cplx (&X)[4]) {
    const cplx s = cadd(a, c), t = csub(a, c), u = cadd(b, d), w = rot<INV>(csub(b, d));
    X[0] = cadd(s, u);
    X[1] = cadd(t, w);
    X[2] = csub(s, u);
    X[3] = csub(t, w);
}

template <bool INV>
__device__ __forceinline__ void dft8(cplx (&v)[8]) {
    cplx E[4], O[4];
    dft4<INV>(v[0], v[2], v[4], v[6], E);
    dft4<INV>(v[1], v[3], v[5], v[7], O);
    constexpr double c = 0.70710678118654752440;
    const double sg = INV ? 1.0 : -1.0;
    const cplx o1 = make_double2(c * (O[1].x - sg * O[1].y), c * (O[1].y + sg * O[1].x));
    const cplx o2 = rot<INV>(O[2]);
    const cplx o3 = make_double2(c * (-O[3].x - sg * O[3].y), c * (-O[3].y + sg * O[3].x));
    v[0] = cadd(E[0], O[0]); v[4] = csub(E[0], O[0]);
    v[1] = cadd(E[1], o1);   v[5] = csub(E[1], o1);
    v[2] = cadd(E[2], o2);   v[6] = csub(E[2], o2);
    v[3] = cadd(E[3], o3);   v[7] = csub(E[3], o3);
}

template <bool INV>
__device__ __forceinline__ cplx twid(const cplx *tw, int i) {
    cplx w = tw[i];
    if (INV) w.y = -w.y;
    return w;
}

// One self-sorting step of radix R after Ns points are done: the butterflies
// of this thread take its values v[r] = x[u + r T]; results go to their sorted
// places in LDS and the next step's values are read back, or, at the last
// step (Ns R = L), stay in v[r] = X[u + r T].
template <int LG, bool INV, int R, int Ns>
__device__ __forceinline__ void fft_step(cplx (&v)[8], int u, const cplx *tw, cplx *row) {
    using F = Fft<LG>;
    constexpr int Q = 8 / R;                   // butterflies per thread
    constexpr bool LAST = Ns * R == F::L;
    cplx y[8];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int j = u + q * F::T, jm = j & (Ns - 1);
        cplx x[8];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = v[q + r * Q];
        if constexpr (Ns > 1) {
            const cplx w1 = twid<INV>(tw, jm * (F::L / (Ns * R)));
            x[1] = cmul(x[1], w1);
            if constexpr (R >= 4) {
                const cplx w2 = cmul(w1, w1), w3 = cmul(w2, w1);
                x[2] = cmul(x[2], w2);
                x[3] = cmul(x[3], w3);
                if constexpr (R == 8) {
                    const cplx w4 = cmul(w2, w2);
                    x[4] = cmul(x[4], w4);
                    x[5] = cmul(x[5], cmul(w4, w1));
                    x[6] = cmul(x[6], cmul(w4, w2));
                    x[7] = cmul(x[7], cmul(w4, w3));
                }
            }
        }
        if constexpr (R == 8) {
            dft8<INV>(x);
        } else if constexpr (R == 4) {
            cplx X[4];
            dft4<INV>(x[0], x[1], x[2], x[3], X);
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = X[r];
        } else {
            const cplx t = x[1];
            x[1] = csub(x[0], t);
            x[0] = cadd(x[0], t);
        }
        const int o = (j - jm) * R + jm;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (LAST) y[q + r * Q] = x[r];
            else row[F::at(o + r * Ns)] = x[r];
        }
    }
    if constexpr (LAST) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = y[r];
    } else {
        F::sync();
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = row[F::at(u + r * F::T)];
        F::sync();
    }
}

// v[r] = x[u + r T] -> X[u + r T], through the thread group's LDS row
template <int LG, bool INV>
__device__ __forceinline__ void fft(cplx (&v)[8], int u, const cplx *tw, cplx *row) {
    fft_step<LG, INV, 8, 1>(v, u, tw, row);
    fft_step<LG, INV, 8, 8>(v, u, tw, row);
    if constexpr (LG == 7) fft_step<LG, INV, 2, 64>(v, u, tw, row);
    if constexpr (LG == 8) fft_step<LG, INV, 4, 64>(v, u, tw, row);
    if constexpr (LG >= 9) fft_step<LG, INV, 8, 64>(v, u, tw, row);
    if constexpr (LG == 10) fft_step<LG, INV, 2, 512>(v, u, tw, row);
}

// ---- passes --------------------------------------------------------------------
struct RowArgs {
    const float *N, *R;
    const uint8_t *mn, *mr;
    const int32_t *org;                // [n][2]: x0, y0
    int64_t pitch;
    int W, H, r, rad;                  // PSF half-width, flag radius
    const cplx *tw;
    cplx *Z;                           // [n][k_x][y]
    uint64_t *bits;                    // [n][y][L / 64]: flagged along x within rad
    double g;                          // scale of R
    double *gp;                        // scale of the reference's PSF, written by the PSF pass
};

// OR of the bits of the word `c` and its neighbours within rad (< 64) places
__device__ __forceinline__ uint64_t dilate_bits(uint64_t p, uint64_t c, uint64_t nx, int rad) {
    unsigned __int128 up = ((unsigned __int128)c << 64) | p;      // moved towards higher x
    unsigned __int128 dn = ((unsigned __int128)nx << 64) | c;     // towards lower x
    for (int d = 0; d < rad;) {
        const int s = min(d + 1, rad - d);
        up |= up << s;
        dn |= dn >> s;
        d += s;
    }
    return (uint64_t)(up >> 64) | (uint64_t)dn;
}

// Row transforms of N + i g R (PSF: of the two stamps wrapped onto the tile,
// centre at the origin, g from their maxima).
template <int LG, bool PSF>
__global__ __launch_bounds__(512) void zogy_rows_kernel(RowArgs a) {
    using F = Fft<LG>;
    constexpr int L = F::L, T = F::T, NF = F::NF, NW = L / 64;
    extern __shared__ cplx sm[];
    __shared__ uint64_t raw[64];               // [NF][NW] flagged pixels
    const int tid = threadIdx.x, f = tid / T, u = tid & (T - 1);
    const int t = blockIdx.x / (L / NF), y0 = (blockIdx.x % (L / NF)) * NF, y = y0 + f;
    cplx *row = sm + f * F::S;
    cplx v[8];
    if constexpr (PSF) {
        const int dv = y <= L / 2 ? y : y - L, K = 2 * a.r + 1;
        __shared__ float top[2][8];
        float mn = 0.f, mr = 0.f;
        for (int i = tid; i < K * K; i += 512) {
            mn = fmaxf(mn, fabsf(a.N[i]));
            mr = fmaxf(mr, fabsf(a.R[i]));
        }
        for (int o = 32; o > 0; o >>= 1) {
            mn = fmaxf(mn, __shfl_xor(mn, o));
            mr = fmaxf(mr, __shfl_xor(mr, o));
        }
        if ((tid & 63) == 0) {
            top[0][tid >> 6] = mn;
            top[1][tid >> 6] = mr;
        }
        __syncthreads();
        for (int i = 0; i < 8; ++i) {
            mn = fmaxf(mn, top[0][i]);
            mr = fmaxf(mr, top[1][i]);
        }
        const bool fin = mn > 0.f && mr > 0.f && mn < __builtin_inff() && mr < __builtin_inff();
        const double g = fin ? ldexp(1.0, ilogbf(mn) - ilogbf(mr)) : 1.0;
        if (blockIdx.x == 0 && tid == 0) *a.gp = g;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int x = u + r * T, du = x <= L / 2 ? x : x - L;
            const bool in = dv >= -a.r && dv <= a.r && du >= -a.r && du <= a.r;
            const int i = (dv + a.r) * K + du + a.r;
            v[r] = in ? make_double2(a.N[i], g * a.R[i]) : make_double2(0.0, 0.0);
        }
    } else {
        const int X0 = a.org[2 * t], Y = a.org[2 * t + 1] + y;
        const bool yin = Y >= 0 && Y < a.H;
        const int64_t o = (int64_t)(yin ? Y : 0) * a.pitch;
        float vn[8], vr[8];
        bool bad[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int X = X0 + u + r * T;
            const bool in = yin && X >= 0 && X < a.W;
            const int64_t i = o + (in ? X : 0);
            vn[r] = a.N[i];
            vr[r] = a.R[i];
            bad[r] = !in || a.mn[i] != 0 || a.mr[i] != 0;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            v[r] = bad[r] ? make_double2(0.0, 0.0) : make_double2(vn[r], a.g * vr[r]);
            const uint64_t b = __ballot(bad[r]);
            // the T bits of this row's pixels [r T, (r + 1) T)
            if constexpr (T >= 64) {
                if ((u & 63) == 0) raw[f * NW + r * (T / 64) + u / 64] = b;
            } else if (u == 0) {
                const uint64_t piece = b >> ((tid & 63) & ~(T - 1));
                if constexpr (T == 32) ((uint32_t *)&raw[f * NW])[r] = (uint32_t)piece;
                if constexpr (T == 16) ((uint16_t *)&raw[f * NW])[r] = (uint16_t)piece;
                if constexpr (T == 8) ((uint8_t *)&raw[f * NW])[r] = (uint8_t)piece;
            }
        }
    }
    fft<LG, false>(v, u, a.tw, row);
#pragma unroll
    for (int r = 0; r < 8; ++r) row[F::at(u + r * T)] = v[r];
    __syncthreads();
    cplx *Z = a.Z + (size_t)t * L * L;
    for (int i = tid; i < L * NF; i += 512) {
        const int rr = i % NF, kx = i / NF;
        Z[(size_t)kx * L + y0 + rr] = sm[rr * F::S + F::at(kx)];
    }
    if constexpr (!PSF) {
        if (tid < NF * NW) {
            const int w = tid % NW;
            a.bits[((size_t)t * L + y0) * NW + tid] =
                dilate_bits(w > 0 ? raw[tid - 1] : 0, raw[tid], w + 1 < NW ? raw[tid + 1] : 0, a.rad);
        }
    }
}

struct ZCoef {
    double Fn, Fr, sn2, sr2, FD;
};

// Filter values per frequency, [k_x][k_y]: D^ = A N^ - B (g R)^ with A = F_r P_r^
// / den and B = F_n P_n^ / (g den), conj(P_D^) = q conj(A B) with q = g den / F_D.
struct Filter {
    cplx *A, *B;
    double *q;
};

// Columns p and -p of pair p (p = 0: the columns 0 and L / 2, each its own
// mirror image), two thread groups per pair; the transform's values v[r] at
// k_y = u + r T and their mirror images m[r] at (-k_x, -k_y).
template <int LG>
struct Column {
    using F = Fft<LG>;
    int u, kx;
    cplx *own;
    const cplx *mirror;
    __device__ Column(cplx *sm) {
        const int tid = threadIdx.x, g = tid / (2 * F::T), side = (tid / F::T) & 1;
        u = tid & (F::T - 1);
        const int p = blockIdx.x * F::NP + g;
        kx = side == 0 ? p : (p == 0 ? F::L / 2 : F::L - p);
        own = sm + (2 * g + side) * F::S;
        mirror = p == 0 ? own : sm + (2 * g + 1 - side) * F::S;
    }
    __device__ void mirrored(const cplx (&v)[8], cplx (&m)[8]) const {
#pragma unroll
        for (int r = 0; r < 8; ++r) own[F::at(u + r * F::T)] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) m[r] = mirror[F::at((F::L - u - r * F::T) & (F::L - 1))];
        __syncthreads();
    }
};

// the two real images' transforms from v = X^ + i Y^ and its mirror image
__device__ __forceinline__ void split(cplx v, cplx m, cplx &X, cplx &Y) {
    X = make_double2(0.5 * (v.x + m.x), 0.5 * (v.y - m.y));
    Y = make_double2(0.5 * (v.y + m.y), 0.5 * (m.x - v.x));
}

// The power of two next to 1 / sqrt(pd2), the scale that S is carried at.
__device__ __forceinline__ double score_scale(double pd2) {
    return pd2 > 0.0 && pd2 < __builtin_inf() ? ldexp(1.0, -(ilogb(pd2) >> 1)) : 1.0;
}

// Filter values from the PSF plane, and each workgroup's sum of |P_D^|^2.
template <int LG>
__global__ __launch_bounds__(256) void zogy_filter_kernel(const cplx *Z, const cplx *tw, ZCoef c,
                                                          double g, const double *gp, Filter fl,
                                                          double *part) {
    using F = Fft<LG>;
    extern __shared__ cplx sm[];
    __shared__ double red[4];
    const Column<LG> col(sm);
    const double ip = 1.0 / *gp;
    cplx v[8], m[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = Z[(size_t)col.kx * F::L + col.u + r * F::T];
    fft<LG, false>(v, col.u, tw, col.own);
    col.mirrored(v, m);
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        cplx Pn, Pr;
        split(v[r], m[r], Pn, Pr);
        Pr = make_double2(ip * Pr.x, ip * Pr.y);
        const double an = Pn.x * Pn.x + Pn.y * Pn.y, ar = Pr.x * Pr.x + Pr.y * Pr.y;
        const double den = sqrt(c.sn2 * c.Fr * c.Fr * ar + c.sr2 * c.Fn * c.Fn * an);
        const double ia = den > 0.0 ? c.Fr / den : 0.0, ib = den > 0.0 ? c.Fn / den / g : 0.0;
        const cplx A = make_double2(ia * Pr.x, ia * Pr.y), B = make_double2(ib * Pn.x, ib * Pn.y);
        const double q = g * (den / c.FD);
        const size_t i = (size_t)col.kx * F::L + col.u + r * F::T;
        fl.A[i] = A;
        fl.B[i] = B;
        fl.q[i] = q;
        const cplx ab = cmul(A, B);
        s += q * q * (ab.x * ab.x + ab.y * ab.y);
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// sum P_D^2 = sum |P_D^|^2 / L^2: one wave over the workgroups' sums, fixed order
__global__ __launch_bounds__(64) void zogy_pd2_kernel(const double *part, int n, double inv_ll,
                                                      double *pd2) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 64) s += part[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (threadIdx.x == 0) *pd2 = s * inv_ll;
}

// Columns of the tiles [blockIdx.y per, ...): forward, filter, inverse.
template <int LG>
__global__ __launch_bounds__(256) void zogy_columns_kernel(cplx *Z, const cplx *tw, Filter fl,
                                                           const double *pd2, int n, int per) {
    using F = Fft<LG>;
    constexpr int L = F::L, T = F::T;
    extern __shared__ cplx sm[];
    const Column<LG> col(sm);
    cplx A[8], B[8];
    double q[8];
    const size_t o = (size_t)col.kx * L + col.u;
    const double sc = score_scale(*pd2);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        A[r] = fl.A[o + r * T];
        B[r] = fl.B[o + r * T];
        q[r] = sc * fl.q[o + r * T];
    }
    const int t1 = min((int)(blockIdx.y + 1) * per, n);
    for (int t = blockIdx.y * per; t < t1; ++t) {
        cplx *z = Z + (size_t)t * L * L + o;
        cplx v[8], m[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = z[r * T];
        fft<LG, false>(v, col.u, tw, col.own);
        col.mirrored(v, m);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            cplx N, R;
            split(v[r], m[r], N, R);
            const cplx D = csub(cmul(A[r], N), cmul(B[r], R));
            cplx ab = cmul(A[r], B[r]);
            ab = make_double2(q[r] * ab.x, -q[r] * ab.y);
            const cplx S = cmul(D, ab);
            v[r] = make_double2(D.x - S.y, D.y + S.x);
        }
        fft<LG, true>(v, col.u, tw, col.own);
#pragma unroll
        for (int r = 0; r < 8; ++r) z[r * T] = v[r];
    }
}

struct OutArgs {
    const cplx *Z, *tw;
    const uint64_t *bits;
    const double *pd2;
    float *D, *snr, *flux;
    uint8_t *mask;
    double FD;
    int r, rad;
};

template <int LG>
__global__ __launch_bounds__(512) void zogy_out_kernel(OutArgs a) {
    using F = Fft<LG>;
    constexpr int L = F::L, T = F::T, NF = F::NF, NW = L / 64;
    extern __shared__ cplx sm[];
    __shared__ uint64_t foot[64];              // [NF][NW]: flagged within rad in x and y
    const int tid = threadIdx.x, f = tid / T, u = tid & (T - 1);
    const int t = blockIdx.x / (L / NF), y0 = (blockIdx.x % (L / NF)) * NF, y = y0 + f;
    const cplx *Z = a.Z + (size_t)t * L * L;
    for (int i = tid; i < L * NF; i += 512) {
        const int rr = i % NF, kx = i / NF;
        sm[rr * F::S + F::at(kx)] = Z[(size_t)kx * L + y0 + rr];
    }
    if (tid < NF * NW) {
        const int yy = y0 + tid / NW;
        uint64_t b = 0;
        for (int v = max(yy - a.rad, 0); v <= min(yy + a.rad, L - 1); ++v)
            b |= a.bits[((size_t)t * L + v) * NW + tid % NW];
        foot[tid] = b;
    }
    __syncthreads();
    cplx *row = sm + f * F::S;
    cplx v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = row[F::at(u + r * T)];
    F::sync();
    fft<LG, true>(v, u, a.tw, row);
    const double inv = 1.0 / ((double)L * L), pd2 = *a.pd2;
    const double sc = score_scale(pd2), is = 1.0 / sqrt(pd2) / sc, ifl = 1.0 / (a.FD * pd2) / sc;
    const bool yedge = y < a.r || y >= L - a.r;
    const size_t o = ((size_t)t * L + y) * L;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int x = u + r * T;
        uint8_t m = (yedge || x < a.r || x >= L - a.r) ? ARGUS_EDGE : 0;
        if ((foot[f * NW + x / 64] >> (x & 63)) & 1) m |= ARGUS_FOOT;
        const double D = v[r].x * inv, S = v[r].y * inv;
        a.D[o + x] = m ? 0.f : (float)D;
        a.snr[o + x] = m ? 0.f : (float)(S * is);
        a.flux[o + x] = m ? 0.f : (float)(S * ifl);
        a.mask[o + x] = m;
    }
}

struct ZCall {
    RowArgs rows;
    OutArgs out;
    ZCoef c;
    const float *psf_n, *psf_r;
    cplx *tw, *Z, *psf;
    Filter fl;
    double *part, *pd2;
    int n;
};

template <int LG>
int zogy_run(argus_ctx *ctx, ZCall &z) {
    using F = Fft<LG>;
    constexpr int L = F::L;
    const size_t row_lds = (size_t)F::NF * F::S * sizeof(cplx);
    const size_t col_lds = (size_t)2 * F::NP * F::S * sizeof(cplx);
    for (const void *f : {(const void *)zogy_rows_kernel<LG, true>, (const void *)zogy_rows_kernel<LG, false>,
                          (const void *)zogy_out_kernel<LG>})
        ARGUS_HIP_CHECK(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)row_lds));
    hipStream_t st = ctx->stream;
    const int pairs = L / 2 / F::NP;           // workgroups that hold every column pair
    // tiles per column workgroup: as many as leave 8 workgroups per CU (its
    // 80 registers of filter values are loaded once per workgroup)
    const int ncu = ctx->n_cu > 0 ? ctx->n_cu : 256;
    const int groups = max(1, min(z.n, 8 * ncu / pairs));
    const int per = (z.n + groups - 1) / groups;
    argus_time_begin(ctx);
    hipLaunchKernelGGL(twiddle_kernel, dim3((L + 255) / 256), dim3(256), 0, st, z.tw, L);
    RowArgs p = z.rows;
    p.N = z.psf_n;
    p.R = z.psf_r;
    p.Z = z.psf;
    hipLaunchKernelGGL((zogy_rows_kernel<LG, true>), dim3(L / F::NF), dim3(512), row_lds, st, p);
    hipLaunchKernelGGL(zogy_filter_kernel<LG>, dim3(pairs), dim3(256), col_lds, st,
                       (const cplx *)z.psf, (const cplx *)z.tw, z.c, z.rows.g, (const double *)z.rows.gp, z.fl, z.part);
    hipLaunchKernelGGL(zogy_pd2_kernel, dim3(1), dim3(64), 0, st, (const double *)z.part, pairs,
                       1.0 / ((double)L * L), z.pd2);
    hipLaunchKernelGGL((zogy_rows_kernel<LG, false>), dim3(z.n * (L / F::NF)), dim3(512), row_lds, st,
                       z.rows);
    hipLaunchKernelGGL(zogy_columns_kernel<LG>, dim3(pairs, (z.n + per - 1) / per), dim3(256), col_lds,
                       st, z.Z, (const cplx *)z.tw, z.fl, (const double *)z.pd2, z.n, per);
    hipLaunchKernelGGL(zogy_out_kernel<LG>, dim3(z.n * (L / F::NF)), dim3(512), row_lds, st, z.out);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    argus_time_end(ctx, "zogy");
    return ARGUS_OK;
}

}  // namespace

int launch_zogy(argus_ctx *ctx, argus_dims d, const float *N, const uint8_t *mn, const float *R,
                const uint8_t *mr, const int32_t *origins, int n, int L, const float *psf_n,
                const float *psf_r, int r, double Fn, double Fr, double sn, double sr, float *D,
                float *snr, float *flux, uint8_t *mask, double *pd2_out) {
    const size_t LL = (size_t)L * L;
    // workspace: a spectrum plane per tile, the PSF plane, the filter values,
    // twiddles, the flag bits, partial sums and sum P_D^2
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const size_t o_psf = al(n * LL * sizeof(cplx)), o_a = o_psf + al(LL * sizeof(cplx)),
                 o_b = o_a + al(LL * sizeof(cplx)), o_q = o_b + al(LL * sizeof(cplx)),
                 o_tw = o_q + al(LL * sizeof(double)), o_bits = o_tw + al(L * sizeof(cplx)),
                 o_part = o_bits + al(n * LL / 8), o_pd2 = o_part + al(L * sizeof(double)),
                 total = o_pd2 + 256;
    int rc = argus_ws_reserve(ctx, total);
    if (rc) return rc;
    char *ws = (char *)ctx->ws;
    ZCall z;
    z.Z = (cplx *)ws;
    z.psf = (cplx *)(ws + o_psf);
    z.fl = Filter{(cplx *)(ws + o_a), (cplx *)(ws + o_b), (double *)(ws + o_q)};
    z.tw = (cplx *)(ws + o_tw);
    z.part = (double *)(ws + o_part);
    z.pd2 = pd2_out ? pd2_out : (double *)(ws + o_pd2);
    z.psf_n = psf_n;
    z.psf_r = psf_r;
    z.n = n;
    z.c.Fn = Fn; z.c.Fr = Fr; z.c.sn2 = sn * sn; z.c.sr2 = sr * sr;
    z.c.FD = Fn * Fr / sqrt(z.c.sn2 * Fr * Fr + z.c.sr2 * Fn * Fn);
    uint64_t *bits = (uint64_t *)(ws + o_bits);
    // (an FP32 image times 2^+-800 is a normal FP64 number)
    const int k = ilogb(Fn) - ilogb(Fr);
    const double g = ldexp(1.0, k < -800 ? -800 : k > 800 ? 800 : k);
    z.rows = RowArgs{N, R, mn, mr, origins, d.pitch, d.width, d.height, r, 2 * r, z.tw, z.Z, bits, g,
                     (double *)(ws + o_pd2) + 1};
    z.out = OutArgs{z.Z, z.tw, bits, z.pd2, D, snr, flux, mask, z.c.FD, r, 2 * r};
    switch (L) {
        case 64: return zogy_run<6>(ctx, z);
        case 128: return zogy_run<7>(ctx, z);
        case 256: return zogy_run<8>(ctx, z);
        case 512: return zogy_run<9>(ctx, z);
        case 1024: return zogy_run<10>(ctx, z);
    }
    return argus_fail(ctx, ARGUS_ESHAPE, "argus_zogy: tile side %d", L);
}
