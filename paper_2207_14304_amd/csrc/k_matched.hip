// Matched-filter coadd of registered images (the per-image matched filter of
// Zackay & Ofek 2017 that the paper's deep coadds use):
//
//   S(q)   = sum_j F_j   sum_u P_j(u)   M_j(q + u) / V_j(q + u)
//   Var(q) = sum_j F_j^2 sum_u P_j(u)^2            / V_j(q + u)
//
// with M_j = cal_j - bg_j (bg_j the bilinear background of a filtered cell
// grid, or 0), over in-image pixels with mask 0 and V > 0.  One workgroup per
// 128 x 16 output pixels; per image the halo tile of M/V and 1/V is staged in
// LDS (every load of a thread issued before any is used), the image's
// F P and F^2 P^2 taps sit in LDS, and a thread owns 8 consecutive pixels of a
// row with the two windows of a PSF row in registers: 2 FMA per tap, pixel
// and image.  FP32 products summed in FP32 along a PSF row; the row sums are
// added in FP64 (a long FP32 sum over all taps and images lost ~1e-6 of the
// bright stars' scores).
#include "internal.h"
#include "background.h"

namespace {

constexpr int BW = 128, BH = 16, PXT = 8, NTHR = 256;

struct MatchedArgs {
    const float *cal[ARGUS_MAX_FRAMES];
    const float *var[ARGUS_MAX_FRAMES];
    const uint8_t *mask[ARGUS_MAX_FRAMES];
    BgGrid bg[ARGUS_MAX_FRAMES];       // grid == nullptr: no background
    float F[ARGUS_MAX_FRAMES];
    const float *psf;                  // [n][K][K]
    float *S, *Var, *snr;
    int64_t pitch;
    int W, H, n, bx;                   // bx: blocks along x
};

template <int R, int TX, int TY, int PX>
struct MLds {
    static constexpr int K = 2 * R + 1;
    static constexpr int TH = TY + 2 * R;
    static constexpr int TWr = TX + 2 * R;
    static constexpr int TW = (TWr + 3) & ~3;
    static constexpr int NT = TX / PX * TY;              // threads
    static constexpr size_t bytes = (size_t)(2 * TH * TW + 2 * K * K + 8) * 4;
};

// Sums of a TX x TY tile, PX consecutive pixels of a row per thread: s the
// scores of the pixels from (lx0, ly) on, v their variances.
template <int R, int TX, int TY, int PX>
__device__ __forceinline__ void matched_tile(const MatchedArgs &a, float *lds, int bx0, int by0,
                                             int ly, int lx0, double (&s)[PX], double (&v)[PX]) {
    using L = MLds<R, TX, TY, PX>;
    constexpr int K = L::K, TH = L::TH, TW = L::TW, TWr = L::TWr, NT = L::NT;
    // unrolled as the compiler sees fit, a small PSF's rows run 12 % faster; a
    // large one's spill
    constexpr bool ROLLED = PX == 4 || R > 4;
    float *At = lds;                   // [TH][TW] M / V
    float *Bt = At + TH * TW;          // [TH][TW] 1 / V
    float *Pt = Bt + TH * TW;          // [K*K][2] F p, F^2 p^2
    const int tid = threadIdx.x;
    const int64_t P = a.pitch;
    // FP32 sums along a PSF row, FP64 across rows and images
#pragma unroll
    for (int i = 0; i < PX; ++i) { s[i] = 0.0; v[i] = 0.0; }
    for (int j = 0; j < a.n; ++j) {
        __syncthreads();                                  // the previous image's reads are done
        const float *cal = a.cal[j], *var = a.var[j];
        const uint8_t *msk = a.mask[j];
        const BgGrid bg = a.bg[j];
        constexpr int NE = TH * TWr, NH = (NE + NT - 1) / NT, NB = PX == 8 ? 8 : 4;
        auto stage = [&](int j0) {
            float hc[NB], hv[NB];
            uint8_t hm[NB];
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                const int i = tid + (j0 + e) * NT;
                const int ii = i < NE ? i : 0;
                int X = bx0 - R + ii % TWr, Y = by0 - R + ii / TWr;
                X = X < 0 ? 0 : (X >= a.W ? a.W - 1 : X);
                Y = Y < 0 ? 0 : (Y >= a.H ? a.H - 1 : Y);
                const int64_t o = (int64_t)Y * P + X;
                hc[e] = cal[o];
                hv[e] = var[o];
                hm[e] = msk[o];
            }
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                const int i = tid + (j0 + e) * NT;
                if (i < NE) {
                    const int cy = i / TWr, cx = i % TWr;
                    const int X = bx0 - R + cx, Y = by0 - R + cy;
                    const bool ok = X >= 0 && X < a.W && Y >= 0 && Y < a.H && hm[e] == 0 &&
                                    hv[e] > 0.f;
                    float m = hc[e];
                    if (bg.grid && ok) m -= bg_at(bg, X, Y);
                    At[cy * TW + cx] = ok ? m / hv[e] : 0.f;
                    Bt[cy * TW + cx] = ok ? 1.f / hv[e] : 0.f;
                }
            }
        };
        if constexpr (ROLLED) {
#pragma unroll 1
            for (int j0 = 0; j0 < NH; j0 += NB) stage(j0);
        } else {
            for (int j0 = 0; j0 < NH; j0 += NB) stage(j0);
        }
        const float *pj = a.psf + (size_t)j * K * K;
        const float F = a.F[j];
        for (int t = tid; t < K * K; t += NT) {
            const float p = pj[t];
            Pt[2 * t] = F * p;
            Pt[2 * t + 1] = (F * F) * (p * p);
        }
        __syncthreads();
        auto row = [&](int dv) {
            // the windows of this PSF row as 16-byte reads (rows are 16-byte
            // aligned; the last read may pass the window by up to three
            // floats, still inside the LDS carve-up)
            constexpr int NW4 = (PX + 2 * R + 3) / 4;
            const float4 *ra = (const float4 *)(At + (ly + dv) * TW + lx0);
            const float4 *rb = (const float4 *)(Bt + (ly + dv) * TW + lx0);
            float wa[4 * NW4], wb[4 * NW4];
#pragma unroll
            for (int q = 0; q < NW4; ++q) {
                const float4 x4 = ra[q], y4 = rb[q];
                wa[4 * q] = x4.x; wa[4 * q + 1] = x4.y; wa[4 * q + 2] = x4.z; wa[4 * q + 3] = x4.w;
                wb[4 * q] = y4.x; wb[4 * q + 1] = y4.y; wb[4 * q + 2] = y4.z; wb[4 * q + 3] = y4.w;
            }
            float rs[PX], rv[PX];
#pragma unroll
            for (int i = 0; i < PX; ++i) { rs[i] = 0.f; rv[i] = 0.f; }
#pragma unroll
            for (int du = 0; du < K; ++du) {
                const float2 pp = *(const float2 *)(Pt + 2 * (dv * K + du));
#pragma unroll
                for (int i = 0; i < PX; ++i) {
                    rs[i] += pp.x * wa[i + du];
                    rv[i] += pp.y * wb[i + du];
                }
            }
#pragma unroll
            for (int i = 0; i < PX; ++i) {
                s[i] += (double)rs[i];
                v[i] += (double)rv[i];
            }
        };
        if constexpr (ROLLED) {
#pragma unroll 1
            for (int dv = 0; dv < K; ++dv) row(dv);
        } else {
            for (int dv = 0; dv < K; ++dv) row(dv);
        }
    }
}

template <int R>
__global__ __launch_bounds__(NTHR, 2) void matched_kernel(MatchedArgs a) {
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x;
    const int bx0 = (blockIdx.x % a.bx) * BW, by0 = (blockIdx.x / a.bx) * BH;
    const int64_t P = a.pitch;
    const int ly = tid / (BW / PXT), lx0 = (tid % (BW / PXT)) * PXT;
    double s[PXT], v[PXT];
    matched_tile<R, BW, BH, PXT>(a, lds, bx0, by0, ly, lx0, s, v);
    const int Y = by0 + ly;
    if (Y >= a.H) return;
    const int64_t orow = (int64_t)Y * P;
#pragma unroll
    for (int i = 0; i < PXT; ++i) {
        const int X = bx0 + lx0 + i;
        if (X < a.W) {
            a.S[orow + X] = (float)s[i];
            a.Var[orow + X] = (float)v[i];
            if (a.snr) a.snr[orow + X] = v[i] > 0.0 ? (float)(s[i] / sqrt(v[i])) : 0.f;
        }
    }
}

// ---- PSF half-widths up to 8: the taps on BF16 matrix instructions -------------
//
// With the PSF constant over a frame, a PSF row's sums over 16 output columns
// are a product with a 32 x 16 Toeplitz matrix, out[y][x] += sum_k A[y+dv][k]
// T_dv[k][x], T_dv[k][x] = P[dv][k - x]: one v_mfma_f32_16x16x32_bf16 for 256
// outputs.  47 % of its products are taps at 15 x 15, but the instruction has
// 32 times the VALU's FP32 rate, so the six products that keep FP32 accuracy
// (h + m + l splits of both operands, residual 2^-27; h h, h m, m h, h l, l h,
// m m) still take 2.5 times less issue time than FMAs; sums stay FP32 along a
// PSF row and FP64 across rows and images.
//
// One workgroup of 8 waves per 64 x 32 outputs, two workgroups a CU (one stages
// while the other multiplies).  Per image the tile of M/V and 1/V is staged in
// LDS as six bf16 planes (16-byte loads: its columns start at x - 8, aligned for
// every half-width) beside the image's split taps, from which a lane reads its
// column of T_dv as words; four waves take the score and four its variance, each
// every fourth PSF row for all 8 blocks of 16 x 16 outputs, and the waves' FP64
// sums meet in LDS at the end.  0 * non-finite would reach outputs outside the
// PSF's support, and values of extreme exponent lose their low parts: a tile
// with such values takes the FP32 form instead (matched_tile; a frame of nothing
// else, 1500 x 1000, 3 images: 128 us against 117 with matched_kernel and 83 with
// the splits).  An infinite variance is only a zero weight, and stays.  4788 x
// 3194, 5 images, 15 x 15: 1.72 -> 0.93 ms (VALU issue 0.49 and MFMA 0.35 of it,
// which hardly overlap).
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x1 __attribute__((ext_vector_type(1)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int POSITIVE_FINITE = 0x180;                   // class mask: positive normal or subnormal

template <int R>
struct XLds {
    static constexpr int TX = 64, TY = 32, NT = 512, K = 2 * R + 1;
    static constexpr int LEFT = 8;                       // tile columns before the outputs
    static constexpr int COLS = TX + 16, ROWS = TY + 2 * R;
    static constexpr int RS = COLS + 8;                  // row stride (16-byte rows, bank spread)
    static constexpr int PL = ROWS * RS;                 // values of a plane
    static constexpr int NB = 8;                         // 16 x 16 blocks, 4 across
    static constexpr int QR = COLS / 4, NQ = QR * ROWS, NIT = (NQ + NT - 1) / NT;
    static constexpr size_t sums = (size_t)4 * NB * 256 * 8;
    static constexpr size_t tile = (size_t)6 * PL * 2;
    // an image's taps after the tile: [score, variance][h, m, l][parity][K][TL]
    // bf16, tap index -16..31 (zero outside the PSF); the second copy starts one
    // tap later, so eight taps from any index are aligned words of one of them
    static constexpr int TL = 48, TP = K * TL;
    static constexpr size_t need = tile + (size_t)12 * TP * 2;
    static constexpr size_t bytes = sums > need ? sums : need;
};

// h + m + l = v (residual 2^-27 v)
template <int N, class V>
__device__ __forceinline__ void split3(float (&v)[N], V &h, V &m, V &l) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        h[i] = (__bf16)v[i];
        v[i] -= (float)h[i];
        m[i] = (__bf16)v[i];
        l[i] = (__bf16)(v[i] - (float)m[i]);
    }
}

template <int R>
__global__ __launch_bounds__(512, 4) void matched_mfma_kernel(MatchedArgs a, int vec) {
    using L = XLds<R>;
    extern __shared__ __align__(16) char xl[];
    __shared__ __align__(16) float scx[L::COLS];         // background weights and nodes of columns
    __shared__ __align__(16) int scn[L::COLS];
    __shared__ float srx[L::ROWS];                       // and rows
    __shared__ int srn[L::ROWS];
    __shared__ uint32_t high;                            // see range()
    __shared__ uint8_t tapok[ARGUS_MAX_FRAMES], taplow[ARGUS_MAX_FRAMES];
    __bf16 *tile = (__bf16 *)xl;                         // planes: M/V h, m, l; 1/V h, m, l
    __bf16 *taps = tile + 6 * L::PL;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, pk = lane >> 4;
    const int lb = argus_xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int x0 = lb % a.bx * L::TX, y0 = lb / a.bx * L::TY;
    const int64_t P = a.pitch;
    const int half = wv >> 2;                            // 0: score, 1: its variance
    if (tid == 0) high = 0;
    if (tid < ARGUS_MAX_FRAMES) tapok[tid] = taplow[tid] = 0;
    {
        // (every image's grid has the same cells)
        BgGrid g = a.bg[0];
        for (int j = 1; j < a.n; ++j)
            if (a.bg[j].grid) g = a.bg[j];
        if (g.grid) {
            if (tid < L::COLS) bg_axis(min(max(x0 - L::LEFT + tid, 0), a.W - 1), g.box, g.gx, g.cxl, scn[tid], scx[tid]);
            else if (tid >= 128 && tid < 128 + L::ROWS)
                bg_axis(min(max(y0 - R + tid - 128, 0), a.H - 1), g.box, g.gy, g.cyl, srn[tid - 128], srx[tid - 128]);
        }
    }
    float4 qc, qv;
    uint32_t qm;
    auto fetch = [&](int j, int e) {
        const float *cal = a.cal[j], *var = a.var[j];
        const uint8_t *msk = a.mask[j];
        {
            const int i = min(tid + e * L::NT, L::NQ - 1);
            const int X = x0 - L::LEFT + 4 * (i % L::QR), Y = min(max(y0 - R + i / L::QR, 0), a.H - 1);
            const int64_t o = (int64_t)Y * P;
            if (vec && X >= 0 && X + 3 < a.W) {
                qc = *(const float4 *)(cal + o + X);
                qv = *(const float4 *)(var + o + X);
                qm = *(const uint32_t *)(msk + o + X);
            } else {
                float c[4], v[4];
                uint32_t m = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t ok = o + min(max(X + k, 0), a.W - 1);
                    c[k] = cal[ok];
                    v[k] = var[ok];
                    m |= (uint32_t)msk[ok] << (8 * k);
                }
                qc = make_float4(c[0], c[1], c[2], c[3]);
                qv = make_float4(v[0], v[1], v[2], v[3]);
                qm = m;
            }
        }
    };
    auto stage = [&](int j) {
        const BgGrid bg = a.bg[j];
        // largest magnitude, and a sum that is NaN after an infinity or NaN
        float big = 0.f, fin = 0.f;
#pragma unroll 1
        for (int e = 0; e < L::NIT; ++e) {
            const int i = tid + e * L::NT;
            if (i >= L::NQ) break;
            fetch(j, e);
            const int cx = 4 * (i % L::QR), cy = i / L::QR;
            const int X = x0 - L::LEFT + cx, Y = y0 - R + cy;
            const float c[4] = {qc.x, qc.y, qc.z, qc.w};
            const float v[4] = {qv.x, qv.y, qv.z, qv.w};
            float A[4], B[4], g[4] = {0.f, 0.f, 0.f, 0.f};
            if (bg.grid) {
                const int iy = srn[cy], iy1 = iy + 1 < bg.gy ? iy + 1 : iy;
                const float ty = srx[cy];
                const float *r0 = bg.grid + (size_t)iy * bg.gx, *r1 = bg.grid + (size_t)iy1 * bg.gx;
                const float4 tx = *(const float4 *)&scx[cx];
                const int4 ix = *(const int4 *)&scn[cx];
                const float tv[4] = {tx.x, tx.y, tx.z, tx.w};
                const int iv[4] = {ix.x, ix.y, ix.z, ix.w};
                auto at = [&](int i, float &p, float &dp, float &q, float &dq) {
                    const int i1 = i + 1 < bg.gx ? i + 1 : i;
                    p = r0[i];
                    dp = r0[i1] - p;
                    q = r1[i];
                    dq = r1[i1] - q;
                };
                float top, dtop, bot, dbot;
                at(iv[0], top, dtop, bot, dbot);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (iv[k] != iv[0]) at(iv[k], top, dtop, bot, dbot);
                    const float t = top + tv[k] * dtop, u = bot + tv[k] * dbot;
                    g[k] = t + ty * (u - t);
                }
            }
            const bool yin = Y >= 0 && Y < a.H;
            float vbig = 0.f, mm[4];
            uint32_t used = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // (an infinite variance is a zero weight)
                const bool in = yin && X + k >= 0 && X + k < a.W && ((qm >> (8 * k)) & 0xffu) == 0;
                const bool ok = in && __builtin_amdgcn_classf(v[k], POSITIVE_FINITE);
                const float m = c[k] - g[k];
                // 1 / V by one Newton step, m / V from it by one correction
                float rv = __builtin_amdgcn_rcpf(v[k]);
                rv = fmaf(fmaf(-v[k], rv, 1.f), rv, rv);
                const float q = m * rv, mv = fmaf(fmaf(-q, v[k], m), rv, q);
                B[k] = ok ? rv : 0.f;
                A[k] = ok ? mv : 0.f;
                big = fmaxf(big, fmaxf(fabsf(A[k]), B[k]));
                vbig = fmaxf(vbig, v[k]);
                if (in) used |= 1u << k;
                mm[k] = m;
                fin = fmaf(A[k], 0.f, fmaf(B[k], 0.f, fin));
            }
            if (vbig > 1e30f) {
                // rare: a weight too small for the split, or none under a value
                // that is not finite
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if ((used >> k) & 1u && v[k] > 1e30f && (v[k] < __builtin_inff() || !(fabsf(mm[k]) < __builtin_inff())))
                        big = __builtin_inff();
            }
            __bf16 *t = tile + cy * L::RS + cx;
            bf16x4 h, m, l;
            split3(A, h, m, l);
            *(bf16x4 *)t = h;
            *(bf16x4 *)(t + L::PL) = m;
            *(bf16x4 *)(t + 2 * L::PL) = l;
            split3(B, h, m, l);
            *(bf16x4 *)(t + 3 * L::PL) = h;
            *(bf16x4 *)(t + 4 * L::PL) = m;
            *(bf16x4 *)(t + 5 * L::PL) = l;
        }
        // the image's taps
        const float *pj = a.psf + (size_t)j * L::K * L::K;
        const float F = a.F[j];
        float tap = 0.f;                                 // largest |F p| (its square for F^2 p^2)
        for (int i = tid; i < L::TP; i += L::NT) {
            const int dv = i / L::TL, t = i % L::TL, du = t - 16 - (L::LEFT - R);
            const float p = du >= 0 && du < L::K ? pj[dv * L::K + du] : 0.f;
            float v1[1] = {F * p}, v2[1] = {(F * F) * (p * p)};
            tap = fmaxf(tap, fabsf(v1[0]));
            fin = fmaf(v1[0], 0.f, fin);
            __bf16 sp[2][3];
            bf16x1 h, m, l;
            split3(v1, h, m, l);
            sp[0][0] = h[0]; sp[0][1] = m[0]; sp[0][2] = l[0];
            split3(v2, h, m, l);
            sp[1][0] = h[0]; sp[1][1] = m[0]; sp[1][2] = l[0];
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                __bf16 *d = taps + 2 * q * L::TP + dv * L::TL;
                d[t] = sp[q / 3][q % 3];
                if (t > 0) d[L::TP + t - 1] = sp[q / 3][q % 3];
            }
        }
        if (__any(big >= 1e4f || tap >= 4.f || fin != 0.f)) {
            const uint32_t h = (__any(!(big < 1e36f) || !(tap < 1e15f) || fin != 0.f) ? 1u : 0u) |
                               (__any(big >= 1e4f) ? 2u : 0u) | (__any(big >= 1e28f) ? 4u : 0u) |
                               (__any(tap >= 4.f) ? 8u : 0u) | (__any(tap >= 1e4f) ? 16u : 0u);
            if (lane == 0) atomicOr(&high, h);
        }
        if (__any(tap >= 1e-14f)) {
            if (lane == 0) tapok[j] = 1;
        } else if (__any(tap > 0.f) && lane == 0) {
            taplow[j] = 1;
        }
    };
    // Whether the sums stay inside the split's range: every value finite, no
    // product above 1e36 (1/V or M/V below 1e4, 1e28, 1e36 with F^2 p^2 below 1e30,
    // 1e8, 16), and image j's taps large enough (1e-28, with 1/V at least 1e-30)
    // that the low parts of all that matter are normal numbers.
    auto range = [&](int j) {
        return !(high & 1u) && (high & 18u) != 18u && (high & 12u) != 12u && (tapok[j] || !taplow[j]);
    };
    bool ok = true;
    double s[L::NB][4];
#pragma unroll
    for (int b = 0; b < L::NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[b][r] = 0.0;
    __syncthreads();
    for (int j = 0; j < a.n; ++j) {
        stage(j);
        __syncthreads();
        if (!(ok = range(j))) break;
        // T_dv of this lane: rows k = 8 pk + e, column x = col, taps k - x
        const int t0 = 8 * pk - col + 16;
        const __bf16 *tp = taps + half * 6 * L::TP + (t0 & 1) * L::TP + (t0 & ~1);
        for (int dv = wv & 3; dv < L::K; dv += 4) {
            auto operand = [&](int q) {
                const uint32_t *w = (const uint32_t *)(tp + 2 * q * L::TP + dv * L::TL);
                const uint4 u = make_uint4(w[0], w[1], w[2], w[3]);
                return __builtin_bit_cast(bf16x8, u);
            };
            const bf16x8 th = operand(0), tm = operand(1), tl = operand(2);
            const __bf16 *td = tile + half * 3 * L::PL + (dv + col) * L::RS + 8 * pk;
#pragma unroll
            for (int b = 0; b < L::NB; b += 2) {
                const __bf16 *t = td + 16 * (b >> 2) * L::RS + 16 * (b & 3);
                const bf16x8 ah = *(const bf16x8 *)t, am = *(const bf16x8 *)(t + L::PL),
                             al = *(const bf16x8 *)(t + 2 * L::PL);
                const bf16x8 bh = *(const bf16x8 *)(t + 16), bm = *(const bf16x8 *)(t + L::PL + 16),
                             bl = *(const bf16x8 *)(t + 2 * L::PL + 16);
                floatx4 c = {0.f, 0.f, 0.f, 0.f}, d = {0.f, 0.f, 0.f, 0.f};
#define ARGUS_MM(X, Y, T)                                                      \
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(X, T, c, 0, 0, 0); \
                d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Y, T, d, 0, 0, 0);
                ARGUS_MM(al, bl, th)
                ARGUS_MM(ah, bh, tl)
                ARGUS_MM(am, bm, tm)
                ARGUS_MM(am, bm, th)
                ARGUS_MM(ah, bh, tm)
                ARGUS_MM(ah, bh, th)
#undef ARGUS_MM
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s[b][r] += (double)c[r];
                    s[b + 1][r] += (double)d[r];
                }
            }
        }
        __syncthreads();
    }
    // outputs of one pixel
    auto put = [&](int X, int Y, double S, double V) {
        if (X >= a.W || Y >= a.H) return;
        const int64_t o = (int64_t)Y * P + X;
        a.S[o] = (float)S;
        a.Var[o] = (float)V;
        if (a.snr) a.snr[o] = V > 0.0 ? (float)(S / sqrt(V)) : 0.f;
    };
    if (!ok) {
        double S4[4], V4[4];
        const int ly = tid >> 4, lx0 = 4 * (tid & 15);
        static_assert(L::TX == 64 && MLds<R, L::TX, L::TY, 4>::NT == L::NT, "four pixels a thread");
        static_assert(MLds<R, L::TX, L::TY, 4>::bytes <= L::bytes, "the FP32 tile fits the planes");
        matched_tile<R, L::TX, L::TY, 4>(a, (float *)xl, x0, y0, ly, lx0, S4, V4);
#pragma unroll
        for (int i = 0; i < 4; ++i) put(x0 + lx0 + i, y0 + ly, S4[i], V4[i]);
        return;
    }
    // the four waves' sums of each block, wave b adding block b's, first the
    // score's then the variance's
    double *sum = (double *)xl;                          // [wave][block][256]
    double tot[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (half == h)
#pragma unroll
            for (int b = 0; b < L::NB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) sum[(((wv & 3) * L::NB + b) * 4 + r) * 64 + lane] = s[b][r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            tot[h][r] = 0.0;
            for (int w = 0; w < 4; ++w) tot[h][r] += sum[((w * L::NB + wv) * 4 + r) * 64 + lane];
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        put(x0 + 16 * (wv & 3) + col, y0 + 16 * (wv >> 2) + 4 * pk + r, tot[0][r], tot[1][r]);
}

template <int R>
int matched_mfma_launch(argus_ctx *ctx, MatchedArgs a) {
    using L = XLds<R>;
    ARGUS_HIP_CHECK(ctx, hipFuncSetAttribute((const void *)matched_mfma_kernel<R>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)L::bytes));
    int vec = a.pitch % 4 == 0;
    for (int j = 0; j < a.n; ++j)
        vec = vec && (uintptr_t)a.cal[j] % 16 == 0 && (uintptr_t)a.var[j] % 16 == 0 &&
              (uintptr_t)a.mask[j] % 4 == 0;
    a.bx = (a.W + L::TX - 1) / L::TX;
    const int nblocks = a.bx * ((a.H + L::TY - 1) / L::TY);
    hipLaunchKernelGGL(matched_mfma_kernel<R>, dim3(nblocks), dim3(L::NT), L::bytes, ctx->stream, a, vec);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}

template <int R>
int matched_launch(argus_ctx *ctx, const MatchedArgs &a, int nblocks) {
    const size_t lds = MLds<R, BW, BH, PXT>::bytes;
    ARGUS_HIP_CHECK(ctx, hipFuncSetAttribute((const void *)matched_kernel<R>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(matched_kernel<R>, dim3(nblocks), dim3(NTHR), lds, ctx->stream, a);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}

}  // namespace

int launch_coadd_matched(argus_ctx *ctx, argus_dims d, int n, const float *const *cal,
                         const float *const *var, const uint8_t *const *mask,
                         const float *const *grids, int box, const float *psf, int r,
                         const float *scales, float *S, float *Var, float *snr) {
    MatchedArgs a{};
    for (int j = 0; j < n; ++j) {
        a.cal[j] = cal[j];
        a.var[j] = var[j];
        a.mask[j] = mask[j];
        a.F[j] = scales ? scales[j] : 1.f;
        a.bg[j] = (grids && grids[j]) ? make_bg_grid(grids[j], box, d.width, d.height) : BgGrid{};
    }
    a.psf = psf;
    a.S = S; a.Var = Var; a.snr = snr;
    a.pitch = d.pitch; a.W = d.width; a.H = d.height; a.n = n;
    a.bx = (d.width + BW - 1) / BW;
    const int nblocks = a.bx * ((d.height + BH - 1) / BH);
    // The matrix form (up to r = 8: an operand of 32 rows holds 16 + 2 r taps) pays
    // for its splits from r = 5 on, or where there are backgrounds, whose
    // interpolation its staging shares among columns, from r = 3 on and at r = 1
    // (3 PSF rows are one turn of its 4 waves, 5 are two).  4788x3194, 5 images,
    // FP32 / matrix form (us): no backgrounds r = 1 336 / 483, 2 406 / 648, 3 535 /
    // 648, 4 653 / 757, 5 980 / 847; with them r = 1 565 / 536, 2 654 / 709, 3 788 /
    // 696, 4 951 / 811.  500x333, 2 images: 4 29 / 27, 5 36 / 28; 3 with them 35 / 28.
    bool grid = false;
    for (int j = 0; j < n; ++j) grid = grid || a.bg[j].grid;
    const bool fp32 = !grid && r <= 4;
    argus_time_begin(ctx);
    int rc;
    switch (r) {
#define ARGUS_MF(RR) case RR: rc = matched_launch<RR>(ctx, a, nblocks); break;
#define ARGUS_MM(RR) case RR: rc = matched_mfma_launch<RR>(ctx, a); break;
#define ARGUS_ME(RR) case RR: rc = fp32 ? matched_launch<RR>(ctx, a, nblocks) : matched_mfma_launch<RR>(ctx, a); break;
        ARGUS_ME(1) ARGUS_MF(2) ARGUS_ME(3) ARGUS_ME(4) ARGUS_MM(5) ARGUS_MM(6) ARGUS_MM(7) ARGUS_MM(8)
        ARGUS_MF(9) ARGUS_MF(10)
#undef ARGUS_MF
#undef ARGUS_MM
#undef ARGUS_ME
        default: return argus_fail(ctx, ARGUS_ESHAPE, "psf_half %d not in 1..10", r);
    }
    if (rc) return rc;
    argus_time_end(ctx, "coadd_matched");
    return ARGUS_OK;
}
