// Fused basis convolution + normal-equation moment accumulation (shared by
// the per-precision translation units k_fit_fp32/fp64/bf16x3.hip; k_fit_wide.hip
// has the FP32 form of wide frames, fit_wide.h).
//
// Every entry of A = sum w X X^T is a moment G_ab[k][l] = sum_p w xt^a yt^b
// c_k c_l of the 32-vector c = (C_0..C_{nb-1}, 1, 0...) with a+b <= 2D, and
// b needs R_ab[k] = sum w xt^a yt^b c_k S with a+b <= D.  Along one image row
// yt is constant, so a workgroup accumulates the 2D+1 xt-moments of each row
// on MFMA (three 16x16 blocks of the symmetric 32x32 moment per power) and
// adds yt^b times them into FP64 running sums.
//
// Precisions of the per-row products and sums:
//   ARGUS_FP32   FP32 operands, v_mfma_f32_16x16x4f32 over 64 pixels (wide
//                frames, D >= 1: six BF16 products of three-way splits);
//   ARGUS_FP64   FP64 operands, v_mfma_f64_16x16x4f64 (FP64 products and sums);
//   ARGUS_BF16X3 x = hi + lo with hi, lo bf16 (round to nearest even), and
//                A B ~ Ahi Bhi + Ahi Blo + Alo Bhi on v_mfma_f32_16x16x32_bf16
//                with FP32 accumulation (Henry, Tang & Heinecke 2019).
#pragma once
#include <type_traits>

#include "internal.h"

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

namespace argus_fit {

constexpr int SW = 64;        // output columns per workgroup strip

// ---------------------------------------------------------------------------
struct FitArgs {
    const float *ref, *rvar, *sci, *svar;
    const uint8_t *rmask, *smask;
    const BasisTables *tab;
    double *partials;
    int64_t pitch;
    int W, H, h, nb, nplanes;
    int RX, RY;                // regions (1x1 for GLOBAL, tiles for PER_TILE)
    int spt, rchunks;          // strips per region, row chunks per region
    int stride;                // doubles per partial
    double sx, sy;             // 2/(W-1), 2/(H-1) (0 for a 1-pixel axis)
    int8_t plist[4][4];        // row-filter planes of each wave (-1: none)
    int8_t plist8[8][2];       // the same for 8 convolution waves
};

__device__ __forceinline__ int qidx(int a, int b, int Dm) {   // a+b <= Dm, a outer
    return a * (Dm + 1) - a * (a - 1) / 2 + b;
}

template <int D>
struct FitShape {
    static constexpr int NA = 2 * D + 1;                       // xt powers in the Gram
    static constexpr int NQ = (2 * D + 1) * (2 * D + 2) / 2;   // Gram moments
    static constexpr int NRA = D + 1;                          // xt powers in the rhs
    static constexpr int NR = (D + 1) * (D + 2) / 2;           // rhs moments
    static constexpr int NT = 3 * NA;                          // (a, block pair) tasks
};

// Per-wave MFMA work on one 64-pixel row: tasks t = WAVE, WAVE+4, ... with
// a = t / 3 and block pair bp = t % 3 in {(0,0), (0,1), (1,1)}.
template <int D, int WAVE, int PREC, int STR = 4>
struct WaveGram {
    // tasks t = WAVE, WAVE + STR, ... of the 3 (2D+1) (power, block pair) tasks
    static constexpr int NT = FitShape<D>::NT;
    static constexpr int NTW = (NT - WAVE + STR - 1) / STR;
    static constexpr int NB = 2 * D + 1;
    double F[NTW > 0 ? NTW : 1][NB][4];

    __device__ void zero() {
#pragma unroll
        for (int j = 0; j < (NTW > 0 ? NTW : 1); ++j)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) F[j][b][r] = 0.0;
    }

    template <typename V>
    __device__ void flush(const V (&acc)[NTW > 0 ? NTW : 1], const double *ypw) {
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            const int a = (WAVE + STR * j) / 3;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (b <= 2 * D - a) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) F[j][b][r] += ypw[b] * (double)acc[j][r];
                }
            }
        }
    }

    // One row on k-major operand tables (FP32, FP64): c[k][p] with row stride CKM
    // and w xt^a [a][p]; at step s the four lane groups pk take the pixels
    // p = 16 pk + s, so a lane's operands of consecutive steps are contiguous and
    // load 16 bytes at once.
    // c'_k = c_k + gam_k c_0 is applied to the operands as they are loaded.
    static constexpr int CKM = SW + 4;
    // Accumulator of one task: 4 FP32 (FP64 for ARGUS_FP64) values per lane.
    using Acc = typename std::conditional<PREC == ARGUS_FP64, doublex4, floatx4>::type;

    // The moments of one row into acc (not yet flushed into the FP64 sums).
    __device__ void row_km_acc(const float *cvec, const float *wx, const double *wxd, int lane,
                               float g0, float g1, Acc (&acc)[NTW > 0 ? NTW : 1]) {
        if constexpr (NTW > 0) {
            const int col = lane & 15, pk = lane >> 4;
            static_assert(PREC != ARGUS_BF16X3, "its rows come split (row_ts_acc)");
            using T = typename std::conditional<PREC == ARGUS_FP32, float, double>::type;
            using TV = typename std::conditional<PREC == ARGUS_FP32, floatx4, doublex4>::type;
            const float *pa = cvec + col * CKM + 16 * pk;
            const float *pb = cvec + (16 + col) * CKM + 16 * pk;
            const float *pz = cvec + 16 * pk;
#pragma unroll
            for (int j = 0; j < NTW; ++j) acc[j] = TV{0, 0, 0, 0};
            // the operands of 4 steps are loaded while the 4 steps before run
            float4 na, nb, nz;
            T nw[NTW][4];
            // (FP64: the weights are read in their own group, as two
            // groups of FP64 weights do not fit the register budget)
            auto load = [&](int u) {
                na = *(const float4 *)(pa + 4 * u);
                nb = *(const float4 *)(pb + 4 * u);
                nz = *(const float4 *)(pz + 4 * u);
                if constexpr (PREC == ARGUS_FP32) {
#pragma unroll
                    for (int j = 0; j < NTW; ++j) {
                        const int a = (WAVE + STR * j) / 3;
                        const float4 w = *(const float4 *)(wx + a * SW + 16 * pk + 4 * u);
                        nw[j][0] = w.x; nw[j][1] = w.y; nw[j][2] = w.z; nw[j][3] = w.w;
                    }
                }
            };
            load(0);
            // FP64: no unrolling across groups (its accumulators and FP64
            // sums leave no room for a second group's operands)
#pragma unroll (PREC == ARGUS_FP32 ? 4 : 1)
            for (int u = 0; u < 4; ++u) {
                const float ca[4] = {na.x, na.y, na.z, na.w};
                const float cb[4] = {nb.x, nb.y, nb.z, nb.w};
                const float cz[4] = {nz.x, nz.y, nz.z, nz.w};
                T w[NTW][4];
                if constexpr (PREC == ARGUS_FP32) {
#pragma unroll
                    for (int j = 0; j < NTW; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[j][e] = nw[j][e];
                } else {
#pragma unroll
                    for (int j = 0; j < NTW; ++j) {
                        const int a = (WAVE + STR * j) / 3;
                        const double2 w0 = *(const double2 *)(wxd + a * SW + 16 * pk + 4 * u);
                        const double2 w1 = *(const double2 *)(wxd + a * SW + 16 * pk + 4 * u + 2);
                        w[j][0] = w0.x; w[j][1] = w0.y; w[j][2] = w1.x; w[j][3] = w1.y;
                    }
                }
                if (u + 1 < 4) load(u + 1);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const T c0 = (T)ca[e] + (T)g0 * (T)cz[e];
                    const T c1 = (T)cb[e] + (T)g1 * (T)cz[e];
#pragma unroll
                    for (int j = 0; j < NTW; ++j) {
                        const int bp = (WAVE + STR * j) % 3;
                        const T A = (bp == 2) ? c1 : c0;
                        const T B = w[j][e] * ((bp == 0) ? c0 : c1);
                        if constexpr (PREC == ARGUS_FP32)
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(A, B, acc[j], 0, 0, 0);
                        else
                            acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(A, B, acc[j], 0, 0, 0);
                    }
                }
            }
        }
    }

    __device__ void row_km(const float *cvec, const float *wx, const double *wxd,
                           const double *ypw, int lane, float g0, float g1) {
        Acc acc[NTW > 0 ? NTW : 1];
        row_km_acc(cvec, wx, wxd, lane, g0, g1, acc);
        flush(acc, ypw);
    }

    // Output element of register r in this lane: column lane % 16; row
    // 4 (lane / 16) + r for the FP32 and BF16 instructions, 4 r + lane / 16 for
    // v_mfma_f64_16x16x4f64.
    __device__ void store(double *part, int lane) {
        if constexpr (NTW > 0) {
            const int col = lane & 15, lg = lane >> 4;
#pragma unroll
            for (int j = 0; j < NTW; ++j) {
                const int t = WAVE + STR * j;
                const int a = t / 3, bp = t % 3;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (b <= 2 * D - a) {
                        double *g = part + (size_t)qidx(a, b, 2 * D) * 768 + bp * 256;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int row = (PREC == ARGUS_FP64) ? 4 * r + lg : 4 * lg + r;
                            g[row * 16 + col] = F[j][b][r];
                        }
                    }
                }
            }
        }
    }
};

// Wave-uniform loads of the filter tables go through the scalar cache.
typedef const __attribute__((address_space(4))) float *cfloat_p;
__device__ __forceinline__ float uload(const float *p) { return *(cfloat_p)p; }

}  // namespace argus_fit

// One launcher per precision, each in its own translation unit.
int fit_accum_launch_fp32(argus_ctx *ctx, const argus_fit::FitArgs &fa, int D, dim3 grid);
// The FP32 fit of degree 1 or 2 on frames at least FIT_WIDE_MIN columns wide
// (fit_wide.h).  The line is not where the speed turns: the wide form is the
// faster one on both sides of it (degree 2, 15 x 15, FP32 form / wide form:
// 1100x977 154 / 132 us, 3000x2000 751 / 639, 6143x4100 2.85 / 2.42 ms, 9576x6388
// 7.04 / 5.94; degree 1: 134 / 110 us, 607 / 484, 2.27 / 1.69 ms, 5.58 / 4.13).  It
// keeps narrower frames' results to the bit; moving it changes them by the FP32
// rounding of either form.
int fit_accum_launch_wide(argus_ctx *ctx, const argus_fit::FitArgs &fa, int D, dim3 grid);
constexpr int FIT_WIDE_MIN = 6144;
int fit_accum_launch_fp64(argus_ctx *ctx, const argus_fit::FitArgs &fa, int D, dim3 grid);
int fit_accum_launch_bf16x3(argus_ctx *ctx, const argus_fit::FitArgs &fa, int D, dim3 grid);
