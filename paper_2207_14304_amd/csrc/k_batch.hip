// Batched cutouts: each cutout of each camera's frame pair gets its own
// spatially constant kernel fit, convolution, difference and detection map.
// A cutout is a standalone image of side L: edges and footprints stay inside
// it.  Four kernels, captured in a HIP graph:
//
//   fit       moments of one 64-column strip of up to CHUNK output rows (a
//             task), a persistent grid pulling tasks from a queue, largest
//             cutouts first;
//   solve     sums of a cutout's partials, FP64 Cholesky of the (nb+1)-unknown
//             system in the registers of one wave, the kernel stamp;
//   subtract  convolution, difference, variance and chi^2 of a tile;
//   detect    detection map of a tile, candidate counts, chi^2 totals.
//
// The split of a cutout into tasks and the order of every sum depend on the
// cutout alone, so it gives the same bits in any batch.  Fit and solve run in
// rounds of at most ROUND partials, which bounds the workspace.  The
// subtraction tile height and the fit's workgroups per CU are chosen by timing
// every candidate on the first run (autotuner).
//
// One workgroup per cutout for all four steps, the form before, took 22.0 ms
// for 1500 cutouts (93 Mpixel, 15x15, FP64 moments) at two waves per SIMD,
// with the 512-pixel cutouts alone setting the time of small batches; this
// form takes 6.6 ms (fit 4.6, subtract 1.6, detect 0.33, solve 0.05); 40 cutouts,
// 14.9 ms before, take 0.28.
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <new>
#include <vector>

#include "fit_accum.h"

namespace {

// A cutout as the kernels read it.
struct BCut {
    int32_t frame, x0, y0, side;
    int64_t out;               // element offset in the output arena
    int32_t task0, nstrip, nchunk;
    int32_t tile0[2];          // first tile of 16 and of 32 rows
    int32_t pad;
};

struct Round {
    int cut0, ncut, task0, ntask;
};

}  // namespace

struct argus_batch {
    int n = 0, n_frames = 0, n_unk = 0, h = 0, nb = 0, nplanes = 0;
    argus_kernel_spec spec{};
    int8_t plist[4][4];
    void *dev = nullptr;            // device: all tables and the workspace
    BasisTables *d_tables = nullptr;  // the batch's own copy: the context's tables
                                      // change with every other spec used on it
    BCut *d_cuts = nullptr;
    int32_t *d_order = nullptr, *d_task = nullptr;   // cutout of each rank, of each fit task
    int32_t *d_tile[2] = {nullptr, nullptr};         // cutout of each tile
    argus_frame *d_frames = nullptr;
    int32_t *d_queue = nullptr;     // one counter per round
    double *d_part = nullptr, *d_c2 = nullptr;       // moments per task, chi^2 per tile
    float *d_stamps = nullptr;
    int ntile[2] = {0, 0};
    std::vector<Round> rounds;
    std::vector<int32_t> widths, heights;
    hipStream_t stream = nullptr;   // private stream for the captured graph
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    // inputs baked into the captured graph
    std::vector<argus_frame> frames;
    const void *outs[9] = {};
    float thr = 0.f;
    int choice = -1, n_cand = 0;
    float tuned_ms = -1.f;
    std::vector<float> cand_ms;     // every candidate's time (ms), candidate order
    int from_cache = 0;             // the choice came from the context's tuning cache
    int64_t area = 0;               // sum of cutout areas (size bucket of the tuning key)
};

namespace {

using argus_fit::SW;

constexpr int CHUNK = 128;     // most output rows of a fit task: its 2h extra input rows are
                               // then about a tenth of its row filters, and 40 cutouts
                               // (150 tasks) still spread over the chip
constexpr int PST = 801;       // doubles of a partial: 3 blocks of 16x16, 32 rhs, fit pixels
constexpr int ROUND = 32768;   // partials of a round (210 MB)
constexpr int BW = 64;         // tile width of subtraction and detection
constexpr int DTILE = 32;      // detection tile rows

struct BatchArgs {
    const argus_frame *frames;
    const BCut *cuts;
    const int32_t *order, *task, *tile;
    int32_t *queue;
    const BasisTables *tab;
    double *part, *c2;
    float *stamps;
    int ntask, nb, n_unk, shape, tile0;    // tile0: first tile of a launch
    int8_t plist[4][4];
    float thr;
    float *diff, *dvar;
    uint8_t *dmask, *det;
    double *coeffs, *chi2;
    int64_t *n_fit;
    int32_t *status, *n_cands;
};

__host__ __device__ constexpr int stamp_stride(int h) {     // K^2 taps and the background
    return ((2 * h + 1) * (2 * h + 1) + 1 + 3) & ~3;
}

__device__ __forceinline__ double lane_value(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// ---- fit ---------------------------------------------------------------------
// Eight waves: 0-3 convolve (their planes are data), 4-7 take the moments of
// the rows convolved one step before, and between them stage what the next
// step needs (4, 5: fit-set weights of the step's two output rows; 6, 7: its
// two input rows).  One step is two rows and one barrier.  A convolution lane
// owns a column and keeps the last 2h+1 row-filtered values of its planes in
// registers, so the column pass reads no LDS; each filter coefficient is
// loaded (scalar) once for the two rows.
//
// FP64: a moment wave takes 16 of the row's 64 pixels for all three 16x16
// blocks and the right-hand side, so an operand is read from LDS and widened
// once for three products, and its sums stay in the MFMA accumulators for the
// whole task.  FP32: a wave takes one block over the row's 64 pixels, sums in
// FP32 in pixel order and adds the row to FP64; the fourth takes the
// right-hand side.
// The filters run tap by tap without pairing the symmetric taps: small
// cutouts' systems amplify FP32 rounding, so its order is kept.
// What bounds it: per 64 pixels a compute unit's four SIMDs issue 48 FP64 MFMA
// of 64 cycles and about 4600 cycles of VALU (2600 of them the filters' (planes
// + basis functions) (2h+1) FMAs); the two hardly overlap and fill 90% of the
// kernel's time.  Chunks of 96, 192 and 256 rows: 1.02, 0.98 and 0.97 of the
// time of 128 at 1500 cutouts, 1.14, 1.20 and 1.46 at 40.
template <int HH, int PREC>
struct FitLds {
    static constexpr int IN = SW + 2 * HH, INP = (IN + 3) & ~3, CKM = SW + 4;
    float c[2][2][32 * CKM];       // [step parity][row]: k-major basis convolutions
    float in[2][2][INP];           // input rows
    float w[2][2][SW];             // fit weights, and times the science pixel
    double ws[2][2][SW];
    uint64_t bits[2][2][2];        // flagged input pixels
    double rhs[4][32];
    int count[2];
};

// One filter's coefficients in scalar registers, loaded as a whole (rows of
// the tables are 128 bytes).
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
template <int K>
struct Taps {
    floatx16 a;
    floatx8 b;
    __device__ __forceinline__ void load(const float *p) {
        a = *(const __attribute__((address_space(4))) floatx16 *)p;
        if constexpr (K > 16) b = *(const __attribute__((address_space(4))) floatx8 *)(p + 16);
    }
    __device__ __forceinline__ float get(int i) const { return i < 16 ? a[i & 15] : b[i & 7]; }
};

template <int HH, int PREC>
__device__ void fit_conv(const BatchArgs &a, FitLds<HH, PREC> &l, int cw, int lane, int steps) {
    using L = FitLds<HH, PREC>;
    constexpr int K = 2 * HH + 1, NP = 4;
    int pl[NP], k0[NP], nk[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        pl[j] = __builtin_amdgcn_readfirstlane(a.plist[cw][j]);
        int f = 0, c = 0;
        if (pl[j] >= 0) {
            for (int k = 0; k < a.nb; ++k)
                if (a.tab->kpl[k] == pl[j]) {
                    if (c == 0) f = k;
                    ++c;
                }
        }
        k0[j] = __builtin_amdgcn_readfirstlane(f);
        nk[j] = __builtin_amdgcn_readfirstlane(c);
    }
    float rw[NP][K + 3];           // windows: sub-step u adds rows K-1+2u and K+2u
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int i = 0; i < K + 3; ++i) rw[j][i] = 0.f;
    auto step = [&](auto uc, int t) {
        constexpr int u = decltype(uc)::value;
        if (t < steps) {
            // (the tables' address is hidden from the loop, so their values
            // are read where they are used instead of being kept, and spilled,
            // across it; reading a filter ahead costs more moves than it hides)
            const BasisTables *tab = a.tab;
            asm volatile("" : "+s"(tab));
            {
                float w0[K], w1[K];
                const float *r0 = l.in[u][0] + lane, *r1 = l.in[u][1] + lane;
#pragma unroll
                for (int uu = 0; uu < K; ++uu) {
                    w0[uu] = r0[2 * HH - uu];
                    w1[uu] = r1[2 * HH - uu];
                }
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    if (pl[j] >= 0) {
                        Taps<K> f;
                        f.load(&tab->rowf[pl[j]][0]);
                        float a0 = 0.f, a1 = 0.f;
#pragma unroll
                        for (int uu = 0; uu < K; ++uu) {
                            a0 += f.get(uu) * w0[uu];
                            a1 += f.get(uu) * w1[uu];
                        }
                        rw[j][K - 1 + 2 * u] = a0;
                        rw[j][K + 2 * u] = a1;
                    }
                }
            }
            if (t >= HH) {
                float *c0 = l.c[u][0] + lane, *c1 = l.c[u][1] + lane;
#pragma unroll
                for (int j = 0; j < NP; ++j) {
#pragma unroll
                    for (int q = 0; q < 7; ++q) {
                        if (q < nk[j]) {
                            Taps<K> f;
                            f.load(&tab->colf[k0[j] + q][0]);
                            float a0 = 0.f, a1 = 0.f;
#pragma unroll
                            for (int jj = 0; jj < K; ++jj) {
                                a0 += f.get(2 * HH - jj) * rw[j][2 * u + jj];
                                a1 += f.get(2 * HH - jj) * rw[j][2 * u + 1 + jj];
                            }
                            c0[(k0[j] + q) * L::CKM] = a0;
                            c1[(k0[j] + q) * L::CKM] = a1;
                        }
                    }
                }
            }
        }
        __syncthreads();
    };
    for (int t = 0; t <= steps; t += 2) {
        step(std::integral_constant<int, 0>{}, t);
        step(std::integral_constant<int, 1>{}, t + 1);
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
            for (int i = 0; i < K - 1; ++i) rw[j][i] = rw[j][i + 4];
    }
}

// Moment wave m (0-3).  Rows [ry0, ry1) of the cutout, columns [sx0, sx1).
template <int HH, int PREC>
__device__ void fit_moments(const BatchArgs &a, FitLds<HH, PREC> &l, const argus_frame &fr,
                            int64_t org, int L, int sx0, int sx1, int ry0, int ry1, int m,
                            int lane, int steps) {
    using LT = FitLds<HH, PREC>;
    constexpr int CKM = LT::CKM, K = 2 * HH + 1;
    const int64_t P = fr.pitch;
    const int col = lane & 15, pk = lane >> 4;
    const int rows = ry1 - ry0, in_rows = rows + 2 * HH;
    const float g0 = col < a.nb ? a.tab->gam[col] : 0.f;
    const float g1 = 16 + col < a.nb ? a.tab->gam[16 + col] : 0.f;
    const float gk = (lane & 31) < a.nb ? a.tab->gam[lane & 31] : 0.f;
    // input row of the step after the staged one (waves 2, 3)
    float pr[2] = {0.f, 0.f};
    uint8_t pm[2] = {0, 0};
    const int X0 = sx0 - HH + lane, X1 = X0 + 64;
    const bool in0 = X0 < L, in1 = lane < 2 * HH && X1 < L;
    auto fetch_in = [&](int t) {
        const int i = 2 * t + (m & 1);
        const int Y = ry0 - HH + (i < in_rows ? i : in_rows - 1);
        const int64_t o = org + (int64_t)Y * P;
        const int xa = in0 ? X0 : L - 1, xb = in1 ? X1 : L - 1;
        pr[0] = gld(fr.ref + o + xa);
        pr[1] = gld(fr.ref + o + xb);
        pm[0] = gld(fr.ref_mask + o + xa);
        pm[1] = gld(fr.ref_mask + o + xb);
    };
    auto stage = [&](int t, int b) {
        const int i = 2 * t + (m & 1);
        const bool ok = i < in_rows;
        const uint64_t b0 = __ballot(ok && in0 && pm[0] != 0);
        const uint64_t b1 = __ballot(ok && in1 && pm[1] != 0);
        float *r = l.in[b][m & 1];
        r[lane] = ok && in0 ? pr[0] : 0.f;
        if (lane < 2 * HH) r[64 + lane] = ok && in1 ? pr[1] : 0.f;
        if (lane == 0) {
            l.bits[b][m & 1][0] = b0;
            l.bits[b][m & 1][1] = b1;
        }
    };
    // weight inputs of this wave's output row of the next step (waves 0, 1)
    float p_s = 0.f, p_sv = 0.f, p_rv = 0.f;
    uint8_t p_sm = 1;
    const bool lane_ok = sx0 + lane < sx1;
    const int64_t ow = org + (lane_ok ? sx0 + lane : sx0);
    auto fetch_w = [&](int t) {
        const int o = 2 * (t - HH) + (m & 1);
        const int64_t q = ow + (int64_t)(ry0 + (o < 0 ? 0 : o < rows ? o : rows - 1)) * P;
        p_s = gld(fr.sci + q);
        p_sv = gld(fr.sci_var + q);
        p_rv = gld(fr.ref_var + q);
        p_sm = gld(fr.sci_mask + q);
    };
    uint32_t hist = 0;                     // bit j: input row i-j has a flagged pixel in reach
    int count = 0;
    auto reach = [&](int b, int r) {
        const uint64_t b0 = l.bits[b][r][0], b1 = l.bits[b][r][1];
        const uint64_t lo = (b0 >> lane) | ((b1 << (63 - lane)) << 1);
        hist = (hist << 1) | ((lo & ((1ull << K) - 1ull)) != 0 ? 1u : 0u);
        return (hist & ((1u << K) - 1u)) != 0;
    };

    doublex4 F[3];
    double r0 = 0.0, r1 = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) F[j] = doublex4{0.0, 0.0, 0.0, 0.0};
    auto moments = [&](int pb) {
        if constexpr (PREC == ARGUS_FP64) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float *c = l.c[pb][r];
                const int p = 16 * m + 4 * pk;
                const float4 va = *(const float4 *)(c + col * CKM + p);
                const float4 vb = *(const float4 *)(c + (16 + col) * CKM + p);
                const float4 vz = *(const float4 *)(c + p);
                const float4 vw = *(const float4 *)(l.w[pb][r] + p);
                const double2 s0 = *(const double2 *)(l.ws[pb][r] + p);
                const double2 s1 = *(const double2 *)(l.ws[pb][r] + p + 2);
                const float ca[4] = {va.x, va.y, va.z, va.w}, cb[4] = {vb.x, vb.y, vb.z, vb.w};
                const float cz[4] = {vz.x, vz.y, vz.z, vz.w}, wv[4] = {vw.x, vw.y, vw.z, vw.w};
                const double sv[4] = {s0.x, s0.y, s1.x, s1.y};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double z = (double)cz[e], w = (double)wv[e];
                    const double c0 = (double)ca[e] + (double)g0 * z;
                    const double c1 = (double)cb[e] + (double)g1 * z;
                    const double b0 = w * c0, b1 = w * c1;
                    F[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(c0, b0, F[0], 0, 0, 0);
                    F[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(c0, b1, F[1], 0, 0, 0);
                    F[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(c1, b1, F[2], 0, 0, 0);
                    r0 += sv[e] * c0;
                    r1 += sv[e] * c1;
                }
            }
        } else if (m < 3) {
            floatx4 acc[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int s = 0; s < SW / 4; ++s) {
                const int p = 4 * s + pk;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const float *c = l.c[pb][r];
                    const float cz = c[p];
                    const float c0 = c[col * CKM + p] + g0 * cz;
                    const float c1 = c[(16 + col) * CKM + p] + g1 * cz;
                    const float A = m == 2 ? c1 : c0;
                    const float B = l.w[pb][r][p] * (m == 0 ? c0 : c1);
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(A, B, acc[r], 0, 0, 0);
                }
            }
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) F[0][e] += (double)acc[r][e];
        } else {
            // right-hand side: FP32 sums over 8 pixels, then FP64
            const int k = lane & 31, half = lane >> 5;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float *c = l.c[pb][r];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float s = 0.f;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int px = q * 16 + half * 8 + i;
                        const float v = c[k * CKM + px] + gk * c[px];
                        s += (float)l.ws[pb][r][px] * v;
                    }
                    r0 += (double)s;
                }
            }
        }
    };

    // (the inputs of step 0 are staged, those of step 1 are in registers)
    if (m >= 2) {
        fetch_in(0);
        stage(0, 0);
        fetch_in(1);
    } else {
        fetch_w(HH);
    }
    __syncthreads();
    const int last = (steps + 2) & ~1;
    for (int t = 0; t < last; ++t) {
        const int b = t & 1;
        if (m >= 2) {
            if (t + 1 < steps) stage(t + 1, b ^ 1);
            if (t + 2 < steps) fetch_in(t + 2);
        } else if (t < steps) {
            const float s = p_s, sv = p_sv, rv = p_rv;
            const uint8_t sm = p_sm;
            if (t >= HH && t + 1 < steps) fetch_w(t + 1);
            bool foot = reach(b, 0);
            if (m == 1) foot = reach(b, 1);
            if (t >= HH) {
                const bool ok = lane_ok && 2 * (t - HH) + m < rows;
                const float tot = sv + rv;
                float w = 0.f;
                if (ok && sm == 0 && !foot && tot > 0.f) {
                    w = 1.0f / tot;
                    ++count;
                }
                l.w[b][m][lane] = w;
                const float sc = ok ? s : 0.f;
                l.ws[b][m][lane] = PREC == ARGUS_FP64 ? (double)w * (double)sc : (double)(w * sc);
            }
            if (m == 0) reach(b, 1);
        }
        if (t - 1 >= HH && t - 1 < steps) moments(b ^ 1);
        __syncthreads();
    }
    // the task's sums, into the convolution tables' place
    double *red = (double *)&l.c[0][0][0];
    if constexpr (PREC == ARGUS_FP64) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[m * 768 + j * 256 + (4 * e + pk) * 16 + col] = F[j][e];
        r0 += __shfl_xor(r0, 16);
        r1 += __shfl_xor(r1, 16);
        r0 += __shfl_xor(r0, 32);
        r1 += __shfl_xor(r1, 32);
        if (lane < 16) {
            l.rhs[m][lane] = r0;
            l.rhs[m][16 + lane] = r1;
        }
    } else if (m < 3) {
#pragma unroll
        for (int e = 0; e < 4; ++e) red[m * 256 + (4 * pk + e) * 16 + col] = F[0][e];
    } else {
        r0 += __shfl_xor(r0, 32);
        if (lane < 32) l.rhs[0][lane] = r0;
    }
    if (m < 2) {
        for (int off = 32; off > 0; off >>= 1) count += __shfl_xor(count, off);
        if (lane == 0) l.count[m] = count;
    }
}

template <int HH, int PREC>
__global__ __launch_bounds__(512, HH <= 7 ? 4 : 2) void batch_fit_kernel(BatchArgs a) {
    using LT = FitLds<HH, PREC>;
    __shared__ __align__(16) LT l;
    __shared__ int s_item;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (;;) {
        if (tid == 0) s_item = atomicAdd(a.queue, 1);
        __syncthreads();
        const int it = s_item;
        if (it >= a.ntask) break;                   // every wave reaches this exit
        const BCut cu = a.cuts[a.task[it]];
        const argus_frame fr = a.frames[cu.frame];
        const int L = cu.side, j = it - cu.task0;
        const int64_t org = (int64_t)cu.y0 * fr.pitch + cu.x0;
        const int rows = L - 2 * HH, rh = (rows + cu.nchunk - 1) / cu.nchunk;
        const int sx0 = HH + (j % cu.nstrip) * SW, sx1 = min(sx0 + SW, L - HH);
        const int ry0 = HH + (j / cu.nstrip) * rh, ry1 = min(ry0 + rh, L - HH);
        // constant tail of c: 1 at index nb (background), zeros after
        for (int i = tid; i < 4 * 32 * LT::CKM; i += 512) {
            const int k = (i / LT::CKM) % 32;
            if (k >= a.nb) (&l.c[0][0][0])[i] = (k == a.nb) ? 1.f : 0.f;
        }
        const int steps = (ry1 - ry0 + 2 * HH + 1) / 2;
        if (wave < 4) {
            __syncthreads();
            fit_conv<HH, PREC>(a, l, wave, lane, steps);
        } else {
            fit_moments<HH, PREC>(a, l, fr, org, L, sx0, sx1, ry0, ry1, wave - 4, lane, steps);
        }
        __syncthreads();
        const double *red = (const double *)&l.c[0][0][0];
        double *part = a.part + (size_t)it * PST;
        for (int i = tid; i < 768; i += 512)
            part[i] = PREC == ARGUS_FP64
                          ? (red[i] + red[768 + i]) + (red[1536 + i] + red[2304 + i])
                          : red[i];
        if (tid < 32)
            part[768 + tid] = PREC == ARGUS_FP64 ? (l.rhs[0][tid] + l.rhs[1][tid]) +
                                                       (l.rhs[2][tid] + l.rhs[3][tid])
                                                 : l.rhs[0][tid];
        if (tid == 0) part[800] = (double)(l.count[0] + l.count[1]);
        __syncthreads();
    }
}

// ---- solve -------------------------------------------------------------------
// One workgroup per cutout: the sums of its partials in task order; then one
// wave factors the Jacobi-scaled matrix with row r in the registers of lane r
// (a pivot column is broadcast by lane reads, no LDS round trip), the
// right-hand side carried along; back substitution by columns from LDS; then
// all threads expand the stamp.  Latency-bound, 1500 systems at once.
template <int HH>
__global__ __launch_bounds__(256) void batch_solve_kernel(BatchArgs a) {
    constexpr int KK = (2 * HH + 1) * (2 * HH + 1);
    __shared__ double G[PST], Lt[32 * 33], xs[32], ds[32];
    __shared__ int s_status;
    const int tid = threadIdx.x;
    const int c = a.order[blockIdx.x];
    const BCut cu = a.cuts[c];
    const int nt = cu.nstrip * cu.nchunk, n = a.n_unk;
    const double *part = a.part + (size_t)cu.task0 * PST;
    for (int i = tid; i < PST; i += 256) {
        double s = 0.0;
#pragma unroll 4
        for (int p = 0; p < nt; ++p) s += part[(size_t)p * PST + i];
        G[i] = s;
    }
    __syncthreads();
    if (tid < 64) {
        const int r = tid;
        const double *R = G + 768;
        const double cnt = G[800];
        int st = cnt < (double)n ? ARGUS_ETOOFEW : ARGUS_OK;
        double d = 1.0, mx = 0.0;
        if (r < n) {
            const double dg = G[(r < 16 ? 0 : 512) + (r & 15) * 16 + (r & 15)];
            d = dg > 0.0 ? 1.0 / sqrt(dg) : 0.0;
            mx = dg * d * d;
        }
        if (r < 32) ds[r] = d;
        if (st == ARGUS_OK && __any(!(d > 0.0))) st = ARGUS_ESINGULAR;
        for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
        const double tol = (double)n * 0x1p-52 * mx;
        double x = 0.0;
        if (st == ARGUS_OK) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            double row[32];
#pragma unroll
            for (int k = 0; k < 32; ++k) {           // column k <= row r
                const int rr = r & 31, kk = k < rr ? k : rr;
                const double g = rr < 16 ? G[kk * 16 + rr]
                                 : kk < 16 ? G[256 + kk * 16 + (rr - 16)]
                                           : G[512 + (kk - 16) * 16 + (rr - 16)];
                row[k] = (rr < n && k < n) ? g * d * ds[k] : 0.0;
            }
            x = r < n ? R[r] * d : 0.0;
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                if (j < n && st == ARGUS_OK) {
                    const double piv = lane_value(row[j], j);
                    if (!(piv > tol)) {
                        st = ARGUS_ESINGULAR;
                    } else {
                        const double ljj = sqrt(piv);
                        const double lr = row[j] / ljj;
                        row[j] = r == j ? ljj : lr;
                        const double y = lane_value(x, j) / ljj;
                        x = r == j ? y : r > j ? x - lr * y : x;
#pragma unroll
                        for (int k = j + 1; k < 32; ++k) row[k] -= lr * lane_value(lr, k);
                    }
                }
            }
            if (r < 32) {
#pragma unroll
                for (int k = 0; k < 32; ++k) Lt[r * 33 + k] = row[k];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (st == ARGUS_OK) {
                const double rd = r < n ? 1.0 / Lt[r * 33 + r] : 0.0;
                for (int k = n - 1; k >= 0; --k) {
                    const double v = lane_value(x * rd, k);
                    if (r == k) x = v;
                    else if (r < k) x -= Lt[k * 33 + r] * v;
                }
                x *= d;
            }
        }
        if (r < n) {
            xs[r] = x;
            a.coeffs[(size_t)c * n + r] = st == ARGUS_OK ? x : __builtin_nan("");
        }
        if (r == 0) {
            s_status = st;
            a.status[c] = st;
            a.n_fit[c] = (int64_t)cnt;
            a.n_cands[c] = 0;                        // counted by the detection
        }
    }
    __syncthreads();
    const bool ok = s_status == ARGUS_OK;
    float *st = a.stamps + (size_t)c * stamp_stride(HH);
    for (int t = tid; t < KK; t += 256) {
        double acc = 0.0;
        if (ok)
            for (int k = 0; k < a.nb; ++k) acc += xs[k] * a.tab->b2d[k][t];
        st[t] = ok ? (float)acc : __builtin_nanf("");
    }
    if (tid == 0) st[KK] = ok ? (float)xs[a.nb] : __builtin_nanf("");
}

// ---- subtract ----------------------------------------------------------------
// Bits d..d+2h of hi:lo ORed into bit d, for every d < 64.
template <int HH>
__device__ __forceinline__ uint64_t dilate(uint64_t lo, uint64_t hi) {
    constexpr int K = 2 * HH + 1;
#pragma unroll
    for (int s = 1; s < K; s = 2 * s < K ? 2 * s : K) {
        const int sh = 2 * s < K ? s : K - s;        // widths 1, 2, 4, .. then K
        lo |= (lo >> sh) | (hi << (64 - sh));
        hi |= hi >> sh;
    }
    return lo;
}

// A 64 x TILE tile: reference and variance with an h-pixel halo in LDS, a
// thread convolves TILE/4 consecutive pixels of a row from registers (two FMA
// per tap and pixel, VALU-bound); the sums go through LDS so that the science
// planes are read and the outputs written a row of 64 at a time.
template <int HH, int TILE>
__global__ __launch_bounds__(256, 4) void batch_subtract_kernel(BatchArgs a) {
    constexpr int K = 2 * HH + 1, TH = TILE + 2 * HH, TWr = BW + 2 * HH, PXT = TILE / 4;
    // 16-byte rows whose neighbours lie 4 banks off the 8-float steps of a row
    constexpr int T4 = (TWr + 3) & ~3, TW = T4 % 8 == 0 ? T4 + 4 : T4;
    constexpr int OW = BW + 4;
    __shared__ __align__(16) float Rt[TH * TW], Vt[TH * TW], St[K][2 * K + 2];
    __shared__ uint64_t M[TH];                       // footprint along the row, per input row
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bid = a.tile0 + argus_xcd_block(blockIdx.x, gridDim.x);
    const int c = a.tile[bid];
    const BCut cu = a.cuts[c];
    const argus_frame fr = a.frames[cu.frame];
    const int L = cu.side, j = bid - cu.tile0[a.shape], ntx = (L + BW - 1) / BW;
    const int tx0 = (j % ntx) * BW, ty0 = (j / ntx) * TILE;
    const int64_t P = fr.pitch, org = (int64_t)cu.y0 * P + cu.x0;

    // halo: 8 elements per thread in flight at once (clamped addresses,
    // out-of-cutout zeros applied at the store)
    constexpr int NH = (TH * TWr + 255) / 256, NB8 = 8;
    for (int j0 = 0; j0 < NH; j0 += NB8) {
        float hr[NB8], hv[NB8];
#pragma unroll
        for (int e = 0; e < NB8; ++e) {
            const int i = tid + (j0 + e) * 256, ii = i < TH * TWr ? i : 0;
            const int cy = ii / TWr, cx = ii % TWr;
            int X = tx0 - HH + cx, Y = ty0 - HH + cy;
            X = X < 0 ? 0 : (X >= L ? L - 1 : X);
            Y = Y < 0 ? 0 : (Y >= L ? L - 1 : Y);
            const int64_t o = org + (int64_t)Y * P + X;
            hr[e] = gld(fr.ref + o);
            hv[e] = gld(fr.ref_var + o);
        }
#pragma unroll
        for (int e = 0; e < NB8; ++e) {
            const int i = tid + (j0 + e) * 256;
            if (i < TH * TWr) {
                const int cy = i / TWr, cx = i % TWr;
                const int X = tx0 - HH + cx, Y = ty0 - HH + cy;
                const bool in = X >= 0 && X < L && Y >= 0 && Y < L;
                Rt[cy * TW + cx] = in ? hr[e] : 0.f;
                Vt[cy * TW + cx] = in ? hv[e] : 0.f;
            }
        }
    }
    // flagged reference pixels: a ballot per input row
    {
        const int Xa = tx0 - HH + lane, Xb = Xa + 64;
        const bool ia = Xa >= 0 && Xa < L, ib = lane < 2 * HH && Xb < L;
        const int xa = ia ? Xa : 0, xb = ib ? Xb : 0;
        constexpr int NM = (TH + 3) / 4;
        uint8_t ma[NM], mb[NM];
#pragma unroll
        for (int e = 0; e < NM; ++e) {
            const int Y = ty0 - HH + wave + 4 * e;
            const int64_t o = org + (int64_t)(Y >= 0 && Y < L ? Y : 0) * P;
            ma[e] = gld(fr.ref_mask + o + xa);
            mb[e] = gld(fr.ref_mask + o + xb);
        }
#pragma unroll
        for (int e = 0; e < NM; ++e) {
            const int cy = wave + 4 * e, Y = ty0 - HH + cy;
            const bool iy = Y >= 0 && Y < L;
            const uint64_t lo = __ballot(iy && ia && ma[e] != 0), hi = __ballot(iy && ib && mb[e] != 0);
            if (lane == 0 && cy < TH) M[cy] = dilate<HH>(lo, hi);
        }
    }
    const float *stp = a.stamps + (size_t)c * stamp_stride(HH);
    for (int t = tid; t < K * K; t += 256) {
        const float k = stp[t];
        St[t / K][2 * (t % K)] = k;
        St[t / K][2 * (t % K) + 1] = k * k;
    }
    const float bg = stp[K * K];
    __syncthreads();

    float m[PXT], v[PXT];
    {
        const int ly = tid / (BW / PXT), lx0 = (tid % (BW / PXT)) * PXT;
#pragma unroll
        for (int i = 0; i < PXT; ++i) { m[i] = 0.f; v[i] = 0.f; }
        for (int vv = 0; vv < K; ++vv) {
            constexpr int NW4 = (PXT + 2 * HH + 3) / 4;
            const float4 *rr = (const float4 *)(Rt + (ly + 2 * HH - vv) * TW + lx0);
            const float4 *qq = (const float4 *)(Vt + (ly + 2 * HH - vv) * TW + lx0);
            float r[4 * NW4], q[4 * NW4];
#pragma unroll
            for (int e = 0; e < NW4; ++e) {
                const float4 a4 = rr[e], b4 = qq[e];
                r[4 * e] = a4.x; r[4 * e + 1] = a4.y; r[4 * e + 2] = a4.z; r[4 * e + 3] = a4.w;
                q[4 * e] = b4.x; q[4 * e + 1] = b4.y; q[4 * e + 2] = b4.z; q[4 * e + 3] = b4.w;
            }
            const float4 *sp = (const float4 *)&St[vv][0];
#pragma unroll
            for (int u2 = 0; u2 <= HH; ++u2) {
                const float4 s4 = sp[u2];            // taps 2 u2 and 2 u2 + 1: k, k^2
#pragma unroll
                for (int i = 0; i < PXT; ++i) {
                    m[i] += s4.x * r[i + 2 * HH - 2 * u2];
                    v[i] += s4.y * q[i + 2 * HH - 2 * u2];
                }
                if (2 * u2 + 1 < K) {
#pragma unroll
                    for (int i = 0; i < PXT; ++i) {
                        m[i] += s4.z * r[i + 2 * HH - 2 * u2 - 1];
                        v[i] += s4.w * q[i + 2 * HH - 2 * u2 - 1];
                    }
                }
            }
        }
    }
    __syncthreads();
    {
        const int ly = tid / (BW / PXT), lx0 = (tid % (BW / PXT)) * PXT;
#pragma unroll
        for (int i = 0; i < PXT; i += 4) {
            *(float4 *)(Rt + ly * OW + lx0 + i) = float4{m[i], m[i + 1], m[i + 2], m[i + 3]};
            *(float4 *)(Vt + ly * OW + lx0 + i) = float4{v[i], v[i + 1], v[i + 2], v[i + 3]};
        }
    }
    // lane = column, TILE/4 consecutive rows per wave
    constexpr int RW = TILE / 4;
    const int X = tx0 + lane;
    const int xc = X < L ? X : L - 1;
    float s[RW], sv[RW], rv[RW];
    uint8_t sm[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int Y = ty0 + wave * RW + i;
        const int64_t o = org + (int64_t)(Y < L ? Y : L - 1) * P + xc;
        s[i] = gld(fr.sci + o);
        sv[i] = gld(fr.sci_var + o);
        rv[i] = gld(fr.ref_var + o);
        sm[i] = gld(fr.sci_mask + o);
    }
    __syncthreads();
    double c2 = 0.0;
    float *dout = a.diff + cu.out, *vout = a.dvar + cu.out;
    uint8_t *mout = a.dmask + cu.out;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int ly = wave * RW + i, Y = ty0 + ly;
        uint64_t f = 0;
#pragma unroll
        for (int vv = 0; vv < K; ++vv) f |= M[ly + vv];
        if (X < L && Y < L) {
            const bool edge = X < HH || X > L - 1 - HH || Y < HH || Y > L - 1 - HH;
            const bool foot = (f >> lane) & 1ull;
            const uint8_t dm = sm[i] | (edge ? ARGUS_EDGE : 0u) |
                               ((!edge && foot) ? ARGUS_FOOT : 0u);
            float dval = 0.f, vval = 0.f;
            if (dm == 0) {
                dval = s[i] - (float)((double)Rt[ly * OW + lane] + (double)bg);
                vval = sv[i] + Vt[ly * OW + lane];
                const float tot = sv[i] + rv[i];
                if (tot > 0.f) c2 += (double)dval * (double)dval / (double)tot;
            }
            const int64_t oo = (int64_t)Y * L + X;
            dout[oo] = dval;
            vout[oo] = vval;
            mout[oo] = dm;
        }
    }
    for (int off = 32; off > 0; off >>= 1) c2 += __shfl_xor(c2, off);
    if (lane == 0) red[wave] = c2;
    __syncthreads();
    if (tid == 0) a.c2[bid] = red[0] + red[1] + red[2] + red[3];
}

// ---- detect ------------------------------------------------------------------
// A 64 x 32 tile of the detection map: S/N with a one-pixel halo in LDS
// (off-cutout neighbours are -inf), a lane per column over 8 rows.  The first
// tile of a cutout also sums its chi^2.  Memory-bound.
__global__ __launch_bounds__(256) void batch_detect_kernel(BatchArgs a, const int32_t *tiles) {
    constexpr int SWD = BW + 2, TH = DTILE + 2, NE = (SWD * TH + 255) / 256, RW = DTILE / 4;
    __shared__ float s[TH][SWD + 2];
    __shared__ int cnt[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bid = a.tile0 + argus_xcd_block(blockIdx.x, gridDim.x);
    const int c = tiles[bid];
    const BCut cu = a.cuts[c];
    const int L = cu.side, j = bid - cu.tile0[1], ntx = (L + BW - 1) / BW;
    const int tx0 = (j % ntx) * BW, ty0 = (j / ntx) * DTILE;
    const float *dout = a.diff + cu.out, *vout = a.dvar + cu.out;
    const uint8_t *mout = a.dmask + cu.out;
    float d[NE], v[NE];
    uint8_t m[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int i = tid + e * 256, ii = i < SWD * TH ? i : 0;
        int X = tx0 - 1 + ii % SWD, Y = ty0 - 1 + ii / SWD;
        X = X < 0 ? 0 : (X >= L ? L - 1 : X);
        Y = Y < 0 ? 0 : (Y >= L ? L - 1 : Y);
        const int64_t o = (int64_t)Y * L + X;
        d[e] = dout[o];
        v[e] = vout[o];
        m[e] = mout[o];
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int i = tid + e * 256;
        if (i < SWD * TH) {
            const int X = tx0 - 1 + i % SWD, Y = ty0 - 1 + i / SWD;
            float sn = -__builtin_inff();
            if (X >= 0 && X < L && Y >= 0 && Y < L)
                sn = (m[e] != 0 || !(v[e] > 0.f)) ? 0.f : d[e] * __builtin_amdgcn_rsqf(v[e]);
            s[i / SWD][i % SWD] = sn;
        }
    }
    __syncthreads();
    const int X = tx0 + lane, r0 = wave * RW;
    int n = 0;
    float w[3][3];                                   // rows above, at and below the pixel
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        w[1][k] = s[r0][lane + k];
        w[2][k] = s[r0 + 1][lane + k];
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            w[0][k] = w[1][k];
            w[1][k] = w[2][k];
            w[2][k] = s[r0 + i + 2][lane + k];
        }
        const int Y = ty0 + r0 + i;
        const float cv = w[1][1];
        const bool det = cv >= a.thr;
        bool cand = det && cv > w[0][0] && cv > w[0][1] && cv > w[0][2] && cv > w[1][0];
        cand = cand && cv >= w[1][2] && cv >= w[2][0] && cv >= w[2][1] && cv >= w[2][2];
        const bool in = X < L && Y < L;
        if (in)
            a.det[cu.out + (int64_t)Y * L + X] = (det ? ARGUS_DET : 0u) | (cand ? ARGUS_CAND : 0u);
        n += __popcll(__ballot(in && cand));
    }
    if (lane == 0) cnt[wave] = n;
    __syncthreads();
    if (tid == 0) {
        const int t = cnt[0] + cnt[1] + cnt[2] + cnt[3];
        if (t) atomicAdd(a.n_cands + c, t);
    }
    if (j == 0 && wave == 0) {
        const int rows = a.shape == 0 ? 16 : 32, nt = ntx * ((L + rows - 1) / rows);
        const double *p = a.c2 + cu.tile0[a.shape];
        double t = 0.0;
        for (int i = lane; i < nt; i += 64) t += p[i];
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
        if (lane == 0) a.chi2[c] = t;
    }
}

__global__ void queue_reset_kernel(int32_t *q, int n) {
    for (int i = threadIdx.x; i < n; i += 256) q[i] = 0;
}

// candidates: subtraction tile height x fit workgroups per CU
constexpr int N_CAND = 6;
constexpr int CAND_TILE[N_CAND] = {16, 16, 16, 32, 32, 32};
constexpr int CAND_WPC[N_CAND] = {1, 2, 3, 1, 2, 3};

template <int HH>
int batch_launch_t(argus_ctx *ctx, const argus_batch *b, BatchArgs ba, int tile, int wg_per_cu,
                   hipStream_t st) {
    int cus = 0;
    ARGUS_HIP_CHECK(ctx, hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    const int nr = (int)b->rounds.size();
    hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(256), 0, st, b->d_queue, nr);
    for (int r = 0; r < nr; ++r) {
        const Round &rd = b->rounds[r];
        ba.queue = b->d_queue + r;
        ba.ntask = rd.ntask;
        ba.task = b->d_task + rd.task0;
        ba.order = b->d_order + rd.cut0;
        const dim3 grid(std::max(1, std::min(cus * wg_per_cu, rd.ntask)));
        if (b->spec.precision == ARGUS_FP64)
            hipLaunchKernelGGL((batch_fit_kernel<HH, ARGUS_FP64>), grid, dim3(512), 0, st, ba);
        else
            hipLaunchKernelGGL((batch_fit_kernel<HH, ARGUS_FP32>), grid, dim3(512), 0, st, ba);
        hipLaunchKernelGGL((batch_solve_kernel<HH>), dim3(rd.ncut), dim3(256), 0, st, ba);
    }
    ba.shape = tile == 16 ? 0 : 1;
    ba.tile = b->d_tile[ba.shape];
    // (a launch holds less than 2^32 threads)
    constexpr int MOST = 1 << 23;
    for (int64_t t = 0; t < b->ntile[ba.shape]; t += MOST) {
        ba.tile0 = (int)t;
        const dim3 tiles((unsigned)std::min<int64_t>(MOST, b->ntile[ba.shape] - t));
        if (tile == 16)
            hipLaunchKernelGGL((batch_subtract_kernel<HH, 16>), tiles, dim3(256), 0, st, ba);
        else
            hipLaunchKernelGGL((batch_subtract_kernel<HH, 32>), tiles, dim3(256), 0, st, ba);
    }
    for (int64_t t = 0; t < b->ntile[1]; t += MOST) {
        ba.tile0 = (int)t;
        const dim3 tiles((unsigned)std::min<int64_t>(MOST, b->ntile[1] - t));
        hipLaunchKernelGGL(batch_detect_kernel, tiles, dim3(256), 0, st, ba, b->d_tile[1]);
    }
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}

int batch_launch(argus_ctx *ctx, const argus_batch *b, const BatchArgs &ba, int cand, hipStream_t st) {
    const int tile = CAND_TILE[cand], wpc = CAND_WPC[cand];
#define ARGUS_BH(HH) case HH: return batch_launch_t<HH>(ctx, b, ba, tile, wpc, st);
    switch (b->h) {
        ARGUS_BH(4) ARGUS_BH(5) ARGUS_BH(6) ARGUS_BH(7) ARGUS_BH(8) ARGUS_BH(9) ARGUS_BH(10)
        default: return argus_fail(ctx, ARGUS_ESHAPE, "batch half width %d not in 4..10", b->h);
    }
#undef ARGUS_BH
}

inline int ilog2(int64_t v) {
    int r = 0;
    while (v > 1) { v >>= 1; ++r; }
    return r;
}

}  // namespace

namespace {

// (throws std::bad_alloc when host memory runs out)
int batch_plan(argus_ctx *ctx, const argus_kernel_spec *spec, const argus_cutout *cutouts,
               int n_cutouts, const int32_t *frame_widths, const int32_t *frame_heights,
               int n_frames, argus_batch **out) {
    int nu, ns;
    int rc = argus_kernel_dims(spec, &nu, &ns);
    if (rc) return argus_fail(ctx, rc, "argus_batch_plan: bad kernel spec");
    if (spec->spatial_degree != 0 || spec->mode != ARGUS_FIT_GLOBAL ||
        (spec->precision != ARGUS_FP32 && spec->precision != ARGUS_FP64))
        return argus_fail(ctx, ARGUS_ESHAPE, "batch fits use degree 0, GLOBAL, FP32 or FP64");
    if (spec->half_width < 4 || spec->half_width > 10)
        return argus_fail(ctx, ARGUS_ESHAPE, "batch half width %d not in 4..10", spec->half_width);
    if (n_cutouts < 1 || !cutouts || n_frames < 1 || !frame_widths || !frame_heights)
        return argus_fail(ctx, ARGUS_EINVAL, "argus_batch_plan: empty or null tables");
    const int h = spec->half_width;
    for (int i = 0; i < n_cutouts; ++i) {
        const argus_cutout &c = cutouts[i];
        if (c.frame < 0 || c.frame >= n_frames)
            return argus_fail(ctx, ARGUS_EINVAL, "cutout %d: frame %d out of range", i, c.frame);
        if (c.side < 2 * h + 2 || c.side > 512)
            return argus_fail(ctx, ARGUS_ESHAPE, "cutout %d: side %d not in %d..512", i, c.side, 2 * h + 2);
        if (c.x0 < 0 || c.y0 < 0 || c.x0 + c.side > frame_widths[c.frame] ||
            c.y0 + c.side > frame_heights[c.frame])
            return argus_fail(ctx, ARGUS_ESHAPE, "cutout %d leaves its frame", i);
        if (c.out_offset < 0) return argus_fail(ctx, ARGUS_EINVAL, "cutout %d: negative offset", i);
    }
    std::unique_ptr<argus_batch, void (*)(argus_batch *)> hold(new argus_batch(), argus_batch_destroy);
    argus_batch *b = hold.get();
    for (int i = 0; i < n_cutouts; ++i) b->area += (int64_t)cutouts[i].side * cutouts[i].side;
    b->n = n_cutouts;
    b->n_frames = n_frames;
    b->n_unk = nu;
    b->h = h;
    b->spec = *spec;
    b->nb = argus_nbasis(spec);
    b->nplanes = argus_nplanes(spec);
    b->widths.assign(frame_widths, frame_widths + n_frames);
    b->heights.assign(frame_heights, frame_heights + n_frames);
    // planes to waves (same balancing as the frame fit)
    {
        int cost[ARGUS_MAX_PLANES], load[4] = {0, 0, 0, 0}, nin[4] = {0, 0, 0, 0};
        int p = 0;
        for (int g = 0; g < spec->n_gauss; ++g)
            for (int i = 0; i <= spec->degree[g]; ++i, ++p) cost[p] = 2 + spec->degree[g] - i;
        for (int w = 0; w < 4; ++w)
            for (int j = 0; j < 4; ++j) b->plist[w][j] = -1;
        bool used[ARGUS_MAX_PLANES] = {};
        for (int k = 0; k < b->nplanes; ++k) {
            int best = -1;
            for (int q = 0; q < b->nplanes; ++q)
                if (!used[q] && (best < 0 || cost[q] > cost[best])) best = q;
            int w = -1;
            for (int c = 0; c < 4; ++c)
                if (nin[c] < 4 && (w < 0 || load[c] < load[w])) w = c;
            used[best] = true;
            b->plist[w][nin[w]++] = (int8_t)best;
            load[w] += cost[best];
        }
    }
    // largest cutouts first; ties by index (deterministic)
    std::vector<int32_t> order(n_cutouts);
    for (int i = 0; i < n_cutouts; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int c) { return cutouts[a].side > cutouts[c].side; });
    // tasks, tiles and rounds
    std::vector<BCut> cuts(n_cutouts);
    std::vector<int32_t> task, tile[2];
    int part_max = 0;
    Round rd{0, 0, 0, 0};
    for (int i = 0; i < n_cutouts; ++i) {
        const int c = order[i];
        const argus_cutout &q = cutouts[c];
        BCut &cu = cuts[c];
        cu = BCut{q.frame, q.x0, q.y0, q.side, q.out_offset};
        const int rows = q.side - 2 * h;
        cu.nstrip = (rows + SW - 1) / SW;
        cu.nchunk = (rows + CHUNK - 1) / CHUNK;
        // (at most 32 tasks each, so a round always takes at least one cutout)
        const int nt = cu.nstrip * cu.nchunk;
        if (rd.ntask + nt > ROUND) {
            b->rounds.push_back(rd);
            rd = Round{i, 0, (int)task.size(), 0};
        }
        cu.task0 = rd.ntask;
        rd.ntask += nt;
        ++rd.ncut;
        part_max = std::max(part_max, rd.ntask);
        task.insert(task.end(), nt, c);
        for (int s = 0; s < 2; ++s) {
            const int th = s ? 32 : 16;
            const size_t k = (size_t)((q.side + BW - 1) / BW) * ((q.side + th - 1) / th);
            if (tile[s].size() + k > (size_t)INT32_MAX)
                return argus_fail(ctx, ARGUS_ESHAPE, "batch of more than 2^31 tiles");
            cu.tile0[s] = (int32_t)tile[s].size();
            tile[s].insert(tile[s].end(), k, c);
        }
    }
    b->rounds.push_back(rd);
    b->ntile[0] = (int)tile[0].size();
    b->ntile[1] = (int)tile[1].size();
    size_t bytes = 0;
    auto place = [&](size_t n) {
        const size_t o = bytes;
        bytes = (bytes + n + 255) & ~(size_t)255;
        return o;
    };
    const size_t off_c = place(cuts.size() * sizeof(BCut)), off_o = place(order.size() * 4),
                 off_k = place(task.size() * 4), off_t0 = place(tile[0].size() * 4),
                 off_t1 = place(tile[1].size() * 4),
                 off_f = place((size_t)n_frames * sizeof(argus_frame)),
                 off_q = place(b->rounds.size() * 4), off_b = place(sizeof(BasisTables)),
                 off_p = place((size_t)part_max * PST * 8), off_s = place(tile[0].size() * 8),
                 off_st = place((size_t)n_cutouts * stamp_stride(h) * 4);
    if (hipMalloc(&b->dev, bytes) != hipSuccess) {
        (void)hipGetLastError();               // (else the next launch's check would report it)
        return argus_fail(ctx, ARGUS_ENOMEM, "batch tables");
    }
    char *dev = (char *)b->dev;
    b->d_cuts = (BCut *)(dev + off_c);
    b->d_order = (int32_t *)(dev + off_o);
    b->d_task = (int32_t *)(dev + off_k);
    b->d_tile[0] = (int32_t *)(dev + off_t0);
    b->d_tile[1] = (int32_t *)(dev + off_t1);
    b->d_frames = (argus_frame *)(dev + off_f);
    b->d_queue = (int32_t *)(dev + off_q);
    b->d_tables = (BasisTables *)(dev + off_b);
    b->d_part = (double *)(dev + off_p);
    b->d_c2 = (double *)(dev + off_s);
    b->d_stamps = (float *)(dev + off_st);
    if (hipMemcpy(b->d_cuts, cuts.data(), cuts.size() * sizeof(BCut), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(b->d_order, order.data(), order.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(b->d_task, task.data(), task.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(b->d_tile[0], tile[0].data(), tile[0].size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(b->d_tile[1], tile[1].data(), tile[1].size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&b->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&b->ev_out, hipEventDisableTiming) != hipSuccess)
        return argus_fail(ctx, ARGUS_EHIP, "batch setup failed");
    if ((rc = launch_basis_tables_to(ctx, spec, b->d_tables))) return rc;
    // the basis tables must be complete before the private stream reads them
    if (hipStreamSynchronize(ctx->stream) != hipSuccess)
        return argus_fail(ctx, ARGUS_EHIP, "batch setup sync failed");
    *out = hold.release();
    return ARGUS_OK;
}

}  // namespace

extern "C" {

int argus_batch_plan(argus_ctx *ctx, const argus_kernel_spec *spec, const argus_cutout *cutouts,
                     int n_cutouts, const int32_t *frame_widths, const int32_t *frame_heights,
                     int n_frames, argus_batch **out) {
    if (!ctx || !out) return ARGUS_EINVAL;
    ctx->err.clear();
    *out = nullptr;
    try {
        return batch_plan(ctx, spec, cutouts, n_cutouts, frame_widths, frame_heights, n_frames, out);
    } catch (const std::bad_alloc &) {
        return argus_fail(ctx, ARGUS_ENOMEM, "batch tables of %d cutouts: out of host memory", n_cutouts);
    }
}

int argus_batch_run(argus_ctx *ctx, argus_batch *b, const argus_frame *frames, float threshold,
                    float *diff, float *diff_var, uint8_t *diff_mask, uint8_t *det_mask,
                    double *coeffs, double *chi2, int64_t *n_fit, int32_t *status,
                    int32_t *n_cands) {
    if (!ctx || !b || !frames) return ARGUS_EINVAL;
    ctx->err.clear();
    if (!diff || !diff_var || !diff_mask || !det_mask || !coeffs || !chi2 || !n_fit || !status ||
        !n_cands)
        return argus_fail(ctx, ARGUS_EINVAL, "argus_batch_run: null output");
    for (int f = 0; f < b->n_frames; ++f) {
        const argus_frame &fr = frames[f];
        if (!fr.ref || !fr.ref_var || !fr.ref_mask || !fr.sci || !fr.sci_var || !fr.sci_mask)
            return argus_fail(ctx, ARGUS_EINVAL, "frame %d: null plane", f);
        if (fr.width != b->widths[f] || fr.height != b->heights[f] || fr.pitch < fr.width)
            return argus_fail(ctx, ARGUS_ESHAPE, "frame %d does not match the plan", f);
    }
    const void *outs[9] = {diff, diff_var, diff_mask, det_mask, coeffs, chi2, n_fit, status, n_cands};
    bool same = b->exec && b->thr == threshold && (int)b->frames.size() == b->n_frames;
    for (int i = 0; same && i < 9; ++i) same = b->outs[i] == outs[i];
    for (int f = 0; same && f < b->n_frames; ++f)
        same = memcmp(&b->frames[f], &frames[f], sizeof(argus_frame)) == 0;
    // order the private stream after the caller's stream
    ARGUS_HIP_CHECK(ctx, hipEventRecord(b->ev_in, ctx->stream));
    ARGUS_HIP_CHECK(ctx, hipStreamWaitEvent(b->stream, b->ev_in, 0));
    if (!same) {
        ARGUS_HIP_CHECK(ctx, hipMemcpyAsync(b->d_frames, frames, (size_t)b->n_frames * sizeof(argus_frame),
                                            hipMemcpyHostToDevice, b->stream));
        ARGUS_HIP_CHECK(ctx, hipStreamSynchronize(b->stream));
        BatchArgs ba{};
        ba.frames = b->d_frames; ba.cuts = b->d_cuts; ba.tab = b->d_tables;
        ba.part = b->d_part; ba.c2 = b->d_c2; ba.stamps = b->d_stamps;
        ba.nb = b->nb; ba.n_unk = b->n_unk;
        memcpy(ba.plist, b->plist, sizeof ba.plist);
        ba.thr = threshold;
        ba.diff = diff; ba.dvar = diff_var; ba.dmask = diff_mask; ba.det = det_mask;
        ba.coeffs = coeffs; ba.chi2 = chi2; ba.n_fit = n_fit; ba.status = status; ba.n_cands = n_cands;
        if (b->choice < 0) {
            // autotune: the context's cache (device, HIP runtime, kernel, half
            // width, precision, size bucket, and the form of the kernels: times of
            // another form say nothing here), else time each candidate once on
            // these inputs and store the outcome
            char kb[160];
            snprintf(kb, sizeof kb, ";kernel=batch;h=%d;prec=%d;log2n=%d;log2area=%d;form=tasks", b->h,
                     b->spec.precision, ilog2(b->n), ilog2(b->area));
            const std::string key = argus_tune_device_key(ctx) + kb;
            const argus_ctx::Tuned *t = argus_tune_lookup(ctx, key);
            if (t && (int)t->ms.size() == N_CAND) {
                b->choice = t->choice;
                b->cand_ms = t->ms;
                b->from_cache = 1;
            } else {
                hipEvent_t e0, e1;
                ARGUS_HIP_CHECK(ctx, hipEventCreate(&e0));
                ARGUS_HIP_CHECK(ctx, hipEventCreate(&e1));
                float best = 1e30f;
                b->cand_ms.assign(N_CAND, 0.f);
                for (int cand = 0; cand < N_CAND; ++cand) {
                    ARGUS_HIP_CHECK(ctx, hipEventRecord(e0, b->stream));
                    int rc = batch_launch(ctx, b, ba, cand, b->stream);
                    if (rc) return rc;
                    ARGUS_HIP_CHECK(ctx, hipEventRecord(e1, b->stream));
                    ARGUS_HIP_CHECK(ctx, hipEventSynchronize(e1));
                    float ms = 0.f;
                    ARGUS_HIP_CHECK(ctx, hipEventElapsedTime(&ms, e0, e1));
                    b->cand_ms[cand] = ms;
                    if (ms < best) { best = ms; b->choice = cand; }
                }
                (void)hipEventDestroy(e0);
                (void)hipEventDestroy(e1);
                argus_tune_store(ctx, key, b->choice, b->cand_ms);
                b->from_cache = 0;
            }
            b->tuned_ms = b->cand_ms[b->choice];
            b->n_cand = N_CAND;
        }
        if (b->exec) { (void)hipGraphExecDestroy(b->exec); b->exec = nullptr; }
        if (b->graph) { (void)hipGraphDestroy(b->graph); b->graph = nullptr; }
        ARGUS_HIP_CHECK(ctx, hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
        int rc = batch_launch(ctx, b, ba, b->choice, b->stream);
        hipGraph_t g = nullptr;
        hipError_t ec = hipStreamEndCapture(b->stream, &g);
        if (rc) return rc;
        if (ec != hipSuccess) return argus_fail(ctx, ARGUS_EHIP, "graph capture failed");
        b->graph = g;
        ARGUS_HIP_CHECK(ctx, hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0));
        b->frames.assign(frames, frames + b->n_frames);
        memcpy(b->outs, outs, sizeof outs);
        b->thr = threshold;
    }
    argus_time_begin(ctx);
    ARGUS_HIP_CHECK(ctx, hipGraphLaunch(b->exec, b->stream));
    ARGUS_HIP_CHECK(ctx, hipEventRecord(b->ev_out, b->stream));
    ARGUS_HIP_CHECK(ctx, hipStreamWaitEvent(ctx->stream, b->ev_out, 0));
    argus_time_end(ctx, "batch");
    return ARGUS_OK;
}

int argus_batch_tuning(const argus_batch *b, float *cand_ms, int capacity, int *n_candidates,
                       int *from_cache) {
    if (!b || capacity < 0 || (capacity > 0 && !cand_ms)) return ARGUS_EINVAL;
    const int n = (int)b->cand_ms.size();
    for (int i = 0; i < n && i < capacity; ++i) cand_ms[i] = b->cand_ms[i];
    if (n_candidates) *n_candidates = n;
    if (from_cache) *from_cache = b->from_cache;
    return ARGUS_OK;
}

int argus_batch_candidate(int index, int *tile_rows, int *wg_per_cu) {
    if (index < 0 || index >= N_CAND) return ARGUS_EINVAL;
    if (tile_rows) *tile_rows = CAND_TILE[index];
    if (wg_per_cu) *wg_per_cu = CAND_WPC[index];
    return ARGUS_OK;
}

int argus_batch_info(const argus_batch *b, int *choice, float *ms, int *n_candidates) {
    if (!b) return ARGUS_EINVAL;
    if (choice) *choice = b->choice;
    if (ms) *ms = b->tuned_ms;
    if (n_candidates) *n_candidates = b->n_cand;
    return ARGUS_OK;
}

void argus_batch_destroy(argus_batch *b) {
    if (!b) return;
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->ev_in) (void)hipEventDestroy(b->ev_in);
    if (b->ev_out) (void)hipEventDestroy(b->ev_out);
    if (b->stream) (void)hipStreamDestroy(b->stream);
    if (b->dev) (void)hipFree(b->dev);
    delete b;
}

}  // extern "C"
