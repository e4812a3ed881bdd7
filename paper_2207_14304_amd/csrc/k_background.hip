// Median-filtered background map of a calibrated frame.
//
// bg_cell: one workgroup per box x box cell (box <= 64, so a thread holds at
//   most 16 pixels in registers).  The cell's level is the exact median of
//   its unmasked values: a radix select on order-preserving 32-bit keys of the
//   FP32 values (digits of 11, 11 and 10 bits, LDS histograms), and for an even
//   count the next key by a minimum; the mean of the middle pair is formed in
//   FP64 and rounded once.
// bg_filter: one thread per cell, median of the present levels of its 3 x 3
//   neighbourhood (a sorting network over 9 values).
// bg_map: bilinear interpolation between cell centres to every pixel (only
//   when the caller asks for the full-resolution map; detection evaluates the
//   same interpolation on the fly).
#include "internal.h"
#include "background.h"

namespace {

constexpr int NTHR = 256, MAXV = 16;     // 16 x 256 = 4096 = 64 x 64 pixels

__device__ __forceinline__ uint32_t f2key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key2f(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

struct CellArgs {
    const float *cal;
    const uint8_t *mask;
    float *levels;
    int64_t pitch;
    int W, H, box, gx, gy;
    int vec;                           // 16-byte rows of cal, 4-byte rows of mask, cells on them
};

// What bounds this kernel is instruction issue and LDS atomics, not its 5
// bytes per pixel (50 us on the full frame).  Whole cells of 32 or 64 columns
// on aligned planes read 4 pixels a lane with no divisions; a sky's keys share
// their first digit, so there a wave adds its first lane's digit with one
// atomic (64 lanes on one address take 64 turns); each thread clears the bins
// it scans, so a digit takes three barriers.  Full frame, 64 x 64 cells: 267 ->
// 122 us, against four 8-bit digits scanned by one wave.  Cells of at most a pixel
// a thread do one of a pass's 16 turns (1201x901, 4 x 4 cells: 414 us with four
// digits, 441 with all turns, 371).
__global__ __launch_bounds__(NTHR) void bg_cell_kernel(CellArgs a) {
    constexpr int NB = 2048, PER = NB / NTHR;
    __shared__ __align__(16) int hist[NB];
    __shared__ int wsum[NTHR / 64];
    __shared__ uint32_t sel[3];          // selected digit, rank within it, its count
    __shared__ uint32_t kmin;
    const int tid = threadIdx.x, lane = tid & 63;
    const int ci = blockIdx.x % a.gx, cj = blockIdx.x / a.gx;
    const int x0 = ci * a.box, y0 = cj * a.box;
    const int cw = min(a.box, a.W - x0), ch = min(a.box, a.H - y0);
    const int np = cw * ch;
    uint32_t key[MAXV];
    uint32_t okbits = 0;
    // every load of a thread is issued before any is used
    float v[MAXV];
    uint8_t m[MAXV];
    bool one = false;                      // at most one value a thread
    if (a.vec && (cw == 64 || cw == 32)) {
        const int lg = cw == 64 ? 4 : 3, row = tid >> lg, c4 = (tid & ((1 << lg) - 1)) * 4;
        const int step = NTHR >> lg;       // rows of a pass over the workgroup
        float4 q[4];
        uint32_t mm[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t o = (int64_t)(y0 + min(row + k * step, ch - 1)) * a.pitch + x0 + c4;
            q[k] = *(const float4 *)(a.cal + o);
            mm[k] = *(const uint32_t *)(a.mask + o);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float e[4] = {q[k].x, q[k].y, q[k].z, q[k].w};
            const bool in = row + k * step < ch;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[4 * k + j] = e[j];
                if (in && ((mm[k] >> (8 * j)) & 0xffu) == 0) okbits |= 1u << (4 * k + j);
            }
        }
    } else {
        one = np <= NTHR;
#pragma unroll
        for (int k = 0; k < MAXV; ++k) {
            const int i = tid + k * NTHR;
            const int ii = i < np ? i : 0;
            const int64_t o = (int64_t)(y0 + ii / cw) * a.pitch + x0 + ii % cw;
            v[k] = a.cal[o];
            m[k] = a.mask[o];
        }
#pragma unroll
        for (int k = 0; k < MAXV; ++k)
            if (tid + k * NTHR < np && m[k] == 0) okbits |= 1u << k;
    }
#pragma unroll
    for (int k = 0; k < MAXV; ++k) key[k] = f2key(v[k]);
#pragma unroll
    for (int i = 0; i < PER; ++i) hist[tid + i * NTHR] = 0;
    if (tid == 0) kmin = 0xffffffffu;
    __syncthreads();
    // k-th smallest key (0-based): the lower middle for an even count
    uint32_t prefix = 0, rank = 0;
    int n = 0;
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
        const uint32_t dmask = pass == 2 ? 1023u : 2047u;
#pragma unroll
        for (int k = 0; k < MAXV; ++k) {
            if (k == 1 && one) break;
            const bool ok = (okbits >> k) & 1u;
            const uint32_t d = (key[k] >> shift) & dmask;
            if (pass == 0) {
                const uint64_t act = __ballot(ok);
                if (act) {
                    const uint32_t d0 =
                        (uint32_t)__builtin_amdgcn_readlane((int)d, __builtin_ctzll(act));
                    const bool same = ok && d == d0;
                    const uint64_t sm = __ballot(same);
                    if (lane == 0) atomicAdd(&hist[d0], __popcll(sm));
                    if (ok && !same) atomicAdd(&hist[d], 1);
                }
            } else if (ok && key[k] >> (pass == 1 ? 21 : 10) == prefix) {
                atomicAdd(&hist[d], 1);
            }
        }
        __syncthreads();
        // each thread owns PER bins: inclusive scan of the sums, bins cleared
        int h[PER], s = 0;
#pragma unroll
        for (int i = 0; i < PER; i += 4) {
            const int4 q = *(const int4 *)&hist[PER * tid + i];
            *(int4 *)&hist[PER * tid + i] = make_int4(0, 0, 0, 0);
            h[i] = q.x; h[i + 1] = q.y; h[i + 2] = q.z; h[i + 3] = q.w;
            s += q.x + q.y + q.z + q.w;
        }
        int inc = s;
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (lane == 63) wsum[tid >> 6] = inc;
        __syncthreads();
        int before = inc - s, tot = 0;
        for (int w = 0; w < NTHR / 64; ++w) {
            if (w < (tid >> 6)) before += wsum[w];
            tot += wsum[w];
        }
        if (pass == 0) {
            n = tot;
            if (n == 0) {
                if (tid == 0) a.levels[blockIdx.x] = __builtin_nanf("");
                return;
            }
            rank = (uint32_t)((n - 1) / 2);
        }
        if ((uint32_t)before <= rank && rank < (uint32_t)(before + s)) {
            int acc = before;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if ((uint32_t)acc <= rank && rank < (uint32_t)(acc + h[i])) {
                    sel[0] = (uint32_t)(PER * tid + i);
                    sel[1] = rank - (uint32_t)acc;
                    sel[2] = (uint32_t)h[i];
                }
                acc += h[i];
            }
        }
        __syncthreads();
        prefix = prefix << (pass == 2 ? 10 : 11) | sel[0];
        rank = sel[1];
    }
    const uint32_t kk1 = prefix;
    float med;
    if (n & 1) {
        med = key2f(kk1);
    } else {
        // upper middle: the same key if it repeats past the rank, else the
        // smallest key above it
        uint32_t kk2 = kk1;
        if (rank + 1 >= sel[2]) {
            uint32_t mn = 0xffffffffu;
#pragma unroll
            for (int k = 0; k < MAXV; ++k)
                if (((okbits >> k) & 1u) && key[k] > kk1 && key[k] < mn) mn = key[k];
            for (int off = 32; off > 0; off >>= 1) {
                const uint32_t t = (uint32_t)__shfl_xor((int)mn, off);
                mn = t < mn ? t : mn;
            }
            if (lane == 0) atomicMin(&kmin, mn);
            __syncthreads();
            kk2 = kmin;
        }
        med = (float)(0.5 * ((double)key2f(kk1) + (double)key2f(kk2)));
    }
    if (tid == 0) a.levels[blockIdx.x] = med;
}

// An odd-even transposition network over 9 values, absent ones +inf at the
// end (values in registers: a sort with run-time indices would live in
// scratch memory).
__global__ void bg_filter_kernel(const float *levels, float *grid, int gx, int gy) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= gx * gy) return;
    const int i = c % gx, j = c / gx;
    float v[9];
    int n = 0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int ii = i + t % 3 - 1, jj = j + t / 3 - 1;
        const bool in = ii >= 0 && ii < gx && jj >= 0 && jj < gy;
        const float l = levels[in ? jj * gx + ii : c];
        const bool has = in && l == l;                      // NaN: no level
        v[t] = has ? l : __builtin_inff();
        n += has ? 1 : 0;
    }
#pragma unroll
    for (int r = 0; r < 9; ++r)
#pragma unroll
        for (int t = r & 1; t + 1 < 9; t += 2) {
            const float lo = fminf(v[t], v[t + 1]), hi = fmaxf(v[t], v[t + 1]);
            v[t] = lo;
            v[t + 1] = hi;
        }
    float a = 0.f, b = 0.f;                                 // the middle pair (n odd: a = b)
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        if (t == (n - 1) / 2) a = v[t];
        if (t == n / 2) b = v[t];
    }
    grid[c] = n == 0 ? 0.f : (n & 1) ? b : (float)(0.5 * ((double)a + (double)b));
}

// Four columns x MAP_ROWS rows a thread: a column's node and weight are formed
// once, and its values on the two node rows once per crossing of a cell centre,
// so a pixel costs one subtraction, one FMA and its 4 bytes (139 -> 48 us on
// the full frame against a pixel a thread).
constexpr int MAP_ROWS = 16;
__global__ __launch_bounds__(NTHR) void bg_map_kernel(BgGrid g, float *map, int64_t pitch, int W,
                                                      int H, int vec) {
    const int x = 4 * (blockIdx.x * NTHR + threadIdx.x), y0 = blockIdx.y * MAP_ROWS;
    if (x >= W) return;
    BgColumns<4> col(g, x);
    for (int y = y0; y < min(y0 + MAP_ROWS, H); ++y) {
        float o[4];
        col.at(g, y, o);
        float *p = map + (int64_t)y * pitch + x;
        if (vec && x + 3 < W) {
            *(float4 *)p = make_float4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (x + e < W) p[e] = o[e];
        }
    }
}

}  // namespace

int launch_background(argus_ctx *ctx, argus_dims d, const float *cal, const uint8_t *mask, int box,
                      float *levels, float *grid, float *map) {
    const int gx = (d.width + box - 1) / box, gy = (d.height + box - 1) / box;
    float *lev = levels;
    if (!lev) {
        int rc = argus_ws_reserve(ctx, (size_t)gx * gy * sizeof(float) + 256);
        if (rc) return rc;
        lev = (float *)ctx->ws;
    }
    // (cells of 33..63 columns may end in one of 32 that starts between words)
    const int vec = d.pitch % 4 == 0 && (uintptr_t)cal % 16 == 0 && (uintptr_t)mask % 4 == 0 && box % 4 == 0;
    CellArgs a{cal, mask, lev, d.pitch, d.width, d.height, box, gx, gy, vec};
    argus_time_begin(ctx);
    hipLaunchKernelGGL(bg_cell_kernel, dim3(gx * gy), dim3(NTHR), 0, ctx->stream, a);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    hipLaunchKernelGGL(bg_filter_kernel, dim3((gx * gy + 255) / 256), dim3(256), 0, ctx->stream,
                       (const float *)lev, grid, gx, gy);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    argus_time_end(ctx, "background");
    if (map) {
        BgGrid g = make_bg_grid(grid, box, d.width, d.height);
        argus_time_begin(ctx);
        const int mvec = d.pitch % 4 == 0 && (uintptr_t)map % 16 == 0;
        hipLaunchKernelGGL(bg_map_kernel,
                           dim3((d.width + 4 * NTHR - 1) / (4 * NTHR), (d.height + MAP_ROWS - 1) / MAP_ROWS),
                           dim3(NTHR), 0, ctx->stream, g, map, d.pitch, d.width, d.height, mvec);
        ARGUS_HIP_CHECK(ctx, hipGetLastError());
        argus_time_end(ctx, "background_map");
    }
    return ARGUS_OK;
}
