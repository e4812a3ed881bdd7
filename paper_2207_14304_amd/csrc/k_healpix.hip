// Resampling of a calibrated frame into HEALPix-aligned segment images.
//
// A segment is one tile (face f, I, J) of NSIDE n; its m x m pixels are the
// HEALPix pixels of NSIDE n m inside the tile: pixel (p, q) (row q, column p)
// sits at face coordinates a = (I m + p + 1/2)/(n m), b = (J m + q + 1/2)/(n m).
// Per segment pixel (FP64 geometry): face coordinates -> HEALPix plane ->
// sphere -> gnomonic frame position -> bilinear interpolation of the frame
// (value: sum w cal; variance: sum w^2 var); NODATA where the position is off
// the frame (or behind the tangent plane) or any of the four neighbours is
// masked.
//
// On the plane the latitude (z, and the polar stretch 1/sigma) depends on a + b
// alone and the unstretched longitude on a - b alone, so a workgroup (32 x 32
// pixels of a segment) forms them once per diagonal in LDS; a pixel then needs
// no square root, remainder or library sine: the longitude is an offset d from
// the block's middle, and sin, cos of ra - ra0 follow from those of the middle
// and the short series of sin d, cos d.  The other bound is the gather: a wave's
// neighbours lie on as many cache lines of the (rotated) frame as it has lanes,
// so the block's bounding box of the frame (46 x 46 at equal scales, twice the
// block's area) is staged in LDS with row loads and the neighbours are read
// there.  210 segments of 600^2 pixels of the full frame: 1178 -> 519 us (of
// which the gathers took 700 us from global memory).  Coarser segments, whose
// boxes do not fit, gather from the frame, a pixel a thread.
#include <algorithm>
#include <set>
#include <tuple>

#include "internal.h"
#include "healpix.h"

namespace {

using namespace argus_hp;

struct HpArgs {
    const float *cal, *var;
    const uint8_t *mask;
    const int32_t *tiles;              // [n][3]: face, I, J
    float *out, *outv;
    uint8_t *outm;
    Wcs w;
    int64_t pitch;
    int W, H, nside, m;
};

// 1 / v for a normal v: the hardware estimate and two Newton steps
__device__ __forceinline__ double recip(double v) {
    double r = __builtin_amdgcn_rcp(v);
    r = fma(fma(-v, r, 1.0), r, r);
    return fma(fma(-v, r, 1.0), r, r);
}

// BS x BS pixels a workgroup.  BOX > 0: neighbours from a box of at most BOX
// frame pixels in LDS, a wave on rows of the block (whole-line stores); else from
// the frame, a wave on 8 x 8 patches (whose neighbours lie on the fewest lines).
template <int BS, int BOX, int WG>
__global__ __launch_bounds__(256, WG) void healpix_resample_kernel(HpArgs a) {
    constexpr bool BOXED = BOX > 0;
    constexpr int ND = 2 * BS - 1;             // diagonals of a block
    constexpr int NK = BS * BS / 256;          // pixels of a thread
    constexpr int CAP = BOXED ? BOX : 1;
    __shared__ double sz[ND], sc[ND], si[ND];  // per a + b: z, cos dec, 1 / sigma
    __shared__ double sx[ND];                  // per a - b: longitude from phi_c
    __shared__ double smid[3];                 // the middle's longitude - ra0, its sin and cos
    __shared__ int sbox[4];                    // -xmin, -ymin, xmax, ymax of the neighbours (maxima)
    __shared__ float2 bv[CAP];                 // the box: value, variance
    __shared__ uint8_t bm[CAP];                // and mask
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // blocks in raster order of their segments, each XCD a contiguous run: the
    // boxes of neighbouring blocks overlap, and share an L2 this way
    const int nx = (a.m + BS - 1) / BS, nb = nx * nx;
    const int lb = argus_xcd_block((int)(blockIdx.y * gridDim.x + blockIdx.x), nb * (int)gridDim.y);
    const int t = lb / nb, p0 = (lb % nb) % nx * BS, q0 = (lb % nb) / nx * BS;
    const int f = a.tiles[3 * t], I = a.tiles[3 * t + 1], J = a.tiles[3 * t + 2];
    const double nm = (double)a.nside * a.m;
    double xc, yc;
    face_centre(f, xc, yc);
    // diagonals of pixel (p0 + pl, q0 + ql): pl + ql (a + b) and
    // pl - ql + BS - 1 (a - b).  The polar stretch is about the centre of the
    // base pixel's quadrant, phi_c = x_c (equatorial base pixels: any reference).
    const double a0 = (double)I * a.m + p0 + 0.5, b0 = (double)J * a.m + q0 + 0.5;
    auto latitude = [&](int i, double &z, double &is) {
        const double ys = yc + QP * ((a0 + b0 + i) / nm - 1.0);
        z = ys * (8.0 / (3.0 * PI));
        is = 1.0;
        if (fabs(ys) > QP) {
            const double sig = 2.0 - fabs(ys) / QP;
            z = (ys > 0 ? 1.0 : -1.0) * (1.0 - sig * sig / 3.0);
            is = sig > 0 ? 1.0 / sig : 0.0;
        }
    };
    auto longitude = [&](int i) { return QP * ((a0 - b0 + (i - (BS - 1))) / nm); };
    if (wv == 0) {
        if (lane < ND) {
            double z, is;
            latitude(lane, z, is);
            sz[lane] = z;
            sc[lane] = sqrt(fmax(1.0 - z * z, 0.0));
            si[lane] = is;
        }
    } else if (wv == 1) {
        if (lane < ND) sx[lane] = longitude(lane);
        if (lane < 4) sbox[lane] = -(1 << 30);
    } else if (wv == 2) {
        double z, is;
        latitude(BS - 1, z, is);
        const double mid = (xc - a.w.ra0) + longitude(BS - 1) * is;
        double s, c;
        sincos(mid, &s, &c);
        if (lane == 0) {
            smid[0] = mid;
            smid[1] = s;
            smid[2] = c;
        }
    }
    __syncthreads();
    const double off = (xc - a.w.ra0) - smid[0], sm = smid[1], cm = smid[2];
    const double r2d = 180.0 / PI;
    const double ax = r2d * a.w.cdi[0], bx = r2d * a.w.cdi[1], ay = r2d * a.w.cdi[2],
                 by = r2d * a.w.cdi[3];
    // column and row of this thread's pixel k
    auto col = [&](int k) { return BOXED ? tid & (BS - 1) : 8 * ((wv + 4 * k) % (BS / 8)) + (lane & 7); };
    auto row = [&](int k) {
        return BOXED ? tid / BS + 256 / BS * k : 8 * ((wv + 4 * k) / (BS / 8)) + (lane >> 3);
    };
    double X[NK], Y[NK];
    int ext[4] = {-(1 << 30), -(1 << 30), -(1 << 30), -(1 << 30)};
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int pl = col(k), ql = row(k), p = p0 + pl;
        const double z = sz[pl + ql], cd = sc[pl + ql];
        const double d = fma(sx[pl - ql + BS - 1], si[pl + ql], off);
        double sd, cs;
        if (fabs(d) <= 0.0625) {
            const double d2 = d * d;
            sd = fma(d2, fma(d2, fma(d2, fma(d2, 1.0 / 362880, -1.0 / 5040), 1.0 / 120), -1.0 / 6), 1.0) * d;
            cs = fma(d2, fma(d2, fma(d2, fma(d2, 1.0 / 40320, -1.0 / 720), 1.0 / 24), -0.5), 1.0);
        } else {
            sincos(d, &sd, &cs);           // close to a pole
        }
        const double s = sm * cs + cm * sd, c = cm * cs - sm * sd;
        const double den = z * a.w.sd0 + cd * a.w.cd0 * c;
        const double rd = recip(den);
        const double xi = cd * s, eta = z * a.w.cd0 - cd * a.w.sd0 * c;
        const double x = fma(fma(ax, xi, bx * eta), rd, a.w.crpix1);
        const double y = fma(fma(ay, xi, by * eta), rd, a.w.crpix2);
        const bool in = p < a.m && q0 + ql < a.m && den > 0.0 && x >= 0.0 && x <= a.W - 1.0 &&
                        y >= 0.0 && y <= a.H - 1.0;
        X[k] = in ? x : -1.0;
        Y[k] = y;
        if (in) {
            const int x0 = min((int)x, max(a.W - 2, 0)), y0 = min((int)y, max(a.H - 2, 0));
            ext[0] = max(ext[0], -x0);
            ext[1] = max(ext[1], -y0);
            ext[2] = max(ext[2], min(x0 + 1, a.W - 1));
            ext[3] = max(ext[3], min(y0 + 1, a.H - 1));
        }
    }
    int bx0 = 0, by0 = 0, bs = 0;
    bool boxed = false;
    if constexpr (BOXED) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            for (int o = 32; o > 0; o >>= 1) ext[e] = max(ext[e], __shfl_xor(ext[e], o));
            if (lane == 0) atomicMax(&sbox[e], ext[e]);
        }
        __syncthreads();
        bx0 = -sbox[0];
        by0 = -sbox[1];
        const int bw = sbox[2] - bx0 + 1, bh = sbox[3] - by0 + 1;
        bs = bw | 1;                           // odd LDS row stride
        // (a box may not fit after all, as where the pixels are sheared near the
        // poles: its block gathers from the frame)
        boxed = bw > 0 && bw <= 64 && bh <= BOX && bs * bh <= BOX;
        if (boxed) {
            const int xl = bx0 + min(lane, bw - 1);
#pragma unroll 4
            for (int r = wv; r < bh; r += 4) {
                const int64_t o = (int64_t)(by0 + r) * a.pitch + xl;
                const float2 v = make_float2(a.cal[o], a.var[o]);
                const uint8_t m = a.mask[o];
                if (lane < bw) {
                    bv[r * bs + lane] = v;
                    bm[r * bs + lane] = m;
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int p = p0 + col(k), q = q0 + row(k);
        if (p >= a.m || q >= a.m) continue;
        float val = 0.f, vv = 0.f;
        uint8_t msk = ARGUS_NODATA;
        if (X[k] >= 0.0) {
            const int x0 = min((int)X[k], max(a.W - 2, 0)), y0 = min((int)Y[k], max(a.H - 2, 0));
            const int x1 = min(x0 + 1, a.W - 1), y1 = min(y0 + 1, a.H - 1);
            const double fx = X[k] - x0, fy = Y[k] - y0;
            float2 n00, n01, n10, n11;
            uint32_t m4;
            if (boxed) {
                const int r0 = (y0 - by0) * bs - bx0, r1 = (y1 - by0) * bs - bx0;
                n00 = bv[r0 + x0];
                n01 = bv[r0 + x1];
                n10 = bv[r1 + x0];
                n11 = bv[r1 + x1];
                m4 = bm[r0 + x0] | bm[r0 + x1] | bm[r1 + x0] | bm[r1 + x1];
            } else {
                const int64_t r0 = (int64_t)y0 * a.pitch, r1 = (int64_t)y1 * a.pitch;
                n00 = make_float2(a.cal[r0 + x0], a.var[r0 + x0]);
                n01 = make_float2(a.cal[r0 + x1], a.var[r0 + x1]);
                n10 = make_float2(a.cal[r1 + x0], a.var[r1 + x0]);
                n11 = make_float2(a.cal[r1 + x1], a.var[r1 + x1]);
                m4 = a.mask[r0 + x0] | a.mask[r0 + x1] | a.mask[r1 + x0] | a.mask[r1 + x1];
            }
            if (m4 == 0) {
                const double w00 = (1 - fx) * (1 - fy), w01 = fx * (1 - fy), w10 = (1 - fx) * fy,
                             w11 = fx * fy;
                val = (float)(w00 * n00.x + w01 * n01.x + w10 * n10.x + w11 * n11.x);
                vv = (float)(w00 * w00 * n00.y + w01 * w01 * n01.y + w10 * w10 * n10.y +
                             w11 * w11 * n11.y);
                msk = 0;
            }
        }
        const int64_t o = ((int64_t)t * a.m + q) * a.m + p;
        a.out[o] = val;
        a.outv[o] = vv;
        a.outm[o] = msk;
    }
}

}  // namespace

int launch_resample_healpix(argus_ctx *ctx, argus_dims d, const float *cal, const float *var,
                            const uint8_t *mask, const argus_wcs *wcs, int nside, int m,
                            const int32_t *tiles, int n_tiles, float *out, float *out_var,
                            uint8_t *out_mask) {
    HpArgs a;
    if (!make_wcs(*wcs, a.w)) return argus_fail(ctx, ARGUS_EINVAL, "singular or non-finite cd matrix");
    a.cal = cal; a.var = var; a.mask = mask; a.tiles = tiles;
    a.out = out; a.outv = out_var; a.outm = out_mask;
    a.pitch = d.pitch; a.W = d.width; a.H = d.height; a.nside = nside; a.m = m;
    // Side of a segment pixel in frame pixels, and the smallest box that 32 x 32
    // segment pixels turned by 45 degrees fit (larger boxes leave fewer workgroups
    // on a CU); past the largest (64 columns, a wave's row) single gathers.  207
    // segments of the full frame (us): 600^2 (scale 1) box of 2250 574, 3000 635,
    // none 868; 550^2 (1.09) 3000 628, 4000 678, none 791; 450^2 (1.33) 4000 480,
    // none 577; without a box 300^2 328, 150^2 187, 60^2 91, where blocks of 32 x 32
    // take 436, 248, 110 and boxes of 16 x 16 342, 249, 100.
    const double seg = sqrt(4.0 * PI / 12.0) / ((double)nside * m) * (180.0 / PI);
    const double ratio = seg / sqrt(fabs(a.w.cd[0] * a.w.cd[3] - a.w.cd[1] * a.w.cd[2]));
    const double side = 32 * ratio * 1.41421356 + 2.0, area = side * side;
    argus_time_begin(ctx);
    auto launch = [&](auto kernel, int bs) {
        const int nx = (m + bs - 1) / bs;
        hipLaunchKernelGGL(kernel, dim3(nx * nx, n_tiles), dim3(256), 0, ctx->stream, a);
    };
    if (area <= 2250.0) launch(healpix_resample_kernel<32, 2250, 7>, 32);
    else if (area <= 3000.0) launch(healpix_resample_kernel<32, 3000, 5>, 32);
    else if (area <= 4000.0) launch(healpix_resample_kernel<32, 4000, 4>, 32);
    else launch(healpix_resample_kernel<16, 0, 7>, 16);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    argus_time_end(ctx, "healpix_resample");
    return ARGUS_OK;
}

// Tiles that the frame's pixels fall in, sampled every `step` pixels along
// both axes and along the last row and column.
int healpix_tiles(const argus_wcs *wcs, int W, int H, int nside, int step, int32_t *tiles,
                  int capacity, int *n_tiles) {
    Wcs w;
    if (!make_wcs(*wcs, w)) return ARGUS_EINVAL;
    std::set<std::tuple<int, int, int>> s;
    auto add = [&](int x, int y) {
        double z, ra, xs, ys, fa, fb;
        pixel_to_sky(w, x, y, z, ra);
        sphere_to_plane(z, ra, xs, ys);
        const int f = plane_to_face(xs, ys, fa, fb);
        if (f < 0) return;
        const int I = std::min((int)(fa * nside), nside - 1);
        const int J = std::min((int)(fb * nside), nside - 1);
        s.insert(std::make_tuple(f, I, J));
    };
    for (int y = 0;; y += step) {
        const int yy = std::min(y, H - 1);
        for (int x = 0;; x += step) {
            add(std::min(x, W - 1), yy);
            if (x >= W - 1) break;
        }
        if (y >= H - 1) break;
    }
    *n_tiles = (int)s.size();
    int i = 0;
    for (const auto &t : s) {
        if (i >= capacity) break;
        tiles[3 * i] = std::get<0>(t);
        tiles[3 * i + 1] = std::get<1>(t);
        tiles[3 * i + 2] = std::get<2>(t);
        ++i;
    }
    return ARGUS_OK;
}
