// Shadow-map rasterization on the device: the light pass whose depth map the
// RBSM pass consumes (Sec. 2 takes it as given).  Included once, by rbsm.hip.
//
// A texel (i, j) samples its centre ((i + 0.5) / W, (j + 0.5) / H) in texture
// coordinates; it holds the nearest surface there: the receiver plane
// r0 + ru (u - 0.5) + rv (v - 0.5) (binary64, rounded to binary32) unless a
// primitive covering the centre has a smaller depth; among equal depths
// (+0 and -0 compare equal) the plane wins, then the primitive of lowest
// index.  A convex counter-clockwise polygon covers a point when no edge
// function (b - a) x (p - a) is negative and every zero lies on an edge that
// owns ties (one running downwards, or horizontally to the left: the
// top-left rule); a slab covers o <= nx u + ny v < o + w.  All coverage
// arithmetic is binary64 without contraction, so decisions are reproducible
// exactly.
//
// One workgroup of four waves per region of 64 x 16R texels (or REP of them,
// one below the other), a thread 4 columns of R rows, its texels in registers
// throughout.  Primitives come in batches of 256, a lane each: those that may
// cover a centre of the region (margins far above the binary64 rounding of
// the edge functions make every such decision safe) go to LDS as edge vectors.
// Each wave then classifies them, a lane each, against its own 64 x 4R
// centres: covering none, every one, or maybe some; ballots keep the outcome
// in scalar registers.  The wave goes through its primitives in index order: a
// covering one is a compare and a select per texel, a partial one tests its
// edges, the products that depend on the column alone computed once for the R
// rows.  In index order a strict compare leaves the plane, then the lowest
// index, among equal depths.
//
// Bound by the write of the map on large maps (8192^2: 41-56 us by run, median
// 47, 71 in some processes for reasons not known; the plane alone 39), by the
// latency of load, bounds and classification on small ones (1024^2: 8 us, the
// plane alone 4).  A workgroup per 64 x 64, 32 x 32 or 16 x
// 16 tile with the primitives' indices listed in LDS and every coordinate
// divided took 74 us at 8192^2, 42 at 4096^2 (now 18), 25 at 2048^2 (now 12)
// and 20 at 1024^2.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rbsm.h"
#include "tile_pass.hpp"

namespace rbsm {

constexpr int kRasT = 256;    // threads per workgroup
constexpr int kRasKeep = 64;  // primitives of a region in LDS at a time

// What decides whether a primitive may cover a centre of a rectangle: a
// polygon's bounding box (xmin, xmax, ymin, ymax), or a slab's (nx, ny, o, w).
struct RasBound {
    double a, b, c, d;
    int kind;  // 0 polygon, 1 slab, 2 neither (covers nothing)
};

__device__ __forceinline__ RasBound bound_of(const rbsm_prim &q) {
    if (q.kind == 1) return RasBound{q.nx, q.ny, q.o, q.w, 1};
    RasBound r{q.x[0], q.x[0], q.y[0], q.y[0], q.kind != 0 || q.nv < 3 || q.nv > 4 ? 2 : 0};
#pragma unroll
    for (int e = 1; e < 4; ++e) {
        if (e == 3 && q.nv != 4) break;
        r.a = fmin(r.a, q.x[e]);
        r.b = fmax(r.b, q.x[e]);
        r.c = fmin(r.c, q.y[e]);
        r.d = fmax(r.d, q.y[e]);
    }
    return r;
}

// May it cover a texel centre in [u0, u1] x [v0, v1]?  Bounds grown by `pad`
// (a texel) so rounding never drops a covering primitive.
__device__ __forceinline__ bool may_touch(const RasBound &q, double u0, double u1, double v0, double v1, double pad) {
    if (q.kind == 1) {
        const double t00 = q.a * u0 + q.b * v0, t10 = q.a * u1 + q.b * v0;
        const double t01 = q.a * u0 + q.b * v1, t11 = q.a * u1 + q.b * v1;
        const double lo = fmin(fmin(t00, t10), fmin(t01, t11)), hi = fmax(fmax(t00, t10), fmax(t01, t11));
        return hi + pad >= q.c && lo - pad < q.c + q.d;
    }
    return q.kind == 0 && q.b + pad >= u0 && q.a - pad <= u1 && q.d + pad >= v0 && q.c - pad <= v1;
}

__device__ __forceinline__ rbsm_prim load_prim(const rbsm_prim *p) {
    const float *src = reinterpret_cast<const float *>(p);
    f32x4u raw[7];
#pragma unroll
    for (int w = 0; w < 7; ++w) raw[w] = gld4u(src + 4 * w);
    rbsm_prim q;
    __builtin_memcpy(&q, raw, sizeof(q));
    return q;
}

// The centre (i + 0.5) / n of texel i of n <= 65536, inv = 1 / n: the
// correctly rounded quotient by one residual step on the rounded reciprocal
// (equal to the division for every i and n).
__device__ __forceinline__ double centre(int i, double n, double inv) {
    const double x = i + 0.5, q = x * inv;
    return __builtin_fma(__builtin_fma(-q, n, x), inv, q);
}

// A primitive as the tests need it.  Polygon: per edge its start (ax, ay),
// its vector (dx, dy), the margin of its corner values (below), and the least
// edge value that is inside: 0 for an edge that owns ties, else the smallest
// positive double.  Slab: e[0] holds nx, ny, o, o + w and the margin.
struct RasEdge {
    double ax, ay, dx, dy, margin, least;
};
struct RasPrim {
    RasEdge e[4];
    float z;
    int nv;  // edges, 0: slab
};

constexpr double kRasMargin = 0x1p-40;

// How q meets the texel centres of [u0, u1] x [v0, v1] (all in [0, 1]):
// 0 none, 2 every one, 1 maybe some.  An edge function is affine, so its exact
// extremes over the rectangle are at corners; binary64 evaluation errs by well
// under 2^-50 times the scale of the margin, so corner values beyond 2^-40
// times that scale fix the sign of every centre's binary64 value.  Slabs
// likewise on nx u + ny v.  Answer 1 is always safe: q is then tested texel by
// texel.
__device__ __forceinline__ int tile_cover(const RasPrim &q, double u0, double u1, double v0, double v1) {
    if (q.nv == 0) {
        const RasEdge &s = q.e[0];
        const double t00 = s.ax * u0 + s.ay * v0, t10 = s.ax * u1 + s.ay * v0;
        const double t01 = s.ax * u0 + s.ay * v1, t11 = s.ax * u1 + s.ay * v1;
        const double lo = fmin(fmin(t00, t10), fmin(t01, t11)), hi = fmax(fmax(t00, t10), fmax(t01, t11));
        if (hi + s.margin < s.dx || lo - s.margin >= s.dy) return 0;
        return lo - s.margin >= s.dx && hi + s.margin < s.dy ? 2 : 1;
    }
    bool all = true;
    for (int e = 0; e < q.nv; ++e) {
        const RasEdge &s = q.e[e];
        const double a0 = s.dx * (v0 - s.ay), a1 = s.dx * (v1 - s.ay);
        const double b0 = s.dy * (u0 - s.ax), b1 = s.dy * (u1 - s.ax);
        const double e00 = a0 - b0, e10 = a0 - b1, e01 = a1 - b0, e11 = a1 - b1;
        if (fmax(fmax(e00, e10), fmax(e01, e11)) < -s.margin) return 0;  // negative at every centre
        all = all && fmin(fmin(e00, e10), fmin(e01, e11)) > s.margin;    // false on NaN
    }
    return all ? 2 : 1;
}

// The record of primitive q.
__device__ __forceinline__ void make_prim(const rbsm_prim &q, RasPrim &p) {
    p.z = q.depth;
    p.nv = q.kind == 1 ? 0 : q.nv;
    if (q.kind == 1) {
        p.e[0].ax = q.nx;
        p.e[0].ay = q.ny;
        p.e[0].dx = q.o;
        p.e[0].dy = q.o + q.w;
        p.e[0].margin = kRasMargin * (fabs(q.nx) + fabs(q.ny));
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (e >= q.nv) break;
        const bool end = e + 1 == q.nv;
        const double ax = q.x[e], ay = q.y[e];
        const double dx = (end ? q.x[0] : q.x[(e + 1) & 3]) - ax, dy = (end ? q.y[0] : q.y[(e + 1) & 3]) - ay;
        p.e[e].ax = ax;
        p.e[e].ay = ay;
        p.e[e].dx = dx;
        p.e[e].dy = dy;
        p.e[e].margin = kRasMargin * (fabs(dx) * (1.0 + fabs(ay)) + fabs(dy) * (1.0 + fabs(ax)));
        p.e[e].least = dy < 0.0 || (dy == 0.0 && dx < 0.0) ? 0.0 : 0x1p-1074;
    }
}

template <int R, int REP>
__global__ __launch_bounds__(kRasT) void raster_kernel(const rbsm_prim *__restrict__ prims, int n, double r0,
                                                       double ru, double rv, int W, int H, double inv_w, double inv_h,
                                                       int64_t pitch, float *__restrict__ map, int tiles_x,
                                                       int chunk_log2) {
    __shared__ RasPrim s_prim[kRasKeep];
    __shared__ int s_count[kRasT / 64];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int tile = (int)xcd_chunked(blockIdx.x, gridDim.x, chunk_log2);
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    const int i0 = tx * 64, i1 = min(i0 + 64, W) - 1;
    const double fw = W, fh = H;
    const double u0 = centre(i0, fw, inv_w), u1 = centre(i1, fw, inv_w);
    const int col = i0 + (lane & 15) * 4;
    double px[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) px[c] = centre(col + c, fw, inv_w);
    rbsm_prim q;       // REP == 1: this thread's primitive of the batch
    RasBound bound{};  // and its bounds
    bound.kind = 2;
    for (int rep = 0; rep < REP; ++rep) {
        const int j0 = (ty * REP + rep) * (16 * R);
        if (REP > 1 && j0 >= H) break;  // uniform
        const int jw = j0 + wave * (4 * R);  // the wave's rows jw .. jw + 4R - 1, a lane's jw + lane / 16 + 4r
        const int row = jw + (lane >> 4);
        double py[R];
        float d[R][4];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            py[r] = centre(row + 4 * r, fh, inv_h);
#pragma unroll
            for (int c = 0; c < 4; ++c) d[r][c] = (float)(r0 + ru * (px[c] - 0.5) + rv * (py[r] - 0.5));
        }
        // depth of the nearest primitive so far that covers the wave's every centre
        float cover = __builtin_inff();
        for (int first = 0; first < n; first += kRasT) {
            // the batch's primitives that may cover a centre of the region
            if (REP == 1 || rep == 0 || n > kRasT) {
                bound.kind = 2;
                if (first + t < n) {
                    const rbsm_prim p = load_prim(prims + first + t);
                    bound = bound_of(p);
                    if (REP == 1) q = p;
                }
            }
            const double v0 = centre(j0, fh, inv_h), v1 = centre(min(j0 + 16 * R, H) - 1, fh, inv_h);
            const bool touch = may_touch(bound, u0, u1, v0, v1, W < H ? inv_w : inv_h);
            const unsigned long long kept = __ballot(touch);
            if (first > 0 || rep > 0) __syncthreads();  // the last batch's counts are read
            if (lane == 0) s_count[wave] = __builtin_popcountll(kept);
            __syncthreads();
            int at = 0, total = 0;
#pragma unroll
            for (int w = 0; w < kRasT / 64; ++w) {
                at += w < wave ? s_count[w] : 0;
                total += s_count[w];
            }
            at += __builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
            total = __builtin_amdgcn_readfirstlane(total);
            for (int lo = 0; lo < total; lo += kRasKeep) {
                if (lo > 0) __syncthreads();  // the last ones are done with
                if (touch && at >= lo && at < lo + kRasKeep) {
                    if (REP > 1) q = load_prim(prims + first + t);
                    make_prim(q, s_prim[at - lo]);
                }
                __syncthreads();
                if (jw >= H) continue;  // a wave past the map's last row
                const int m = min(total - lo, kRasKeep);
                int c = 0;
                bool slab = false;
                if (lane < m) {
                    const double w0 = centre(jw, fh, inv_h), w1 = centre(min(jw + 4 * R, H) - 1, fh, inv_h);
                    c = tile_cover(s_prim[lane], u0, u1, w0, w1);
                    slab = s_prim[lane].nv == 0;
                }
                const unsigned long long full = __ballot(c == 2), slabs = __ballot(slab);
                for (unsigned long long left = __ballot(c != 0); left != 0ull; left &= left - 1ull) {
                    const int k = __builtin_ctzll(left);
                    const RasPrim &p = s_prim[k];
                    const float z = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(p.z)));
                    if (!(z < cover)) continue;  // every texel holds at most `cover` (or a NaN, which stays)
                    bool in[R][4];
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int e = 0; e < 4; ++e) in[r][e] = true;
                    if ((full >> k) & 1ull) {
                        cover = z;
                    } else if ((slabs >> k) & 1ull) {
                        const RasEdge &s = p.e[0];
#pragma unroll
                        for (int r = 0; r < R; ++r)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const double v = s.ax * px[e] + s.ay * py[r];
                                in[r][e] = v >= s.dx && v < s.dy;
                            }
                    } else {
                        const int nv = __builtin_amdgcn_readfirstlane(p.nv);
                        for (int g = 0; g < nv; ++g) {
                            const RasEdge s = p.e[g];
                            double b[4];
#pragma unroll
                            for (int e = 0; e < 4; ++e) b[e] = s.dy * (px[e] - s.ax);
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const double a = s.dx * (py[r] - s.ay);
#pragma unroll
                                for (int e = 0; e < 4; ++e) in[r][e] = in[r][e] && !(a - b[e] < s.least);
                            }
                        }
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int e = 0; e < 4; ++e) d[r][e] = in[r][e] && z < d[r][e] ? z : d[r][e];
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int y = row + 4 * r;
            if (y >= H) continue;
            float *dst = map + (int64_t)y * pitch + col;
            if (col + 3 <= i1) {  // one 16-byte store, dword aligned
                f32x4u v;
                v.x = d[r][0]; v.y = d[r][1]; v.z = d[r][2]; v.w = d[r][3];
                *(__attribute__((address_space(1))) f32x4u *)dst = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e <= i1) gst(dst + e, d[r][e]);
            }
        }
    }
}

inline void launch_raster(const rbsm_prim *prims, int n, double r0, double ru, double rv, int W, int H, int64_t pitch,
                          float *map, hipStream_t stream) {
    // Larger regions spread the reading and bounding of the primitives (a
    // record per lane: 64 cache lines a load) over more texels; smaller ones
    // make workgroups enough for every CU.  64-triangle scenes, us for <1, 1>
    // / <2, 1> / <2, 2>: 1024^2 7.9 / 8.3 / 11.6, 1500 x 1100 9.3 / 7.9 /
    // 11.5, 2048^2 15.7 / 12.4 / 12.5, 4096^2 37.8 / 23.8 / 18.2, 8192^2 115 /
    // 66 / 41 (<4, 1> 43).
    const int64_t area = (int64_t)W * H;
    const int rows = area <= ((int64_t)1 << 20) ? 16 : (area <= ((int64_t)1 << 22) ? 32 : 64);  // texel rows a workgroup
    const int tiles_x = (W + 63) / 64;
    const dim3 grid((unsigned)((int64_t)tiles_x * ((H + rows - 1) / rows)));
    const auto kernel = rows == 16 ? &raster_kernel<1, 1> : (rows == 32 ? &raster_kernel<2, 1> : &raster_kernel<2, 2>);
    // regions in chunks of 32 (of 8 on the smaller maps) to each XCD: 8192^2,
    // three maps written in turn, 42.6 us; chunks of 8 44.7, of 128 45.9,
    // contiguous ranges 49.7
    const int chunk_log2 = rows == 64 ? 5 : 3;
    hipLaunchKernelGGL(kernel, grid, dim3(kRasT), 0, stream, prims, n, r0, ru, rv, W, H, 1.0 / W, 1.0 / H, pitch, map,
                       tiles_x, chunk_log2);
}

}  // namespace rbsm
