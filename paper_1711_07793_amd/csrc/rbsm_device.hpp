// Device-side building blocks of the RBSM / RSMSS per-fragment pass for gfx950.
//
// Every function here works on one texel neighbourhood of one fragment; the
// kernels decide how fragments map to lanes.  Arithmetic is binary32 in the
// order of the paper's listings, compiled without FMA contraction, so results
// are bit-reproducible against any IEEE binary32 evaluation in that order.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rbsm {

// Discontinuity bits of a texel: its left / right / top (+y) / bottom (-y)
// neighbour has the opposite shadow test result (Eq. 3).
enum : unsigned { BIT_L = 1u, BIT_R = 2u, BIT_T = 4u, BIT_B = 8u };

struct MapView {
    const float *__restrict__ t;
    int64_t pitch;
    int W, H;
};

// Loads and stores of device buffers through global-address-space pointers:
// pointers read from a job table in memory are otherwise generic, and the
// compiler then emits flat instructions, which count against the LDS counter
// too, so every LDS wait also waits for memory (and back-to-back loads of one
// fragment were serialised).
template <class T>
__device__ __forceinline__ T gld(const T *p) {
    return *(const __attribute__((address_space(1))) T *)p;
}
template <class T>
__device__ __forceinline__ void gst(T *p, T v) {
    *(__attribute__((address_space(1))) T *)p = v;
}
// 12-byte loads (three consecutive texels, 4-byte aligned) through a native
// vector type whose alignment is lowered to 4, so the load is exactly 12 bytes.
typedef float f32x3 __attribute__((ext_vector_type(3), aligned(4)));
__device__ __forceinline__ f32x3 gld3(const float *p) {
    return *(const __attribute__((address_space(1))) f32x3 *)p;
}
// 16-byte load of four consecutive texels at 4-byte alignment (map rows).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4u gld4u(const float *p) {
    return *(const __attribute__((address_space(1))) f32x4u *)p;
}

// Nearest-texel fetch with clamp-to-edge.
__device__ __forceinline__ float texel(const MapView &m, int i, int j) {
    i = min(max(i, 0), m.W - 1);
    j = min(max(j, 0), m.H - 1);
    return gld(m.t + ((int64_t)j * m.pitch + i));
}

// Eq. 1: lit (1) unless the biased fragment depth lies behind the blocker.
__device__ __forceinline__ bool lit(float zb, float t) { return !(zb > t); }

struct Addr {
    int i0, j0;   // texel of the fragment
    float fx, fy; // sub-texel position in [0, 1)
    float zb;     // z - bias
};

// Texel and sub-texel position of a light-space fragment.  The integer index
// is clamped to +-2^20, which cannot change any read on maps of at most 2^16
// texels per side with reach below 2^10.
__device__ __forceinline__ Addr address(float u, float v, float z, int W, int H, float bias) {
    Addr a;
    const float X = u * (float)W;
    const float Y = v * (float)H;
    const float flx = floorf(X), fly = floorf(Y);
    a.fx = X - flx;
    a.fy = Y - fly;
    a.i0 = (int)fminf(fmaxf(flx, -1048576.0f), 1048576.0f);
    a.j0 = (int)fminf(fmaxf(fly, -1048576.0f), 1048576.0f);
    a.zb = z - bias;
    return a;
}

// One axis of the normalized discontinuity space (Eq. 5): the code counts the
// walks that found an end (2 -> 1, 1 -> 0, 0 -> -1); with exactly one end the
// coordinate is the fragment's distance to the end texel's boundary over the
// number of edge texels on the axis; 1 with no end, 0 with two.
struct Axis {
    float nrd;
    int code;
};

__device__ __forceinline__ Axis normalize_axis(int rn, int rp, float f) {
    const int ends = (rn > 0) + (rp > 0);
    const int an = abs(rn), ap = abs(rp);
    const float len = (float)(an + ap - 1);
    const float a = rp > 0 ? (float)rp - f : (float)(an - 1) + f;
    const float q = a / len;
    Axis r;
    r.code = ends == 2 ? 1 : (ends == 0 ? -1 : 0);
    r.nrd = ends == 1 ? q : (ends == 0 ? 1.0f : 0.0f);
    return r;
}

// Listing 4 without shape branches: U/O (code 1 on either axis, which the
// short-U/O test d == 0.75 implies) shadow, and with nrd = 1 on an axis
// without ends the I shape falls out of the L-line test.
__device__ __forceinline__ float vis_hard(Axis x, Axis y) {
    const bool keep = (x.code != 1) & (y.code != 1) & !(y.nrd < 1.0f - x.nrd);
    return keep ? 1.0f : 0.0f;
}

// Listing 5 without shape branches: code-1 axes contribute 0 (O flips the
// test, U ramps along the other axis), an axis without ends contributes 1
// (the I shape returns the test), and the rest is the L ramp
// clamp((d.z + sign*ty) + sign*tx, 0, 1) with sign = 1 - 2 d.z.
__device__ __forceinline__ float vis_rsmss(bool s, Axis x, Axis y) {
    const float tx = x.code == 1 ? 0.0f : x.nrd;
    const float ty = y.code == 1 ? 0.0f : y.nrd;
    const float v = s ? (ty + tx) : ((1.0f - ty) - tx);
    const float lo = v > 0.0f ? v : 0.0f;
    return lo < 1.0f ? lo : 1.0f;
}

}  // namespace rbsm
