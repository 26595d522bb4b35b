// RPCF: the RSMSS value averaged over the (2r+1)^2 texels around a
// fragment's texel, each evaluated with the fragment's own sub-texel position
// and depth (PCF over the filtered edge, Sec. 5.3).  Included once, by
// rbsm.hip.
//
// Every term of one fragment tests texels against the same depth, so the pass
// first turns the fragment's (2r+3)^2 neighbourhood into shadow-test bits: a
// word per row and, transposed, a word per column.  A term's discontinuity
// mask (Eq. 2-3) is then a few shifts and XORs, and the terms without a
// discontinuity contribute their test result, so a row's worth of them is one
// popcount.  Only the terms with a discontinuity need traversals (Listing 3),
// normalization (Eq. 5) and Listing 5; their number varies wildly between
// fragments, so they are listed over a wave's 64 fragments and evaluated one
// lane per term.  On the words a traversal is a shift and a count of ones.
// The few that run out of the words before they stop are listed again and go
// on in global memory.  A box too large for 32-bit words (r > 14) is done in
// parts, one after the other.
//
// The average is the exact mean of the (2r+1)^2 binary32 terms, rounded to
// binary32.  Terms are summed as integers (multiples of 2^-52), what that
// leaves of the rare terms below 2^-29 in binary64, and the sum is divided by
// (2r+1)^2 once, in binary64: it stays within 5e-13 of the exact mean and
// within 2^-40 of it relatively, so the result is that mean rounded, up to one
// binary32 step at a near-tie.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "rbsm_device.hpp"
#include "tile_pass.hpp"

namespace rbsm {

constexpr int kRpcfT = 128;      // threads per workgroup, one fragment each
constexpr int kWinMaxR = 14;     // largest r whose 2r+3 rows and columns fit 32-bit words
constexpr int kWinPart = 22;     // beyond it: terms per side of a part, at most
constexpr int kWinLate = 128;    // terms per wave with a traversal that leaves the window
constexpr float kWinSmall = 0x1p-29f;  // a binary32 value from here on is a multiple of 2^-52

// Shadow-test bit of texel depth t for depth zb (Eq. 1): the sign bit of
// t - zb.  The difference is negative exactly when zb > t, except for
// t = -0, zb = +0 (difference -0, test lit) and for NaN; callers pass
// canon(t), which turns -0 into +0 and NaN (lit at every depth) into +inf.
__device__ __forceinline__ uint32_t push_bit(uint32_t w, float t, float zb) {
    return __builtin_amdgcn_alignbit(w, __float_as_uint(t - zb), 31);  // (w << 1) | sign
}

__device__ __forceinline__ float canon(float t) { return t != t ? __builtin_inff() : t + 0.0f; }

// A word of NR bits.
template <int NR>
struct WinWord {
    using T = typename std::conditional<(NR <= 16), uint16_t, uint32_t>::type;
};

// Transposes the S x S bit matrix a (bit x of a[y] becomes bit y of a[x]),
// S = 16 or 32, swapping blocks of J bits, then of J / 2, ...; words of a
// known to be zero fold away.
template <int S, int J = S / 2>
__device__ __forceinline__ void transpose_bits(uint32_t (&a)[S]) {
    // the bits whose position has bit J clear
    constexpr uint32_t m = J == 16  ? 0x0000ffffu
                           : J == 8 ? 0x00ff00ffu
                           : J == 4 ? 0x0f0f0f0fu
                           : J == 2 ? 0x33333333u
                                    : 0x55555555u;
#pragma unroll
    for (int k = 0; k < S; ++k) {
        if (k & J) continue;
        const uint32_t p = a[k], q = a[k + J];
        a[k] = (p & m) | ((q << J) & ~m);
        a[k + J] = ((p >> J) & m) | (q & ~m);
    }
    if constexpr (J > 1) transpose_bits<S, J / 2>(a);
}

// Steps and outcome of one traversal: it goes on for `go` steps and stops at
// the next, ending the edge there or not (after maxd steps: not).
struct WalkEnd {
    int go;
    uint32_t end;  // 1: step go + 1 ends the edge
};

// The coordinate of Eq. 5 on one axis from its two traversals (n towards
// smaller, p towards larger coordinates), as normalize_axis and the code-1
// rule of vis_rsmss: with exactly one end the distance over the length, 1 with
// none, 0 with two.  The quotient comes from the correctly rounded reciprocal
// of the length and one residual step, which gives the correctly rounded
// quotient (checked for every significand over every length up to 129; a
// position below 2^-100 may lose denormal bits).
__device__ __forceinline__ float win_axis(WalkEnd n, WalkEnd p, float f, const lds_float *rcp) {
    const int len = n.go + p.go + 1;
    const float a = (float)(p.end ? p.go + 1 : n.go) + (p.end ? -f : f);
    const float y = rcp[len];
    const float q0 = a * y;
    const float q = __builtin_fmaf(__builtin_fmaf(-q0, (float)len, a), y, q0);
    // selected with masks, not a select: no branch splits the reads above
    const uint32_t one = 0u - (n.end ^ p.end), none = (n.end | p.end) - 1u;
    return __uint_as_float((__float_as_uint(q) & one) | (0x3f800000u & none));
}

// One wave per 64 fragments (two waves per workgroup share a staged band).
//
// Each lane tests its fragment's NR x NR window (NR >= 2r+3 texels square,
// the (2r+3)^2 neighbourhood and up to a few texels more on each side) into
// NR row words, transposed in registers into NR column words; both stay in
// LDS, [word][lane].  With them every traversal of a term is a shift and a
// count of ones: along its row word for the horizontal pair, along its column
// word for the vertical pair.  The terms with a discontinuity of the wave's 64
// fragments are listed in LDS lane by lane round-robin (row by row, a ballot
// and a popcount per listed term of a lane, so no scan and no barrier), and
// evaluated one lane per term in full waves.  Neighbouring list entries belong
// to different fragments, so the words are read and the results added
// without bank or address conflicts.  A term with a traversal that runs out
// of the window before it stops goes to a second list and is finished from
// global memory, again in full waves.
//
// Results are summed as integers: a term v in [0, 1] adds the bits of 1 + v
// (binary64), a multiple of 2^-52, so the sum does not depend on the order of
// the list.  Only a term below 2^-29 can have bits under 2^-52: a ballot finds
// those, and their rounding errors are added to the fragment's own binary64
// sum one at a time.  (Looking for them costs 2% up to r = 6 and beyond r = 14,
// where the two registers of that sum are dear, nothing between; a second
// listing of their waves' terms cost 2-6%.)  64 bits hold fewer than
// 4096 such terms of value 1: a box in one part has at most 29^2, and after each
// of several parts the whole part of the sum moves to a counter of its own.
//
// A wave whose fragments all pass, or all fail, every test of the band (the
// band's depth range against theirs) is done at once: the mean is 1 or 0.
//
// MULTI: the (2r+1)^2 box in parts x parts parts of part_side terms a side
// (the last ones fewer), each with its own window, summed one after the other.
//
// Bound by VALU issue (about 120 instructions a listed term, 2 a test) and,
// where the words leave LDS for 8 to 10 waves per CU (r >= 11), by latency.
// Against one lane per term with per-step walks on a staged band and 64-bit
// column words (two scenes each): 4K fenced frame r = 5 0.87 / 1.71 ms ->
// 0.46 / 0.63, 1080p r = 13 2.23 / 1.75 -> 1.09 / 0.99, 720p r = 15 2.11 / 3.31
// -> 0.88 / 0.88, 640x360 r = 32 (one lane per fragment before) 26.5 -> 1.4.
// Keeping both kinds of words at 16 bits up to NR = 16 gives 28 waves per CU.
// Waves per SIMD: what LDS leaves room for.  MULTI at NR = 24 fits 6 workgroups
// (3 waves per SIMD, 164 VGPRs): held to 4 waves it spilled 24 registers, and
// 762 MB of a 4K r = 15 frame's writes were scratch (720p r = 21 1174 us against
// 1109, r = 32 2084 against 1965).  MULTI at NR = 20 spills 5 registers at 4
// waves, NR = 16 3 at 7; a wave fewer is slower (r = 5 522 -> 534 us at 6).
template <int NR, bool MULTI>
constexpr int kWinWaves = NR <= 16 ? 7 : MULTI && NR == 24 ? 3 : 4;  // per SIMD; a CU: 4 SIMDs, 2 waves a workgroup

template <int NR, bool MULTI>
__global__ __launch_bounds__(kRpcfT) __attribute__((amdgpu_waves_per_eu(kWinWaves<NR, MULTI>))) void
rpcf_window_kernel(
    MapView m, const float *__restrict__ frags, int64_t n, int64_t vw, int64_t tiles_x, int tw_log2, float bias,
    int maxd, int r, int parts, int part_side, int cap, int list_cap, int chunk_log2, float *__restrict__ out) {
    using Word = typename WinWord<NR>::T;
    constexpr int S = NR <= 16 ? 16 : 32;  // transposed size
    constexpr uint32_t kAll = NR == 32 ? 0xffffffffu : (1u << (NR & 31)) - 1u;
    // Dynamic LDS.  Of the NR rows and columns N = side + 2 stay (all NR in 16-bit
    // words, which leave LDS enough):
    //   row words [wave][N][lane], those of rows c0 - 1 .. c0 + side;
    //   the other rows' words of wave 0, the band (cap texels), the other
    //   rows' words of wave 1: all overwritten by column words [wave][N][lane]
    //   (columns c0 - 1 .. c0 + side), each wave's own words by its own;
    //   the reciprocals of the edge lengths 1 .. 2 maxd + 1;
    //   the lists of terms [wave][list_cap]
    extern __shared__ char s_dyn[];
    __shared__ int s_red[2][6];
    __shared__ unsigned long long s_sum[kRpcfT];
    __shared__ uint16_t s_late[2][kWinLate];
    const int side = MULTI ? part_side : 2 * r + 1;
    const int N = NR <= 16 ? NR : side + 2, xwords = (NR - N) * 64;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int tw = 1 << tw_log2, th = kRpcfT >> tw_log2;
    const int64_t tile = xcd_chunked(blockIdx.x, gridDim.x, chunk_log2);
    const int64_t tyi = tile / tiles_x, txi = tile - tyi * tiles_x;
    const int64_t px = (txi << tw_log2) + (t & (tw - 1)), py = tyi * th + (t >> tw_log2);
    const int64_t k = py * vw + px;
    const bool valid = px < vw && k < n;
    Addr A{};
    if (valid) A = address(gld(frags + 3 * k), gld(frags + 3 * k + 1), gld(frags + 3 * k + 2), m.W, m.H, bias);
    Word *const words = reinterpret_cast<Word *>(s_dyn);  // wave 0's row words, wave 1's, wave 0's column words
    float *const band = reinterpret_cast<float *>(words + 128 * N + xwords);
    Word *const xrows = wave == 0 ? words + 128 * N : reinterpret_cast<Word *>(band + cap);
    float *const s_rcp = reinterpret_cast<float *>(reinterpret_cast<Word *>(band + cap) + xwords);
    for (int l = t + 1; l <= 2 * maxd + 1; l += kRpcfT) s_rcp[l] = 1.0f / (float)l;

    // texel box of the tile's fragments
    {
        const int b0 = wave_min(valid ? A.i0 : INT32_MAX), b1 = wave_min(valid ? -A.i0 : INT32_MAX);
        const int b2 = wave_min(valid ? A.j0 : INT32_MAX), b3 = wave_min(valid ? -A.j0 : INT32_MAX);
        if (lane == 0) {
            s_red[wave][0] = b0;
            s_red[wave][1] = b1;
            s_red[wave][2] = b2;
            s_red[wave][3] = b3;
        }
    }
    s_sum[t] = 0ull;
    __syncthreads();
    const int b0 = __builtin_amdgcn_readfirstlane(min(s_red[0][0], s_red[1][0]));
    const int b1 = __builtin_amdgcn_readfirstlane(min(s_red[0][1], s_red[1][1]));
    const int b2 = __builtin_amdgcn_readfirstlane(min(s_red[0][2], s_red[1][2]));
    const int b3 = __builtin_amdgcn_readfirstlane(min(s_red[0][3], s_red[1][3]));
    if (b0 == INT32_MAX) return;  // no fragment in this tile (uniform)

    // the window: its part of the kernel's box at positions c0, c0 + 1, ...
    const int c0 = 1 + ((NR - (side + 2)) >> 1);
    const int64_t hw64 = (int64_t)(-b1) - b0 + NR, hh64 = (int64_t)(-b3) - b2 + NR;
    const bool staged = hw64 * hh64 <= cap;
    const int hw = (int)hw64, hh = (int)hh64;
    // this lane's words of row / column k0, k0 + 1, ...
    const int k0 = NR <= 16 ? 0 : c0 - 1;
    Word *const rw = words + wave * (64 * N) + lane, *const cw = rw + 128 * N;
    // where the word of row y of the window is until the columns are made
    auto row_at = [&](int y) -> Word * {
        const int q = y - k0;
        if (q >= 0 && q < N) return rw + q * 64;
        return xrows + lane + (q < 0 ? y : y - N) * 64;  // rows 0 .. k0 - 1, then k0 + N .. NR - 1
    };
    int lit_terms = 0, edge_terms = 0;  // of this lane
    double rest = 0.0;                  // of its listed terms, what s_sum leaves out
    // this lane's listed terms, in units of 2^-52
    auto edge_sum = [&]() -> unsigned long long {
        return s_sum[t] - (unsigned long long)edge_terms * 0x3ff0000000000000ull;
    };
    // One part of the box.  True where every lane's tests are all the same
    // (plain_lit: lit), which its terms then are.
    auto run_part = [&](int part, bool &plain_lit) -> bool {
        const int px0 = MULTI ? (part % parts) * side : 0, py0 = MULTI ? (part / parts) * side : 0;
        const int nx = MULTI ? min(side, 2 * r + 1 - px0) : side, ny = MULTI ? min(side, 2 * r + 1 - py0) : side;
        const int ox = px0 - r - c0, oy = py0 - r - c0;  // the window's first texel, from the fragment's
        const int hx = b0 + ox, hy = b2 + oy;
        if (MULTI && part > 0) __syncthreads();  // the last part's column words are read: the band overwrites them
        bool lit_all = false, dark_all = false;
        if (staged) {
            // one column per lane, rows alternating between the waves, 8 loads in flight
            float lo_t = __builtin_inff(), hi_t = -__builtin_inff();
            for (int xb = 0; xb < hw; xb += 64) {
                const int x = min(xb + lane, hw - 1);
                const int gx = clampi(hx + x, m.W);
                for (int yb = wave; yb < hh; yb += 16) {
                    float v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)  // rows past the band re-read its last one
                        v[u] = gld(m.t + (int64_t)clampi(hy + min(yb + 2 * u, hh - 1), m.H) * m.pitch + gx);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const float c = canon(v[u]);
                        lo_t = fminf(lo_t, c);
                        hi_t = fmaxf(hi_t, c);
                        if (yb + 2 * u < hh && xb + lane < hw) band[(yb + 2 * u) * hw + x] = c;
                    }
                }
            }
            // signed integers in the order of the depths
            auto ord = [](float f) {
                const int b = __float_as_int(f);
                return b ^ ((b >> 31) & 0x7fffffff);
            };
            const int tmin = wave_min(ord(lo_t)), tmax = wave_min(-ord(hi_t));
            const float z = A.zb + 0.0f;  // -0 as +0
            const int zmax = -wave_min(valid ? -ord(z) : INT32_MAX), zmin = wave_min(valid ? ord(z) : INT32_MAX);
            if (lane == 0) {
                s_red[wave][4] = tmin;
                s_red[wave][5] = tmax;
            }
            __syncthreads();
            lit_all = zmax <= min(s_red[0][4], s_red[1][4]);
            dark_all = zmin > -min(s_red[0][5], s_red[1][5]);
        } else {
            __syncthreads();
        }
        // every window of the tile inside the map
        const bool inside = hx >= 0 && hy >= 0 && hx + hw64 <= m.W && hy + hh64 <= m.H;
        // row words (bit x: texel hx + x of the row is in shadow)
        const bool done = (bool)__builtin_amdgcn_readfirstlane((int)(lit_all || dark_all));
        uint32_t any = 0u, every = kAll;
        if (!done) {
            const lds_float *line = (const lds_float *)band + (valid ? (A.j0 - b2) * hw + (A.i0 - b0) : 0);
            for (int y = 0; y < NR; ++y) {
                uint32_t w = 0u;
                float v[NR];
                if (staged) {
#pragma unroll
                    for (int x = 0; x < NR; ++x) v[x] = line[x];
                    line += hw;
                } else if (inside) {  // 16-byte loads
                    const float *row = m.t + ((int64_t)(valid ? A.j0 + oy + y : 0) * m.pitch + (valid ? A.i0 + ox : 0));
#pragma unroll
                    for (int x = 0; x < NR; x += 4) {
                        const f32x4u q = gld4u(row + x);
                        v[x] = canon(q.x);
                        v[x + 1] = canon(q.y);
                        v[x + 2] = canon(q.z);
                        v[x + 3] = canon(q.w);
                    }
                } else {
                    const int gy = clampi(A.j0 + oy + y, m.H);
                    const float *row = m.t + (int64_t)gy * m.pitch;
#pragma unroll
                    for (int x = 0; x < NR; ++x) v[x] = canon(gld(row + clampi(A.i0 + ox + x, m.W)));
                }
#pragma unroll
                for (int x = NR - 1; x >= 0; --x) w = push_bit(w, v[x], A.zb);
                any |= w;
                every &= w;
                *row_at(y) = (Word)w;
            }
        }
        __syncthreads();  // the band is free: column words overwrite it
        // every test of each lane's window the same: its mean is its own test
        const bool plain = !valid || any == 0u || every == kAll;
        if (done || __ballot(!plain) == 0ull) {
            plain_lit = done ? lit_all : any == 0u;
            if (MULTI) lit_terms += plain_lit ? nx * ny : 0;
            return true;
        }
        {
            uint32_t a[S];
#pragma unroll
            for (int y = 0; y < S; ++y) a[y] = y < NR ? (uint32_t)*row_at(y) : 0u;
            transpose_bits<S>(a);
#pragma unroll
            for (int x = 0; x < NR; ++x) {
                const int q = x - k0;
                if (q >= 0 && q < N) cw[q * 64] = (Word)a[x];
            }
        }

        const Word *const rwl = rw - lane - k0 * 64, *const cwl = cw - lane - k0 * 64;  // the wave's row, column 0
        uint16_t *const list = reinterpret_cast<uint16_t *>(s_rcp + 2 * maxd + 2) + wave * list_cap;
        uint16_t *const late = s_late[wave];
        const lds_float *const rcp = (const lds_float *)s_rcp;
        const bool map_32 = (int64_t)m.pitch * m.H <= (int64_t)(0xFFFFFFFFu / 4u);  // byte offsets fit 32 bits
        // the lowest and the highest maxd bits of a word: the steps of a traversal
        const uint32_t first = maxd < 32 ? (1u << (maxd & 31)) - 1u : ~0u;
        const uint32_t last_bits = maxd < 32 ? ~(0xffffffffu >> (maxd & 31)) : ~0u;
        // the value of listed term en = lane | x << 6 | y << 11; LATE: traversals
        // that leave the window go on in global memory, else `leaves` is set.
        // Every lane of the wave takes part (the fragments' values come by
        // cross-lane reads).
        auto term = [&](uint32_t en, auto late_tag, bool &leaves) -> float {
            constexpr bool LATE = decltype(late_tag)::value;
            const int L = en & 63u, x = (en >> 6) & 31u, y = en >> 11;
            const Word *pr = rwl + y * 64 + L, *pc = cwl + x * 64 + L;
            const uint32_t w = pr[0], wt = pr[64], wb = pr[-64];
            const uint32_t c = pc[0], cl = pc[-64], cr = pc[64];
            // all ones for a term in shadow: then bit 1 of a word means a test
            // that differs from the term's
            const uint32_t flip = (uint32_t)__builtin_amdgcn_sbfe((int)w, x, 1) & kAll;
            const uint32_t dh = w ^ flip, dt = wt ^ flip, db = wb ^ flip, dv = c ^ flip, dl = cl ^ flip, dr = cr ^ flip;
            // a step goes on where its texel's test is the term's and that of a
            // side neighbour shared with the term's mask (Eq. 3) is not
            const uint32_t mt = (uint32_t)__builtin_amdgcn_sbfe((int)dt, x, 1);
            const uint32_t mb = (uint32_t)__builtin_amdgcn_sbfe((int)db, x, 1);
            const uint32_t ml = (uint32_t)__builtin_amdgcn_sbfe((int)dl, y, 1);
            const uint32_t mr = (uint32_t)__builtin_amdgcn_sbfe((int)dr, y, 1);
            const uint32_t gh = ~dh & ((dt & mt) | (db & mb)), gv = ~dv & ((dl & ml) | (dr & mr));
            bool leave[4];
            auto up = [&](uint32_t go, uint32_t d, int p, bool &lv) {
                WalkEnd e;
                e.go = __builtin_ctz(~((go >> (p + 1)) & first));
                e.end = __builtin_amdgcn_ubfe((d >> (p + 1)) & first, e.go, 1);
                lv = p + e.go >= NR - 1 && e.go < maxd;
                return e;
            };
            auto down = [&](uint32_t go, uint32_t d, int p, bool &lv) {
                WalkEnd e;
                e.go = __builtin_clz(~((go << (32 - p)) & last_bits));
                e.end = (((d << (32 - p)) & last_bits) << e.go) >> 31;
                lv = e.go >= p && e.go < maxd;
                return e;
            };
            WalkEnd e0 = down(gh, dh, x, leave[0]), e1 = up(gh, dh, x, leave[1]);  // left, right
            WalkEnd e2 = down(gv, dv, y, leave[2]), e3 = up(gv, dv, y, leave[3]);  // bottom, top
            const bool s = flip == 0u;
            if (!LATE) {
                leaves = leave[0] | leave[1] | leave[2] | leave[3];
            } else {
                const int i = __shfl(A.i0, L) + ox + x, j = __shfl(A.j0, L) + oy + y;
                const float zb = __shfl(A.zb, L);
                uint32_t dirs = (leave[0] ? 1u : 0u) | (leave[1] ? 2u : 0u) |
                                (leave[2] ? 4u : 0u) | (leave[3] ? 8u : 0u);
                while (dirs != 0u) {  // each lane its next direction
                    const int dir = __builtin_ctz(dirs);
                    dirs &= dirs - 1u;
                    const bool horiz = dir < 2;
                    const int d = (dir & 1) ? 1 : -1, p0 = horiz ? i : j, pmax = (horiz ? m.W : m.H) - 1;
                    const bool ca = (horiz ? mt : ml) != 0u, cb = (horiz ? mb : mr) != 0u;
                    // the step that was found is the first outside the window
                    const int k1 = 1 + (dir == 0 ? e0.go : dir == 1 ? e1.go : dir == 2 ? e2.go : e3.go);
                    int q;
                    if (map_32) {
                        const unsigned pitch4 = 4u * (unsigned)m.pitch, fmul = horiz ? pitch4 : 4u;
                        const int f = horiz ? j : i, fa = horiz ? j + 1 : i - 1, fb = horiz ? j - 1 : i + 1;
                        const int nf = horiz ? m.H : m.W;
                        const GlobalWalkReader g{(const char *)m.t, (unsigned)clampi(f, nf) * fmul,
                                                 (unsigned)clampi(fa, nf) * fmul, (unsigned)clampi(fb, nf) * fmul,
                                                 horiz ? 4u : pitch4};
                        q = walk_range<4>(g, k1, maxd, p0, d, pmax, zb, s, ca, cb);
                    } else {
                        const MapLineReader g{m, horiz ? j : i, horiz ? j + 1 : i - 1, horiz ? j - 1 : i + 1, horiz};
                        q = walk_range<4>(g, k1, maxd, p0, d, pmax, zb, s, ca, cb);
                    }
                    const WalkEnd e{q == 0 ? maxd : abs(q) - 1, q > 0 ? 1u : 0u};
                    if (dir == 0) e0 = e;
                    if (dir == 1) e1 = e;
                    if (dir == 2) e2 = e;
                    if (dir == 3) e3 = e;
                }
            }
            const float tx = win_axis(e0, e1, __shfl(A.fx, L), rcp), ty = win_axis(e2, e3, __shfl(A.fy, L), rcp);
            const float v = s ? (ty + tx) : ((1.0f - ty) - tx);
            const float at0 = v > 0.0f ? v : 0.0f;
            return at0 < 1.0f ? at0 : 1.0f;
    };
        auto add = [&](uint32_t en, float v) {
            atomicAdd(&s_sum[wave * 64 + (en & 63u)], (unsigned long long)__double_as_longlong(1.0 + (double)v));
        };
        // a small term, not 0: s_sum rounds it
        auto is_small = [&](float v) { return __float_as_uint(v) - 1u < __float_as_uint(kWinSmall) - 1u; };
        // what was rounded off goes to the fragments' lanes, one term (a bit of `which`) at a time
        auto add_small = [&](uint32_t en, float v, unsigned long long which) {
            for (; which != 0ull; which &= which - 1ull) {
                const int from = __builtin_ctzll(which);
                const double x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), from));
                if (lane == (__builtin_amdgcn_readlane((int)en, from) & 63)) rest += x - ((1.0 + x) - 1.0);
            }
        };

        const uint32_t range = valid ? ((2u << (nx - 1)) - 1u) << c0 : 0u;  // the part's columns
        const int y1 = c0 + ny - 1;
        int listed = 0, n_late = 0;         // of the wave
        int y = c0 - 1;
        // rows y - 1, y, y + 1 and (on its way) y + 2
        uint32_t wm = 0u, w = rw[(y - k0) * 64], wp = rw[(y - k0 + 1) * 64], wn = rw[(y - k0 + 2) * 64], bits = 0u;
        auto below = [&](unsigned long long has) -> int {
            return __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
    };
        bool last = false;
        while (!last) {
            // list terms, each lane its next one, until a batch waits or the rows
            // are through
            do {
                if (__ballot(bits != 0u) == 0ull) {
                    if (y == y1) {
                        last = true;
                        break;
                    }
                    ++y;
                    wm = w;
                    w = wp;
                    wp = wn;
                    wn = rw[min(y + 2 - k0, N - 1) * 64];
                    bits = ((w ^ (w << 1)) | (w ^ (w >> 1)) | (w ^ wm) | (w ^ wp)) & range;
                    lit_terms += __builtin_popcount(~(bits | w) & range);
                    edge_terms += __builtin_popcount(bits);
                }
                const unsigned long long has = __ballot(bits != 0u);
                const uint32_t row = (uint32_t)lane | (uint32_t)y << 11;
                if (bits != 0u) list[listed + below(has)] = (uint16_t)(row | (uint32_t)__builtin_ctz(bits) << 6);
                listed += __builtin_popcountll(has);
                bits &= bits - 1u;
            } while (listed <= list_cap - 64);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            // evaluate the full waves of terms (at the end: all of them)
            const int todo = last ? listed : listed & ~63;
            for (int e = 0; e < todo || (last && n_late > 0); e += 64) {
                const bool on = e + lane < todo;
                const uint32_t en = on ? list[e + lane] : (uint32_t)c0 * 0x840u;  // idle lanes: row and column c0
                bool leaves = false;
                const float v = term(en, std::false_type{}, leaves);
                leaves = leaves && on;
                if (on && !leaves) add(en, v);
                // (the ballots of bools stay scalar masks; __ballot goes through an int)
                const unsigned long long lv = __builtin_amdgcn_ballot_w64(leaves);
                const unsigned long long sm = __builtin_amdgcn_ballot_w64(is_small(v));
                if ((lv | sm) != 0ull) {
                    if (leaves) late[n_late + below(lv)] = (uint16_t)en;
                    n_late += __builtin_popcountll(lv);
                    add_small(en, v, sm & ~lv & __builtin_amdgcn_ballot_w64(on));
                }
                // the terms that left the window, a full wave of them at a time
                while (n_late >= 64 || (last && e + 64 >= todo && n_late > 0)) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    // the newest ones, so that none is moved
                    const int from = max(n_late - 64, 0);
                    const bool lon = from + lane < n_late;
                    const uint32_t el = late[lon ? from + lane : 0];
                    bool unused;
                    const float lval = term(el, std::true_type{}, unused);
                    if (lon) add(el, lval);
                    add_small(el, lval, __ballot(lon && is_small(lval)));
                    n_late = from;
                }
            }
            const int left = listed - todo;
            const uint16_t keep = lane < left ? list[todo + lane] : (uint16_t)0;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < left) list[lane] = keep;
            listed = left;
        }
        if (MULTI) {
            // the whole part of the sum joins the lit terms: up to 65^2 terms of
            // value 1 do not fit 64 bits at 2^-52, those of one part (at most
            // kWinPart^2) and a remainder below 1 do
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const unsigned long long sum = edge_sum();
            lit_terms += (int)(sum >> 52);
            s_sum[t] = sum & ((1ull << 52) - 1ull);
            edge_terms = 0;
        }
        return false;
    };
    bool plain_lit = false;
    if (MULTI) {
        for (int part = 0; part < parts * parts; ++part) (void)run_part(part, plain_lit);
    } else if (run_part(0, plain_lit)) {
        if (valid) out[k] = plain_lit ? 1.0f : 0.0f;
        return;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (valid) {
        const double acc = (double)lit_terms + ((double)edge_sum() * 0x1p-52 + rest);
        out[k] = (float)(acc / (double)((2 * r + 1) * (2 * r + 1)));
    }
}

// Launch of the window kernel: a band for a tile whose texel footprint spans up
// to 17 x 17 texels (the column words' room where that is more), tiles dealt
// to the XCDs in chunks of 32 (their cost varies with the edges; contiguous
// ranges left XCDs idle: 4K r = 5 5-7% slower).  The list of terms is the
// longest of 128, 192, .. 512 with which a CU still holds as many workgroups as
// with the shortest (longer lists are evaluated in fewer, fuller batches).  It
// follows the radius' words and, by the reciprocals, MAXDIST.  Against 192 for
// most radii, where r = 21 and 32 lost a workgroup: 720p r = 21 1136 -> 1063 us,
// r = 32 2018 -> 1903, r = 5, 9, 12 and 18 1 to 2% less.
template <int NR, bool MULTI>
void launch_window(const MapView &mv, const float *frags, int64_t n, int64_t view_width, float bias, int maxd, int r,
                   int parts, float *out, hipStream_t stream) {
    using Word = typename WinWord<NR>::T;
    const int side = (2 * r + parts) / parts;  // terms a side of a part
    const int N = NR <= 16 ? NR : side + 2;
    const int words = 2 * N * 64 * (int)sizeof(Word), extra = (NR - N) * 64 * (int)sizeof(Word);  // bytes
    const int band = std::max(words - 2 * extra, (NR + 16) * (NR + 16) * 4);
    const int fixed = words + 2 * extra + band + 4 * (2 * maxd + 2);  // bytes beside the lists
    constexpr int kCuLds = 160 * 1024, kLdsUnit = 1280;               // of a CU; what it is given out in
    constexpr int kStatic = 2 * 6 * 4 + kRpcfT * 8 + 2 * kWinLate * 2;
    constexpr int kMost = 2 * kWinWaves<NR, MULTI>;                   // workgroups the registers leave room for
    auto groups = [&](int list) {
        const int units = (fixed + 2 * 2 * list + kStatic + kLdsUnit - 1) / kLdsUnit;
        return std::min(kMost, kCuLds / (units * kLdsUnit));
    };
    int list = 128;
    while (list < 512 && groups(list + 64) == groups(128)) list += 64;
    const size_t lds = (size_t)(fixed + 2 * 2 * list);
    const int64_t vw = view_width > 0 ? view_width : n;
    const int tw_log2 = view_width > 0 ? 4 : 7;  // 16 x 8 pixels, or 128 consecutive fragments
    const int th = kRpcfT >> tw_log2;
    const int64_t tiles_x = (vw + (1 << tw_log2) - 1) >> tw_log2;
    const int64_t tiles = tiles_x * (((n + vw - 1) / vw + th - 1) / th);
    constexpr int kChunkLog2 = 5;
    hipLaunchKernelGGL((rpcf_window_kernel<NR, MULTI>), dim3((unsigned)tiles), dim3(kRpcfT), lds, stream, mv, frags, n,
                       vw, tiles_x, tw_log2, bias, maxd, r, parts, side, band / 4, list, kChunkLog2, out);
}

// The window is 2r+3 rounded up to a multiple of 4 (of 2 measured slower up
// to r = 6: fewer tests, but more traversals leave it).  Beyond r = 14 the box
// goes in parts of at most 22 x 22 terms, whose 24 x 24 windows leave LDS for
// 6 workgroups per CU; parts of 30 terms (32 x 32 windows) leave it for 4.
// Parts of at most 18 terms a side (r = 15..17 in two, 22..26 in three) take 20
// x 20 windows, which test 30% fewer texels and leave LDS for 7 or 8: 720p r =
// 15 787 -> 709 us, r = 22 1421 -> 1178 (24 x 24 at 4 waves per SIMD before).
inline void launch_rpcf(const MapView &mv, const float *frags, int64_t n, int64_t view_width, float bias, int maxd,
                        int r, float *out, hipStream_t stream) {
    if (r > kWinMaxR) {
        const int parts = (2 * r + kWinPart) / kWinPart;  // of 2r+1 terms
        if ((2 * r + parts) / parts <= 18)
            launch_window<20, true>(mv, frags, n, view_width, bias, maxd, r, parts, out, stream);
        else
            launch_window<24, true>(mv, frags, n, view_width, bias, maxd, r, parts, out, stream);
        return;
    }
    switch ((2 * r + 3 + 3) & ~3) {
        case 8: launch_window<8, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
        case 12: launch_window<12, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
        case 16: launch_window<16, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
        case 20: launch_window<20, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
        case 24: launch_window<24, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
        case 28: launch_window<28, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
        default: launch_window<32, false>(mv, frags, n, view_width, bias, maxd, r, 1, out, stream); break;
    }
}

}  // namespace rbsm
