// Realistic gap currents of all-to-all networks from a grid of voltages.
//
// With one weight g the gap current of every cell is the same function of its
// own voltage (Section 2.3.1, Algorithm 1):
//   I(v) = g (0.8 F(v) + 0.2 (n v - sum_j v_j)),
//   F(v) = sum_j (v - v_j) exp(-(v - v_j)^2 / 100).
// F is a sum of Gaussians of 10 mV width, so its values at whole millivolts
// determine it: between two of them it is interpolated from the twelve
// nearest (the Lagrange polynomial of degree 11), with an error below
// 8e-10 mV per sending cell, a thousandth of the rounding of one voltage
// difference of fp32 voltages near -60 mV. Sums over the cells are then needed
// at the grid points near the cells' voltages only (12 + the spread in mV)
// instead of at every cell: n (12 + spread) terms instead of n^2. Everything
// on the way is in fp64: near synchrony F at the cells is a small difference
// of the large values around them.
//
// Grid points are taken in groups of kGridGroup = 16. For a sending cell v and
// a group starting at t0, with d = t0 - v,
//   exp(-(d + k)^2 / 100) = exp(-d^2 / 100) * exp(-d / 50)^k * exp(-k^2 / 100):
// two exponentials per cell and group, then a multiplication, an addition and
// a fused multiply-add per grid point; the last factor is taken once per sum.
//
// Measured per step against every unordered pair once (or, in the batch, every
// ordered pair): 16,384 cells 39.8 -> 12.3 us (k_grid_sums 4.5 of it), 8,192
// 18.7 -> 11.6, 40,000 178 -> 14.7, a batch of 256 networks of 64-2,048 cells
// a third of them all-to-all 75.8 -> 54.4. With voltages over 150 mV 5,000 cells
// 14.0 -> 15.7, 16,384 41 -> 17.4; over 250 mV 18.9 and 21.1; 2,000 cells (their
// pairs then) 13.7 -> 14.5; with some beyond the grid ahead (every pair, ordered,
// one workgroup for 64 rows up to 16,384 cells, for 256 above) 5,000 cells 34,
// 16,384 90, 40,000 780. What remains is latency: two
// launches, and in each a chain of loads, fp64 exponentials and exchanges
// between lanes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace infoli {

// All-to-all networks from this size on (library choice). Below it the pairs
// of a 64-row tile are fewer than the sums' overhead: lone networks of 256 /
// 400 / 777 cells took 6.0 / 6.9 / 8.9 us per step with every pair, 6.4 / 6.8 /
// 7.9 on the grid.
constexpr int kGridCells = 512;
constexpr int kGridQ = 12;              // grid points of one interpolation
constexpr int kGridLeft = 5;            // of them below floor(v)
constexpr int kGridGroup = 16;          // grid points per group
constexpr int kGridMaxGroups = 12;      // groups of a tile's own sums, or a workgroup's of the persistent
                                        // kernel (voltages up to 180 mV apart)
constexpr int kGridAheadLo = -160;      // k_grid_sums: first grid point (mV)
constexpr int kGridAheadGroups = 20;    //   and groups: up to 159 mV
constexpr double kGridReach = 64.0;     // k_grid_sums skips a group farther than this from a cell:
                                        // every term beyond is below 56 exp(-31) = 1.4e-12 mV
constexpr int kGridChunks = 128;        // k_grid_sums: workgroups (shares of the cells), at most

__host__ __device__ constexpr int grid_per(int n) {      // cells per share, whole waves
    return n <= 64 * kGridChunks ? 64 : ((n + kGridChunks - 1) / kGridChunks + 63) / 64 * 64;
}
__host__ __device__ constexpr int grid_chunks(int n) { return (n + grid_per(n) - 1) / grid_per(n); }
// floats of a network's partial sums: [groups][chunks][16] doubles, then each
// share's voltage sum
__host__ __device__ constexpr int64_t grid_floats(int n) {
    return (2 * (int64_t)grid_chunks(n) * (kGridAheadGroups * kGridGroup + 1) + 63) / 64 * 64;
}
// doubles of LDS of a tile: the waves' sums, then the grid (room for all of
// k_grid_sums' groups, one constant for both kinds of tiles: with two a batch of
// 256 networks took 1 % longer)
__host__ __device__ constexpr int grid_lds_doubles(int waves) { return (waves + 1) * kGridAheadGroups * kGridGroup; }
// Groups a tile of so many rows sums itself at most; where its voltages need more
// it takes its pairs. One row per lane (600 cells: 7.0 us a step with one group,
// 9.4 with three, 8.4 with all pairs; 2,000: 9.4, 14.2, 14.6): two. More rows,
// where the chip is full of such tiles (64 networks of 2,048 cells: eleven groups
// 55 us, all pairs 73; 1,000 cells 25 and 27): three for each 64.
__host__ __device__ constexpr int grid_tile_groups(int rows) { return rows <= 64 ? 2 : 3 * ((rows + 63) / 64); }
static_assert(grid_tile_groups(256) <= kGridMaxGroups, "a tile of 256 rows");

// e^x to about 1e-13 for |x| below a few thousand (0 or infinity beyond the
// range of fp64): x = n ln 2 + r, |r| <= ln 2 / 2, the Taylor series of e^r to
// r^10 (the next term is below 3e-13), scaled by 2^n.
__device__ __forceinline__ double grid_exp(double x) {
    const double n = rint(x * 1.4426950408889634074);
    const double r = fma(n, -0.69314718055994530942, x);
    double p = 1.0 / 3628800.0;
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)n);
}

// Adds cell v's terms at the group's grid points t0, t0 + 1, .. (without the
// factor exp(-k^2 / 100)). Distances beyond 400 mV are taken as 400 in the
// exponentials (which vanish there), so that a far finite voltage adds zeros
// and an infinite or NaN one NaNs, as its terms would.
__device__ __forceinline__ void grid_add(double (&acc)[kGridGroup], double t0, float v) {
    const double d = t0 - (double)v;
    const double c = d > 400.0 ? 400.0 : d < -400.0 ? -400.0 : d;
    double p = grid_exp(c * c * -0.01);
    const double r = grid_exp(c * -0.02);
    double dk = d;
#pragma unroll
    for (int k = 0; k < kGridGroup; ++k) {
        acc[k] = fma(dk, p, acc[k]);
        p *= r;
        dk += 1.0;
    }
}

// Exchanges within the 16 lanes of a row by DPP, without a trip through LDS.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor7 = 0x141, kDppXor8 = 0x128;
template <int CTRL>
__device__ __forceinline__ float dpp_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_lane(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// op over the 64 lanes, the same in each (op: +, min or max)
template <typename T, typename F>
__device__ __forceinline__ T grid_wave(T v, F&& op) {
    v = op(v, dpp_lane<kDppXor1>(v));
    v = op(v, dpp_lane<kDppXor2>(v));
    v = op(v, dpp_lane<kDppXor7>(v));
    v = op(v, dpp_lane<kDppXor8>(v));
    v = op(v, __shfl_xor(v, 16, 64));
    return op(v, __shfl_xor(v, 32, 64));
}

// Sum over the 64 lanes: lane l ends with point (l & 15)'s sum (four exchanges
// that halve the points a lane holds, each with a lane whose bit H differs and
// whose higher bits below 16 do not, then two that add the four groups of
// sixteen lanes).
template <int H>
__device__ __forceinline__ void grid_halve(double (&v)[kGridGroup], int lane) {
    constexpr int ctrl = H == 8 ? kDppXor8 : H == 4 ? kDppXor7 : H == 2 ? kDppXor2 : kDppXor1;
    const bool hi = (lane & H) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double send = hi ? v[i] : v[i + H];
        const double keep = hi ? v[i + H] : v[i];
        v[i] = keep + dpp_lane<ctrl>(send);
    }
}
__device__ __forceinline__ double grid_lane_sum(double (&acc)[kGridGroup], int lane) {
    grid_halve<8>(acc, lane);
    grid_halve<4>(acc, lane);
    grid_halve<2>(acc, lane);
    grid_halve<1>(acc, lane);
    double s = acc[0];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    return s;
}

// F(v) from the grid values f[i] at the points lo + i.
__device__ __forceinline__ double grid_value(const double* f, int lo, float v) {
    const float fl = floorf(v);
    const double s = (double)(v - fl);               // in [0, 1), exact
    const double* q = f + ((int)fl - kGridLeft - lo);
    // weight m: prod_{j != m} (s + kGridLeft - j) / (m - j), the products of the
    // factors before and after m, the denominators (-1)^(11 - m) m! (11 - m)!
    constexpr double inv[kGridQ] = {-1.0 / 39916800, 1.0 / 3628800,  -1.0 / 725760, 1.0 / 241920,
                                    -1.0 / 120960,   1.0 / 86400,    -1.0 / 86400,  1.0 / 120960,
                                    -1.0 / 241920,   1.0 / 725760,   -1.0 / 3628800, 1.0 / 39916800};
    double after[kGridQ];
    after[kGridQ - 1] = 1.0;
#pragma unroll
    for (int m = kGridQ - 1; m > 0; --m) after[m - 1] = after[m] * (s + (double)(kGridLeft - m));
    double before = 1.0, sum = 0.0;
#pragma unroll
    for (int m = 0; m < kGridQ; ++m) {
        sum = fma(q[m], before * after[m] * inv[m], sum);
        before *= s + (double)(kGridLeft - m);
    }
    return sum;
}

// Partial sums of a large network's grid, ahead of its step: one workgroup per
// share of the cells, wave w taking groups w, w + 8, ..; a group no cell of the
// share reaches is zero. P: [group][share][16] sums, then the shares' voltage
// sums.
static __global__ __launch_bounds__(512) void k_grid_sums(const float* __restrict__ vd, int n,
                                                          double* __restrict__ P) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = grid_per(n), C = grid_chunks(n), c = blockIdx.x;
    const int j0 = c * per, j1 = min(n, j0 + per);
    const double ck = grid_exp((double)((lane & 15) * (lane & 15)) * -0.01);
    for (int g = wave; g < kGridAheadGroups; g += 8) {
        const double t0 = kGridAheadLo + g * kGridGroup;
        double acc[kGridGroup];
#pragma unroll
        for (int k = 0; k < kGridGroup; ++k) acc[k] = 0.0;
        bool any = false;
        float v = j0 + lane < j1 ? vd[j0 + lane] : 0.0f;
        for (int j = j0 + lane; j - lane < j1; j += 64) {
            const float next = j + 64 < j1 ? vd[j + 64] : 0.0f;
            const float dist = fabsf((float)(t0 + 7.5) - v);
            if (__any(j < j1 && !(dist >= (float)kGridReach && dist <= 3.0e38f))) {
                any = true;
                if (j < j1) grid_add(acc, t0, v);
            }
            v = next;
        }
        const double s = any ? grid_lane_sum(acc, lane) * ck : 0.0;
        if (lane < kGridGroup) P[((int64_t)g * C + c) * kGridGroup + lane] = s;
    }
    if (wave == 7) {
        double s = 0.0;
        for (int j = j0 + lane; j < j1; j += 64) s += (double)vd[j];
        s = grid_wave(s, [](double x, double y) { return x + y; });
        if (lane == 0) P[(int64_t)kGridAheadGroups * C * kGridGroup + c] = s;
    }
}

}  // namespace infoli
