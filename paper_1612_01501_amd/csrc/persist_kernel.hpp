// Many steps of small networks in one launch: one workgroup owns one whole
// network (up to kPersistCells cells), keeps its cells' state in registers
// across steps and exchanges the voltages through a double buffer in LDS. The
// workgroup barrier at the end of each step is the step barrier of Section 2.2
// (step n+1 sees only step-n voltages); no cross-workgroup synchronisation
// exists, so every workgroup always runs to completion. Dry runs (timing)
// write the final state only: no spikes, outputs or flags.
//
// A step is one compute unit's work: n^2 pair terms of nine issue slots and 370
// slots a cell, which at 96 cells are 0.55 and 0.3 us of its 64 lanes. Up to
// kPersistSplit cells (SPLIT) the sixteen waves take parts, so that the parts'
// latencies overlap: dendrite, soma and axon of the cells in waves of their
// own, the pair terms in the others, a row's terms split over several threads
// and added in a fixed order; only the dendrite's voltage waits for them.
// Larger networks give a thread per cell, with all threads sharing the gap
// currents first (all-to-all: sums on the voltage grid, gap_grid.hpp, or every
// pair where the caller asks for pairs).
// Measured per step against 256 threads that each walked whole rows: 96 cells
// all-to-all 2.75 -> 1.32 us, 192 4.58 -> 2.91, 200 (grid) 4.67 -> 3.84, 1,000
// 8.74 -> 7.08; 100 cells with 25 connections each 4.63 -> 2.22; 1,000 uncoupled
// cells 3.51 -> 2.12. Where a launch has more networks than the chip compute
// units, and they are small, 256 threads take one (a thread per cell or two), so
// that a unit holds several: their registers stay at four waves per SIMD and a
// launch of one form, or without networks for the grid, compiles no more
// (1,024 networks of 64 to 192 cells of three forms: 11.6 us with 1,024 threads,
// 8.9 with 256, 8.4 as whole rows per thread).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cell_model.hpp"
#include "step_kernel.hpp"

namespace infoli {

constexpr int kPersistBlock = 1024;
constexpr int kPersistMaxCpt = 2;                               // cells per thread
constexpr int kPersistCells = kPersistBlock * kPersistMaxCpt;   // 2048
constexpr int kPersistSmall = 256;                              // threads where compute units hold several networks
constexpr int kPersistSplit = 192;                              // cells of a split network: three waves a part
constexpr int kPersistParts = 12;                               // threads per row of its pair terms, at most
constexpr int kPersistPulses = 64;                              // pulses per network

// What the networks of a launch couple by: a launch compiles its form only, one of
// several forms takes kFormAny. Pairs without the grid are forms of their own
// (the caller's choice, or no network past a split one's cells): their code beside
// the grid's cost a step on the grid 0.2 us (200 cells 3.55 -> 3.78).
enum : int {
    kFormNone = 0,      // no gap junctions, or the simplified all-to-all closed form
    kFormPairs = 1,     // realistic all-to-all
    kFormRows = 2,      // CSR rows or a dense weight matrix
    kFormAny = 3,
    kFormOrdered = 4    // added to kFormPairs or kFormAny: pairs only, no grid
};

// Gap current of row r from the voltages v in LDS, its terms shared by `parts`
// threads (this one's: every parts-th connection from `sub` on): all-to-all,
// explicit weights or CSR rows; unscaled by g.
template <int FORM>
__device__ __forceinline__ float persist_row(const StepArgs& a, const InstDesc& d, const float* v, int r, int sub,
                                             int parts) {
    const int n = d.n;
    const float vi = v[r];
    float acc0 = 0.0f, acc1 = 0.0f;
    if ((FORM & kFormRows) && d.conn == CONN_CSR) {
        const int64_t* rp = a.row_ptr + d.rp_off;
        const int64_t e = rp[r + 1];
        const uint16_t* c16 = a.col16 + d.w_off;
        const int32_t* c32 = a.col + d.w_off;
        const float* wv = a.w + d.w_off;
        constexpr int U = 4;      // connections in flight
        for (int64_t k = rp[r] + sub; k < e; k += U * parts) {
            int j[U];
            float w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = k + u * parts;
                const bool ok = q < e;
                j[u] = !ok ? r : d.col16 ? (int)c16[q] : c32[q];      // (the row itself: a zero term)
                w[u] = ok && d.has_w ? wv[q] : 1.0f;
            }
#pragma unroll
            for (int u = 0; u < U; u += 2) {
                const float d0 = vi - v[j[u]], d1 = vi - v[j[u + 1]];
                acc0 = fmaf(w[u], d.sgj ? d0 : d0 * gap_factor(d0), acc0);
                acc1 = fmaf(w[u + 1], d.sgj ? d1 : d1 * gap_factor(d1), acc1);
            }
        }
    } else if ((FORM & kFormRows) && d.conn == CONN_DENSE) {
        const float* wr = a.w + d.w_off + (int64_t)r * n;
        for (int j = sub; j < n; j += parts) {
            const float dv = vi - v[j];
            acc0 = fmaf(wr[j], d.sgj ? dv : dv * gap_factor(dv), acc0);
        }
    } else if (FORM & kFormPairs) {
        // a consecutive share, a multiple of four cells, read four at a time
        // (the lanes of a wave mostly share theirs), the last ones singly
        const int len = ((n + parts - 1) / parts + 3) & ~3;
        const int j1 = min(n, (sub + 1) * len);
        int j = sub * len;
        for (; j + 4 <= j1; j += 4) {
            const float4 u = *reinterpret_cast<const float4*>(v + j);
            const float d0 = vi - u.x, d1 = vi - u.y, d2 = vi - u.z, d3 = vi - u.w;
            acc0 = fmaf(d0, gap_factor(d0), acc0);
            acc1 = fmaf(d1, gap_factor(d1), acc1);
            acc0 = fmaf(d2, gap_factor(d2), acc0);
            acc1 = fmaf(d3, gap_factor(d3), acc1);
        }
        for (; j < j1; ++j) {
            const float dv = vi - v[j];
            acc0 = fmaf(dv, gap_factor(dv), acc0);
        }
    }
    return acc0 + acc1;
}

template <int BLOCK, int CPT, bool SPLIT, int FORM>
__global__ __launch_bounds__(BLOCK, 4) void k_persist(StepArgs a, const float* __restrict__ xin,
                                                           float* __restrict__ xout, int64_t step0,
                                                           int64_t n_steps) {
    constexpr int CELLS = SPLIT ? kPersistSplit : BLOCK * CPT;
    constexpr int W = BLOCK / 64;
    constexpr int GP = kGridMaxGroups * kGridGroup;
    __shared__ __align__(16) float s_v[2][3][CELLS];              // Vd, Vs, Va of the current and the next step
    __shared__ float s_ig[SPLIT ? kPersistParts * CELLS : CELLS];   // (split: the parts' sums)
    __shared__ DevPulse s_pulse[kPersistPulses];
    __shared__ double s_red[W];
    __shared__ float s_mm[3][W];
    __shared__ double s_g[!SPLIT && (FORM & kFormPairs) && !(FORM & kFormOrdered) ? (W + 1) * GP : 1];
    const InstDesc& d = a.inst[blockIdx.x];
    const int n = d.n;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr bool uniform = (FORM & kFormAny) == kFormPairs, any = (FORM & kFormAny) == kFormAny;
    constexpr bool grids = !SPLIT && (FORM & kFormPairs) && !(FORM & kFormOrdered);
    const int conn = uniform ? CONN_UNIFORM : d.conn;
    const bool sgj = uniform ? false : (bool)d.sgj;
    const float g = d.g;
    const bool summed = (FORM == kFormNone || any) && conn == CONN_UNIFORM && sgj;   // the closed form g (n Vd_i - sum_j Vd_j)
    const bool grid = grids && (uniform || (conn == CONN_UNIFORM && !sgj && !d.pairs && n > kPersistSplit));
    const float scale = conn == CONN_DENSE || (conn == CONN_CSR && d.has_w) ? 1.0f : g;
    const int n_pulses = d.n_pulses;
    const CellParams p = d.p;
    const float dt = a.dt;

    // split: waves [0, nw) dendrites, [nw, 2 nw) somas, [2 nw, 3 nw) axons, the
    // others pair terms; else every thread whole cells
    const int nw = (n + 63) / 64;
    const int role = SPLIT ? wave / nw : 0;
    const bool dend = SPLIT ? role == 0 : true, soma = SPLIT ? role == 1 : true, axon = SPLIT ? role == 2 : true;
    const int gap_t = SPLIT ? tid - 3 * nw * 64 : tid;            // thread of the gap work (< 0: none)
    const int gap_n = SPLIT ? BLOCK - 3 * nw * 64 : BLOCK;
    // threads per row of the pair terms; consecutive threads for the rows read
    // from memory, consecutive rows where the lanes share the cells they read
    const bool by_row = ((FORM & kFormRows) && (conn == CONN_CSR || conn == CONN_DENSE)) ||
                        (!SPLIT && (FORM & kFormPairs) && !(uniform && grids) && conn == CONN_UNIFORM && !sgj && !grid);
    int parts = 1;
    if (SPLIT && !by_row) parts = min(kPersistParts, max(1, gap_n / n));
    else if (by_row)
        while (2 * parts * n <= gap_n && parts < (SPLIT ? 8 : 64)) parts *= 2;
    const int lparts = 31 - __builtin_clz(parts);                 // (by_row: a power of two)

    float x[CPT][NSV], bias[CPT];
    int cell_i[CPT], count[CPT];
#pragma unroll
    for (int m = 0; m < CPT; ++m) {
        const int li = SPLIT ? (role < 3 ? tid - role * nw * 64 : n) : tid + m * BLOCK;
        cell_i[m] = li;
        bias[m] = 0.0f;
        count[m] = 0;
#pragma unroll
        for (int v = 0; v < NSV; ++v) x[m][v] = 0.0f;
        if (li < n) {
            const int64_t cell = d.cell_off + li;
#pragma unroll
            for (int v = 0; v < NSV; ++v) x[m][v] = xin[v * a.stride + cell];
            bias[m] = a.bias[cell];
            if (axon) count[m] = a.spike_count[cell];
            if (dend) s_v[0][0][li] = x[m][SV_VD];
            if (soma) s_v[0][1][li] = x[m][SV_VS];
            if (axon) s_v[0][2][li] = x[m][SV_VA];
        }
    }
    for (int k = tid; k < n_pulses; k += BLOCK) s_pulse[k] = a.pulses[d.pulse_off + k];
    __syncthreads();
    int64_t slot = a.out_slots ? step0 % a.out_slots : 0;
    const int64_t stream_steps = d.stream_off >= 0 ? d.stream_steps : 0;
    const float* stream = a.i_stream + d.stream_off;

    for (int64_t s = 0; s < n_steps; ++s) {
        const int64_t step = step0 + s;
        const float(*cur)[CELLS] = s_v[s & 1];
        float(*nxt)[CELLS] = s_v[(s + 1) & 1];
        const float* vd = cur[0];

        // gap currents from the step-n voltages
        float ig[CPT];
        if (SPLIT) {
            if (FORM != kFormNone && gap_t >= 0 && conn != CONN_NONE && !summed) {
                if (by_row) {
                    const int r = gap_t >> lparts, sub = gap_t & (parts - 1);
                    if (r < n) s_ig[sub * CELLS + r] = persist_row<FORM>(a, d, vd, r, sub, parts);
                } else if (gap_t < parts * n) {
                    const int sub = gap_t / n, r = gap_t - sub * n;
                    s_ig[sub * CELLS + r] = persist_row<FORM>(a, d, vd, r, sub, parts);
                }
            }
        } else if (by_row) {
            for (int r = gap_t >> lparts; r < ((n + (gap_n >> lparts) - 1) / (gap_n >> lparts)) * (gap_n >> lparts);
                 r += gap_n >> lparts) {
                float t = r < n ? persist_row<FORM>(a, d, vd, r, gap_t & (parts - 1), parts) : 0.0f;
                for (int h = parts >> 1; h > 0; h >>= 1) t += __shfl_xor(t, h, 64);
                if (r < n && (gap_t & (parts - 1)) == 0) s_ig[r] = t;
            }
        }
        double tot = 0.0;
        if (summed && (!SPLIT || wave == W - 1)) {
            // the sum in fp64 in a fixed order (split: by the last wave)
            double t = 0.0;
            for (int j = SPLIT ? lane : tid; j < n; j += SPLIT ? 64 : BLOCK) t += (double)vd[j];
            t = grid_wave(t, [](double x, double y) { return x + y; });
            if (lane == 0) s_red[SPLIT ? 0 : wave] = t;
        }
        if (grid) {
            // sums at the grid points around the cells' voltages (as a tile's)
            float lo = vd[0], hi = lo;
            bool bad = false;
#pragma unroll
            for (int m = 0; m < CPT; ++m)
                if (cell_i[m] < n) {
                    const float v = x[m][SV_VD];
                    lo = fminf(lo, v);
                    hi = fmaxf(hi, v);
                    bad = bad || !(fabsf(v) <= 1.0e6f);
                }
            lo = grid_wave(lo, [](float x, float y) { return fminf(x, y); });
            hi = grid_wave(hi, [](float x, float y) { return fmaxf(x, y); });
            bad = __any(bad);
            if (lane == 0) {
                s_mm[0][wave] = lo;
                s_mm[1][wave] = hi;
                s_mm[2][wave] = bad ? 1.0f : 0.0f;
            }
            __syncthreads();
            bool far = false;
            for (int w = 0; w < W; ++w) {
                lo = fminf(lo, s_mm[0][w]);
                hi = fmaxf(hi, s_mm[1][w]);
                far = far || s_mm[2][w] != 0.0f;
            }
            const int g0 = far ? 0 : (int)floorf(lo) - kGridLeft;
            const int g1 = far ? 0 : (int)floorf(hi) + kGridQ - kGridLeft;
            const int groups = __builtin_amdgcn_readfirstlane((g1 - g0 + kGridGroup - 1) / kGridGroup);
            double t = 0.0;
#pragma unroll
            for (int m = 0; m < CPT; ++m)
                if (cell_i[m] < n) t += (double)x[m][SV_VD];
            t = grid_wave(t, [](double x, double y) { return x + y; });
            if (lane == 0) s_red[wave] = t;
            const bool ok = !far && groups <= kGridMaxGroups;
            const int used = (min(n, BLOCK) + 63) / 64;      // waves that hold cells
            if (ok) {
                const double ck = grid_exp((double)((lane & 15) * (lane & 15)) * -0.01);
                // (group, cells of one wave) over all waves, whether they hold cells or not
                for (int q = wave; q < groups * used; q += W) {
                    const int gr = q / used, cw = q - gr * used;
                    double acc[kGridGroup];
#pragma unroll
                    for (int k = 0; k < kGridGroup; ++k) acc[k] = 0.0;
#pragma unroll
                    for (int m = 0; m < CPT; ++m) {
                        const int j = cw * 64 + lane + m * BLOCK;
                        if (j < n) grid_add(acc, g0 + gr * kGridGroup, vd[j]);
                    }
                    const double f = grid_lane_sum(acc, lane) * ck;
                    if (lane < kGridGroup) s_g[cw * GP + gr * kGridGroup + lane] = f;
                }
            }
            __syncthreads();
            for (int w = 0; w < W; ++w) tot += s_red[w];
            double* s_f = s_g + W * GP;
            if (ok) {
                for (int k = tid; k < groups * kGridGroup; k += BLOCK) {
                    double f = s_g[k];
                    for (int w = 1; w < used; ++w) f += s_g[w * GP + k];
                    s_f[k] = f;
                }
                __syncthreads();
            }
#pragma unroll
            for (int m = 0; m < CPT; ++m) {
                ig[m] = 0.0f;
                if (cell_i[m] < n) {
                    const float v = x[m][SV_VD];
                    const double lin = (double)n * (double)v - tot;
                    if (ok) {
                        ig[m] = (float)((double)g * (0.8 * grid_value(s_f, g0, v) + 0.2 * lin));
                    } else {
                        float acc = 0.0f;
                        for (int j = 0; j < n; ++j) {
                            const float dv = v - vd[j];
                            acc = fmaf(dv, gap_factor(dv), acc);
                        }
                        ig[m] = g * acc;
                    }
                }
            }
        } else if (!SPLIT && conn != CONN_NONE) {
            __syncthreads();                       // the rows' currents, or the waves' sums, are in LDS
            if (summed)
                for (int w = 0; w < W; ++w) tot += s_red[w];
        }

        // compartments; output; next voltages
        float y[CPT][NSV], iapp[CPT];
#pragma unroll
        for (int m = 0; m < CPT; ++m) {
            const int li = cell_i[m];
            if (li >= n) continue;
            if (dend) {
                iapp[m] = bias[m];
                for (int k = 0; k < n_pulses; ++k) {
                    const DevPulse& pl = s_pulse[k];
                    if (step >= pl.n0 && step < pl.n1 && li >= pl.c0 && li < pl.c1) iapp[m] += pl.amp;
                }
                if (step < stream_steps) iapp[m] += stream[step * (int64_t)n + li];
            }
            if (SPLIT) {                           // the voltages other waves advance
                x[m][SV_VD] = cur[0][li];
                x[m][SV_VS] = cur[1][li];
                x[m][SV_VA] = cur[2][li];
            }
            if (dend) cell_step_dgates(p, x[m], dt, y[m]);
            if (soma) {
                cell_step_soma(p, x[m], dt, y[m]);
                nxt[1][li] = y[m][SV_VS];
            }
            if (axon) {
                cell_step_axon(p, x[m], dt, y[m]);
                nxt[2][li] = y[m][SV_VA];
                if (a.out_slots && !a.dry) a.out_ring[slot * a.stride + d.cell_off + li] = y[m][SV_VA];
                if (x[m][SV_VA] < 0.0f && y[m][SV_VA] >= 0.0f) {
                    if (a.spike_cap > 0 && !a.dry) {
                        const float frac = (0.0f - x[m][SV_VA]) / (y[m][SV_VA] - x[m][SV_VA]);
                        a.spike_times[(d.cell_off + li) * a.spike_cap + (count[m] % a.spike_cap)] =
                            ((float)step + frac) * dt;
                    }
                    count[m] += 1;
                }
            }
        }
        if (SPLIT) __syncthreads();                // the parts' sums (or the voltages') are in LDS
#pragma unroll
        for (int m = 0; m < CPT; ++m) {
            const int li = cell_i[m];
            if (li >= n) continue;
            if (dend) {
                float cur_ig = 0.0f;
                if (summed) {
                    cur_ig = g * (float)((double)n * (double)x[m][SV_VD] - (SPLIT ? s_red[0] : tot));
                } else if (grid) {
                    cur_ig = ig[m];
                } else if (conn != CONN_NONE) {
                    if (SPLIT)
                        for (int q = 0; q < parts; ++q) cur_ig += s_ig[q * CELLS + li];
                    else
                        cur_ig = s_ig[li];
                    cur_ig *= scale;
                }
                cell_step_vd(p, x[m], cur_ig, iapp[m], dt, y[m]);
                nxt[0][li] = y[m][SV_VD];
#pragma unroll
                for (int v : {SV_VD, SV_CA, SV_R, SV_S, SV_Q}) x[m][v] = y[m][v];
            }
            if (soma)
#pragma unroll
                for (int v : {SV_VS, SV_K, SV_L, SV_H, SV_N, SV_X}) x[m][v] = y[m][v];
            if (axon)
#pragma unroll
                for (int v : {SV_VA, SV_HA, SV_XA}) x[m][v] = y[m][v];
        }
        if (a.out_slots) slot = slot + 1 == a.out_slots ? 0 : slot + 1;
        __syncthreads();
    }

    bool bad = false;
#pragma unroll
    for (int m = 0; m < CPT; ++m) {
        const int li = cell_i[m];
        if (li >= n) continue;
        const int64_t cell = d.cell_off + li;
        float chk = 0.0f;
        auto put = [&](int v) {
            xout[v * a.stride + cell] = x[m][v];
            chk += x[m][v];
        };
        if (dend)
#pragma unroll
            for (int v : {SV_VD, SV_CA, SV_R, SV_S, SV_Q}) put(v);
        if (soma)
#pragma unroll
            for (int v : {SV_VS, SV_K, SV_L, SV_H, SV_N, SV_X}) put(v);
        if (axon) {
#pragma unroll
            for (int v : {SV_VA, SV_HA, SV_XA}) put(v);
            if (!a.dry) a.spike_count[cell] = count[m];
        }
        bad = bad || !isfinite(chk);
    }
    if (bad && !a.dry) atomicOr(a.flags, 1);
}

}  // namespace infoli
