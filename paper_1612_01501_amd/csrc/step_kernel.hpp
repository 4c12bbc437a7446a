// One synchronous simulation step for a list of tiles (Section 2.2): every
// workgroup takes one tile = a block of consecutive cells of one network,
// computes their gap-junction currents from the step-n dendritic voltages
// (Section 2.3, Algorithm 1) and then their compartment update into the
// step-n+1 buffer. Reads only the step-n buffer and writes only the step-n+1
// buffer, so the kernel boundary is the step barrier.
//
// Gap-current layouts (per network):
//   UNIFORM_ALL  lanes = receiving cells (64 per tile); the waves of the
//                workgroup split the sending cells j, whose prescaled Vd is
//                staged in LDS in chunks and read as wave-wide broadcasts.
//                w = g is factored out and the linear part 0.2*sum_j dV is
//                taken in closed form, 0.2*(n*Vd_i - sum_j Vd_j), in fp64.
//                From kGridCells cells on by default: sums on a grid of
//                voltages, interpolated at each row (gap_grid.hpp).
//   DENSE        lanes = four consecutive sending cells each of four rows
//                (coalesced weight rows), the waves a share of the columns,
//                butterfly reduction.
//   BITMAP       (CSR networks with one weight g, when faster) the coupling
//                pattern as one bit per pair: 16 receiving cells per wave,
//                four lane groups per cell take interleaved 32-sender blocks
//                of a 128-sender group (conflict-free LDS rows), waves split
//                the groups; every pair is evaluated and masked.
//   BLOCKED CSR  (networks too large for one LDS copy of Vd) Vd is staged in
//                LDS one column block at a time; each row's edges of that
//                block (16-byte chunks of columns relative to the block)
//                gather from LDS; partial sums stay in registers across blocks.
//   CHUNKED CSR  Vd of the network in LDS; a tile's column chunks as one flat
//                run, a chunk per thread, the rows' sums from LDS slots.
//   CSR          groups of L lanes per row stride over the row's edges and
//                gather Vd of the neighbours, from a copy of the network's
//                Vd staged in LDS when the tile's edges outnumber the cells,
//                else from global memory; columns are 16-bit when every
//                network has at most 65,536 cells. Butterfly reduction per
//                group.
// Every reduction has a fixed order: results are bitwise reproducible.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include <stdint.h>

#include "cell_model.hpp"
#include "gap_grid.hpp"

namespace infoli {

enum : int { CONN_NONE = 0, CONN_UNIFORM = 1, CONN_DENSE = 2, CONN_CSR = 3 };

constexpr int kMaxTileRows = 256;   // rows (cells) per tile, any layout (<= BLOCK)
constexpr int kUniformRows = 64;    // rows per UNIFORM_ALL tile (one per lane)
constexpr int kChunk = 8192;        // Vd values staged in LDS per pass
constexpr int kBatch = 16;          // CSR edges per lane per batch of loads
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at any 4-byte boundary

// log2(e)/100: exp(-dV^2/100) = 2^(-(dV*a)^2) with a = sqrt(log2(e)/100).
constexpr float kL2eOver100 = 0.014426950408889634f;
constexpr float kPreScale = 0.12011224087864498f;      // sqrt(log2(e)/100)
constexpr float kInvPreScale = 8.325546111576977f;     // 1/kPreScale
constexpr float kSentinel = 1.0e19f;                   // prescaled pad: term == -0

struct InstDesc {
    int64_t cell_off;      // flattened index of the network's cell 0
    int64_t rp_off;        // CSR: offset of the network's row_ptr[0]
    int64_t w_off;         // DENSE: offset of w[0][0]; CSR: offset of edge 0
    int64_t stream_off;    // offset of the network's dense input stream, -1 none
    int64_t stream_steps;
    int32_t n;
    int32_t conn;
    float g;
    int32_t has_w;         // CSR: per-edge weights present
    int32_t pulse_off;
    int32_t n_pulses;
    int32_t lanes_per_row; // CSR: lanes per row (4..64)
    int32_t vd_lds;        // CSR: stage the network's Vd in LDS (n <= kChunk)
    int32_t col16;         // CSR: columns stored as uint16
    int32_t bitmap;        // CSR with uniform g: gap from the coupling bitmap
    int32_t blocked;       // CSR: Vd staged in LDS one column block at a time
    int32_t nblk;          // blocked: number of column blocks
    int32_t wide;          // run in the wide launch group
    int32_t chunked;       // CSR from the chunked rows layout
    int32_t flat;          //   as one flat run of chunks per tile, Vd in LDS
    int32_t sgj;           // simplified (linear) gap junctions: term w * dV
    int32_t pcell;         // per-cell parameters in StepArgs::cparams
    int32_t stream;        // blocked: the flat chunk stream (row tags) instead of row groups
    int32_t sym;           // UNIFORM: sums a kernel ahead of the step wrote into psym: each
                           // unordered pair once (k_pairs_sym), or for the simplified term the
                           // voltage sum (k_vsum)
    int64_t bits_off;      // bitmap: offset of the network's first word
    int64_t ca_off;        // chunked rows: offset of the [n + 1] row chunk starts, -1 none
    int64_t chk_off;       // chunked rows: first chunk of the network
    int64_t cb_off;        // chunked blocks: offset of the [n][nblk + 1] chunk starts, -1 none
    int64_t chkb_off;      // chunked blocks: first chunk of the network
    int64_t psym_off;      // sym: offset of the network's partial sums in StepArgs::psym
    int32_t sym_ki;        // sym: row blocks per workgroup of k_pairs_sym
    int32_t stream_round;  // stream: chunks per round (0: kStreamRound)
    int64_t p0_n0, p0_n1;  // the first pulse (StepArgs::pulses[pulse_off]), an empty window without
    float p0_amp;          // pulses: read with the descriptor, not by a load of its own that the
    int32_t p0_c0, p0_c1;  // cells' waves would wait for before their gap work
    int32_t pairs;         // UNIFORM, realistic: the caller asked for pairs (pair_path)
    int32_t grid_wide;     // UNIFORM on the grid: run in the wide launch group, with others like it alone
    int32_t grid;          // UNIFORM, realistic: sums on the voltage grid, 1 each tile its own, 2
                           // k_grid_sums ahead of the step (partial sums at psym_off)
    CellParams p;
};

// Rows [row0, row1) of a network, and what its first loads need, so that they
// wait for this record only and not for the descriptor behind it.
struct Tile {
    int32_t inst;
    int32_t row0;
    int32_t row1;
    int32_t n;             // the network's cells
    int64_t cell_off;      // its cell 0
    int64_t chk0;          // chunked CSR in LDS: the tile's first chunk (flat_first)
    int64_t row_chk;       //   where the chunk starts of its rows are in StepArgs::ca
    int32_t chunks;        //   and its chunks
    int32_t chk_base;      //   the first one's index in the network
};

struct DevPulse {
    int64_t n0, n1;        // active for steps n0 <= step < n1
    float amp;
    int32_t c0, c1;        // on local cells c0 <= i < c1
    int32_t pad0;
};

struct StepArgs {
    const InstDesc* inst;
    const Tile* tiles;
    const DevPulse* pulses;
    const float* bias;         // [cells]
    const int64_t* row_ptr;    // CSR row pointers of all networks
    const int32_t* col;        // CSR columns (local cell index)
    const uint16_t* col16;     // CSR columns, 16-bit form
    const uint32_t* bits;      // coupling bitmaps
    int32_t blk_cols;          // blocked CSR: cells per column block
    const int32_t* ca;         // chunked rows: per row, first chunk (relative to the network's)
    const int32_t* cb;         // chunked blocks: per row and block, first chunk
    const uint4* chk;          // chunks of eight 16-bit columns
    const float* chkw;         // per-edge weights in the chunk layout (8 per chunk)
    const uint8_t* rtag;       // chunked blocks: per chunk, its row mod 256
    const float* w;            // DENSE matrices and CSR weights
    const float* i_stream;     // dense input streams
    int32_t* spike_count;      // [cells]
    float* spike_times;        // [cells][spike_cap]
    int32_t* flags;            // [0]: non-finite state seen
    float* igap_out;           // gap-only mode: [cells]
    const int64_t* d_step;     // when set, step = *d_step + step offset
    int64_t stride;            // state row stride (floats)
    float dt;
    int32_t spike_cap;
    int32_t gap_only;
    int32_t dry;               // timing runs: write the next state only
    int32_t out_slots;         // output ring: slots (steps), 0 => none
    float* out_ring;           // [out_slots][stride]: Va after step s in slot s mod out_slots
    const float* cparams;      // [20][stride]: per-cell parameters (networks with pcell)
    const float* psym;         // partial row sums of the sym networks (k_pairs_sym)
    int32_t lds_floats;        // LDS floats of the launch's staged region (var_vd_first variants)
};

// Kernel variants by the tiles a launch holds; the narrow ones are compiled
// without the paths they exclude and their registers, so that more waves per
// SIMD keep loads in flight.
//   kVarAll      any tile
//   kVarNoGap    networks without gap junctions (the compartment update alone)
//   kVarFlat     those, flat chunked rows without per-edge weights, and the
//                simplified all-to-all form with the sum taken once
//   kVarStream   chunk stream tiles (column blocks) only
//   kVarDense    dense weight matrices or no gap junctions (256 threads)
//   kVarNoW      no per-edge weights, per-cell parameters or dense matrices
//   kVarFlatW    flat chunked rows or no gap junctions, with per-edge weights or
//                per-cell parameters
//   kVarFlatUni  kVarFlat's tiles and all-to-all networks
enum : int {
    kVarAll = 0, kVarNoGap = 1, kVarFlat = 2, kVarStream = 3, kVarDense = 4, kVarNoW = 5, kVarFlatW = 6, kVarFlatUni = 7
};
constexpr bool var_weights(int v) { return v == kVarAll || v == kVarFlatW; }      // per-edge weights
constexpr bool var_cells(int v) { return v == kVarAll || v == kVarFlatW; }        // per-cell parameters
constexpr bool var_uniform(int v) { return v == kVarAll || v == kVarNoW || v == kVarFlatUni; }
constexpr bool var_gathers(int v) { return v == kVarAll || v == kVarNoW; }        // CSR forms beside the flat one
// the staged voltages first in LDS (no static LDS; the sums' arrays follow the
// launch's region, lds_floats from its start): a gather's LDS address is then its
// column times four, with no base to add
constexpr bool var_vd_first(int v) { return v == kVarFlat || v == kVarFlatW || v == kVarFlatUni; }
constexpr size_t vd_first_bytes(int block) {       // the arrays behind the region
    return block / 64 * sizeof(double) + (block + kMaxTileRows) * sizeof(float);
}
// waves per SIMD the register allocator aims at (1: its own choice)
constexpr int var_waves(int v) { return v == kVarNoW ? 5 : v == kVarFlatUni ? 6 : 1; }

// The parameters of one cell: the network's, or the cell's own (SoA rows).
__device__ __forceinline__ CellParams cell_params_of(const StepArgs& a, const InstDesc& d, int64_t cell) {
    CellParams p = d.p;
    if (d.pcell) {
        float* f = reinterpret_cast<float*>(&p);
#pragma unroll
        for (int v = 0; v < 20; ++v) f[v] = a.cparams[v * a.stride + cell];
    }
    return p;
}

// Output ring slot of step s (s >= 0).
__device__ __forceinline__ int64_t out_slot(const StepArgs& a, int64_t s) {
    return (s % a.out_slots) * a.stride;
}

__device__ __forceinline__ float wave_sum_xor(float v, int width) {
    // butterfly over `width` consecutive lanes (power of two <= 64)
    for (int m = width >> 1; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

__device__ __forceinline__ float gap_factor(float dv) {
    // 0.8*exp(-dv^2/100) + 0.2 via the hardware 2^x
    return fmaf(0.8f, __builtin_amdgcn_exp2f(-(dv * dv) * kL2eOver100), 0.2f);
}

// The same factor of a voltage difference prescaled by kPreScale (Vd staged
// in LDS times sqrt(log2(e)/100)): 0.8 * 2^(-dv'^2) + 0.2; the sum over a row
// is scaled back by kInvPreScale once.
__device__ __forceinline__ float gap_factor_ps(float dvs) {
    return fmaf(0.8f, __builtin_amdgcn_exp2f(-(dvs * dvs)), 0.2f);
}

// The factor multiplying w * dV: the realistic one (of a prescaled
// difference when PS), or 1 for simplified gap junctions (Section 2.3.2),
// which is linear, so a prescaled row sum scales back the same way.
template <bool SGJ, bool PS>
__device__ __forceinline__ float pair_factor(float dv) {
    if constexpr (SGJ) return 1.0f;
    else return PS ? gap_factor_ps(dv) : gap_factor(dv);
}

// Blocks of the all-to-all path that takes each unordered pair once
// (k_pairs_sym below).
constexpr int kSymCells = 4096;     // all-to-all networks from this size on (library choice)
constexpr int kSymMaxKi = 16;       // row blocks per workgroup, at most

__host__ __device__ constexpr int sym_blocks(int n) { return (n + 63) / 64; }
__host__ __device__ constexpr int sym_kmax(int n) { return sym_blocks(n) / 2; }
__host__ __device__ constexpr int sym_shares(int n, int ki) {       // workgroups per column block
    return sym_kmax(n) > ki ? (sym_kmax(n) + ki - 1) / ki : 1;
}
// floats of a network's partial sums: [B][K][64] row sums of block pairs,
// [B][S][64] column sums, [B][64] own-block row sums, then B fp64 sums of
// each block's voltages (a multiple of 64 floats in all)
__host__ __device__ constexpr int64_t sym_vsum_off(int n, int ki) {
    return (int64_t)sym_blocks(n) * 64 * (sym_kmax(n) + sym_shares(n, ki) + 1);
}
__host__ __device__ constexpr int64_t sym_floats(int n, int ki) {
    return (sym_vsum_off(n, ki) + 2 * (int64_t)sym_blocks(n) + 63) / 64 * 64;
}

// The simplified term's closed form g (n Vd_i - sum_j Vd_j) needs one sum of
// all voltages. Each tile adding all n of them is O(n^2 / 64) loads per
// step; from kSgjSumCells cells on, a context's only such network has k_vsum
// write one fp64 sum per kVsumCells cells ahead of the step instead (one
// more launch; measured 0.1 us slower per step at 8,192 cells, 1.0 us faster
// at 12,288).
constexpr int kVsumCells = 4096;
constexpr int kSgjSumCells = 12288;
__host__ __device__ constexpr int vsum_groups(int n) { return (n + kVsumCells - 1) / kVsumCells; }
__host__ __device__ constexpr int64_t vsum_floats(int n) { return (2 * (int64_t)vsum_groups(n) + 63) / 64 * 64; }

template <int BLOCK>
__device__ __forceinline__ void gap_uniform(const StepArgs& a, const InstDesc& d, const Tile& t,
                                            const float* __restrict__ vd, float* s_ig,
                                            float4* s_v4, float* s_part, double* s_red) {
    constexpr int W = BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nrows = t.row1 - t.row0;
    const int n = d.n;
    const bool valid = lane < nrows;
    const float vi = valid ? vd[t.row0 + lane] : 0.0f;
    const float vis = vi * kPreScale;
    float* s_v = reinterpret_cast<float*>(s_v4);
    float acc0 = 0.0f, acc1 = 0.0f;
    double vsum = 0.0;
    if (d.sgj) {
        // simplified: g (n Vd_i - sum_j Vd_j), the sum in fp64
        for (int k = threadIdx.x; k < n; k += BLOCK) vsum += (double)vd[k];
    } else if (d.sym) {
        // the realistic form's linear part from the blocks' sums k_pairs_sym wrote
        const double* bs = reinterpret_cast<const double*>(a.psym + d.psym_off + sym_vsum_off(n, d.sym_ki));
        for (int k = threadIdx.x; k < sym_blocks(n); k += BLOCK) vsum += bs[k];
    }
    if (d.sym && !d.sgj && valid) {
        // the row's partial sums from k_pairs_sym, in a fixed order: its
        // block's own pairs, its row sums of block pairs (k = 1 .. KR), the
        // column sums of its block; each wave adds a consecutive run,
        // loading a batch at a time so that the loads overlap
        const int r = t.row0 + lane, R = r >> 6, l = r & 63;
        const int B = sym_blocks(n), K = sym_kmax(n), S = sym_shares(n, d.sym_ki);
        const int KR = (B & 1) ? (B - 1) / 2 : B / 2 - 1 + (R >= B / 2 ? 1 : 0);
        const float* P = a.psym + d.psym_off;
        const float* prow = P + (int64_t)R * K * 64 + l;
        const float* pcol = P + (int64_t)B * K * 64 + (int64_t)R * S * 64 + l;
        const float* pdiag = P + (int64_t)B * K * 64 + (int64_t)B * S * 64 + (int64_t)R * 64 + l;
        const int E = 1 + KR + S, per = (E + W - 1) / W;
        const int q0 = wave * per, q1 = min(E, q0 + per);
        constexpr int kQ = 16;
        for (int qb = q0; qb < q1; qb += kQ) {
            float v[kQ];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                const int q = qb + u;
                v[u] = q >= q1 ? 0.0f : q == 0 ? *pdiag : q <= KR ? prow[(int64_t)(q - 1) * 64]
                                                                   : pcol[(int64_t)(q - 1 - KR) * 64];
            }
#pragma unroll
            for (int u = 0; u < kQ; ++u) acc0 += v[u];
        }
    }
    for (int c0 = 0; c0 < (d.sgj || d.sym ? 0 : n); c0 += kChunk) {
        const int cn = min(kChunk, n - c0);
        // per-wave share, a multiple of 8 values; the tail is padded with a
        // sentinel whose term is exactly -0
        const int per = (((cn + W - 1) / W) + 7) & ~7;
        __syncthreads();
        for (int k = threadIdx.x; k < W * per; k += BLOCK) {
            if (k < cn) {
                const float v = vd[c0 + k];
                s_v[k] = v * kPreScale;
                vsum += (double)v;
            } else {
                s_v[k] = kSentinel;
            }
        }
        __syncthreads();
        const float4* p = s_v4 + (wave * per) / 4;
        for (int q = 0; q < per / 4; q += 2) {
            const float4 u = p[q];
            const float4 v = p[q + 1];
            float d0 = vis - u.x, d1 = vis - u.y, d2 = vis - u.z, d3 = vis - u.w;
            acc0 = fmaf(d0, __builtin_amdgcn_exp2f(-(d0 * d0)), acc0);
            acc1 = fmaf(d1, __builtin_amdgcn_exp2f(-(d1 * d1)), acc1);
            acc0 = fmaf(d2, __builtin_amdgcn_exp2f(-(d2 * d2)), acc0);
            acc1 = fmaf(d3, __builtin_amdgcn_exp2f(-(d3 * d3)), acc1);
            d0 = vis - v.x; d1 = vis - v.y; d2 = vis - v.z; d3 = vis - v.w;
            acc0 = fmaf(d0, __builtin_amdgcn_exp2f(-(d0 * d0)), acc0);
            acc1 = fmaf(d1, __builtin_amdgcn_exp2f(-(d1 * d1)), acc1);
            acc0 = fmaf(d2, __builtin_amdgcn_exp2f(-(d2 * d2)), acc0);
            acc1 = fmaf(d3, __builtin_amdgcn_exp2f(-(d3 * d3)), acc1);
        }
    }
    s_part[wave * 64 + lane] = acc0 + acc1;
    // fixed-order reduction of sum_j Vd_j (fp64)
    for (int m = 32; m > 0; m >>= 1) vsum += __shfl_xor(vsum, m, 64);
    if (lane == 0) s_red[wave] = vsum;
    __syncthreads();
    if (threadIdx.x < 64 && valid) {
        float e = 0.0f;
        for (int w = 0; w < W; ++w) e += s_part[w * 64 + lane];
        double tot = 0.0;
        for (int w = 0; w < W; ++w) tot += s_red[w];
        const float lin = (float)((double)n * (double)vi - tot);
        s_ig[lane] = d.sgj ? d.g * lin : d.g * (0.8f * (e * kInvPreScale) + 0.2f * lin);
    }
}

// The simplified all-to-all form with the voltage sum taken once per step:
// the workgroup adds the fp64 group sums k_vsum wrote in a fixed order, then
// each of the tile's rows (up to kMaxTileRows) takes g (n Vd_i - sum).
template <int BLOCK>
__device__ __forceinline__ void gap_uniform_sum(const StepArgs& a, const InstDesc& d, const Tile& t,
                                                const float* __restrict__ vd, float* s_ig, double* s_red) {
    constexpr int W = BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const double* gs = reinterpret_cast<const double*>(a.psym + d.psym_off);
    double vsum = 0.0;
    for (int k = threadIdx.x; k < vsum_groups(d.n); k += BLOCK) vsum += gs[k];
    for (int m = 32; m > 0; m >>= 1) vsum += __shfl_xor(vsum, m, 64);
    if (lane == 0) s_red[wave] = vsum;
    __syncthreads();
    double tot = 0.0;
    for (int w = 0; w < W; ++w) tot += s_red[w];
    for (int k = threadIdx.x; k < t.row1 - t.row0; k += BLOCK)
        s_ig[k] = d.g * (float)((double)d.n * (double)vd[t.row0 + k] - tot);
}

// Every pair of the tile's rows, 64 rows at a time: a lane per row, a wave's share
// of the cells 64 at a time, a lane each to load (the next ones ahead) and then one
// after the other for all rows, their terms' sums added up in fp64 (2,000 cells
// 14.3 us a step; through LDS, read four at a time by all lanes, 16.5). Where k_grid_sums took
// the voltages' sum and it is not finite, a voltage is not, and no row's terms are
// (an infinite difference times e^-inf is a NaN).
template <int BLOCK>
__device__ __forceinline__ void gap_uniform_pairs(const StepArgs& a, const InstDesc& d, const Tile& t,
                                                  const float* __restrict__ vd, float* s_ig, double* s_red,
                                                  double* s_w) {
    constexpr int W = BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = d.n;
    const int nrows = t.row1 - t.row0;
    double vsum = 0.0;
    const auto wave_total = [&]() {
        vsum = grid_wave(vsum, [](double x, double y) { return x + y; });
        if (lane == 0) s_red[wave] = vsum;
    };
    const auto total = [&]() {
        double tot = 0.0;
        for (int w = 0; w < W; ++w) tot += s_red[w];
        return tot;
    };
    if (d.grid == 2) {
        const int C = grid_chunks(n);
        const double* vs = reinterpret_cast<const double*>(a.psym + d.psym_off) + (int64_t)kGridAheadGroups * C * kGridGroup;
        for (int c = threadIdx.x; c < C; c += BLOCK) vsum += vs[c];
        wave_total();
        __syncthreads();
        if (!(fabs(total()) <= 1.0e300)) {
            if ((int)threadIdx.x < nrows) s_ig[threadIdx.x] = __builtin_nanf("");
            return;
        }
    }
    const int per = ((n + W - 1) / W + 63) / 64 * 64;
    const int j0 = min(n, wave * per), j1 = min(n, j0 + per);
    for (int r0 = 0; r0 < nrows; r0 += 64) {
        const bool sum = d.grid != 2 && r0 == 0;
        const float v = vd[t.row0 + min(r0 + lane, nrows - 1)];
        double acc = 0.0;
        float next = vd[min(j0 + lane, n - 1)];
        for (int j = j0; j < j1; j += 64) {
            const float u = next;
            next = vd[min(j + 64 + lane, n - 1)];
            const auto cell = [&](int k) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(u), k)); };
            const int m = min(64, j1 - j);
            float a0 = 0.0f, a1 = 0.0f;
            int k = 0;
            for (; k + 16 <= m; k += 16) {
#pragma unroll
                for (int e = 0; e < 16; e += 2) {
                    const float d0 = v - cell(k + e), d1 = v - cell(k + e + 1);
                    a0 = fmaf(d0, __builtin_amdgcn_exp2f(-(d0 * d0) * kL2eOver100), a0);
                    a1 = fmaf(d1, __builtin_amdgcn_exp2f(-(d1 * d1) * kL2eOver100), a1);
                }
            }
            for (; k < m; ++k) {
                const float d0 = v - cell(k);
                a0 = fmaf(d0, __builtin_amdgcn_exp2f(-(d0 * d0) * kL2eOver100), a0);
            }
            acc += (double)(a0 + a1);
            if (sum && lane < m) vsum += (double)u;
        }
        s_w[wave * 64 + lane] = acc;
        if (sum) wave_total();
        __syncthreads();
        if ((int)threadIdx.x < 64 && r0 + lane < nrows) {
            double f = 0.0;
            for (int w = 0; w < W; ++w) f += s_w[w * 64 + lane];
            const double lin = (double)n * (double)v - total();
            s_ig[r0 + lane] = (float)((double)d.g * (0.8 * f + 0.2 * lin));
        }
        __syncthreads();
    }
}

// All-to-all networks with the realistic term on the voltage grid
// (gap_grid.hpp): up to BLOCK rows, one per thread. The tile takes the grid
// points its own rows' voltages need; it sums the cells' terms there itself,
// or (d.grid 2) adds the shares' sums k_grid_sums wrote, in a fixed order either
// way. A tile whose rows hold a voltage that is not finite or, ahead, outside
// the grid, or are so far apart that its own sums cost more than the pairs,
// takes every pair (grid_tile_groups).
template <int BLOCK>
__device__ __forceinline__ void gap_uniform_grid(const StepArgs& a, const InstDesc& d, const Tile& t,
                                                 const float* __restrict__ vd, float* s_ig, float* s_part,
                                                 double* s_red, double* s_g) {
    constexpr int W = BLOCK / 64;
    constexpr int GP = kGridAheadGroups * kGridGroup;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = d.n;
    const int nrows = t.row1 - t.row0;
    const float v = vd[t.row0 + min((int)threadIdx.x, nrows - 1)];
    float lo = grid_wave(v, [](float x, float y) { return fminf(x, y); });
    float hi = grid_wave(v, [](float x, float y) { return fmaxf(x, y); });
    const bool bad = __any(!(fabsf(v) <= 1.0e6f));      // (a NaN too: min and max pass it by)
    if (lane == 0) {
        s_part[wave] = lo;
        s_part[W + wave] = hi;
        s_part[2 * W + wave] = bad ? 1.0f : 0.0f;
    }
    __syncthreads();
    bool far = false;
    for (int w = 0; w < W; ++w) {
        lo = fminf(lo, s_part[w]);
        hi = fmaxf(hi, s_part[W + w]);
        far = far || s_part[2 * W + w] != 0.0f;
    }
    int g0 = far ? 0 : (int)floorf(lo) - kGridLeft;             // first grid point
    const int g1 = far ? 0 : (int)floorf(hi) + kGridQ - kGridLeft;   // one past the last
    bool ok = !far;
    if (d.grid == 2) {
        ok = ok && g0 >= kGridAheadLo && g1 <= kGridAheadLo + kGridAheadGroups * kGridGroup;
        g0 -= (g0 - kGridAheadLo) & (kGridGroup - 1);           // whole groups of k_grid_sums
    }
    const int groups = __builtin_amdgcn_readfirstlane((g1 - g0 + kGridGroup - 1) / kGridGroup);
    ok = ok && (d.grid == 2 || groups <= grid_tile_groups(nrows));
    double vsum = 0.0;
    if (!ok) {
        gap_uniform_pairs<BLOCK>(a, d, t, vd, s_ig, s_red, s_g);
        return;
    }
    if (d.grid == 2) {
        // thread: two grid points, every (BLOCK / 8)-th share
        const double* P = reinterpret_cast<const double*>(a.psym + d.psym_off);
        const int C = grid_chunks(n);
        const int np = threadIdx.x & 7, c0 = threadIdx.x >> 3;
        const int gb = (g0 - kGridAheadLo) / kGridGroup;
        for (int g = 0; g < groups; ++g) {
            const double2* q = reinterpret_cast<const double2*>(P + (int64_t)(gb + g) * C * kGridGroup) + np;
            double2 s = make_double2(0.0, 0.0);
#pragma unroll
            for (int u = 0; u < (kGridChunks + BLOCK / 8 - 1) / (BLOCK / 8); ++u) {
                const int c = c0 + u * (BLOCK / 8);
                const double2 x = q[(int64_t)min(c, C - 1) * 8];
                s.x += c < C ? x.x : 0.0;
                s.y += c < C ? x.y : 0.0;
            }
            for (int m = 8; m < 64; m <<= 1) {
                s.x += __shfl_xor(s.x, m, 64);
                s.y += __shfl_xor(s.y, m, 64);
            }
            if (lane < 8) {
                s_g[wave * GP + g * kGridGroup + 2 * np] = s.x;
                s_g[wave * GP + g * kGridGroup + 2 * np + 1] = s.y;
            }
        }
        const double* vs = P + (int64_t)kGridAheadGroups * C * kGridGroup;
        for (int c = threadIdx.x; c < C; c += BLOCK) vsum += vs[c];
    } else {
        const double ck = grid_exp((double)((lane & 15) * (lane & 15)) * -0.01);
        for (int g = 0; g < groups; ++g) {
            const double t0 = g0 + g * kGridGroup;
            double acc[kGridGroup];
#pragma unroll
            for (int k = 0; k < kGridGroup; ++k) acc[k] = 0.0;
            for (int j = threadIdx.x; j < n; j += BLOCK) {
                const float vj = vd[j];
                grid_add(acc, t0, vj);
                if (g == 0) vsum += (double)vj;
            }
            const double s = grid_lane_sum(acc, lane) * ck;
            if (lane < kGridGroup) s_g[wave * GP + g * kGridGroup + lane] = s;
        }
    }
    vsum = grid_wave(vsum, [](double x, double y) { return x + y; });
    if (lane == 0) s_red[wave] = vsum;
    __syncthreads();
    double* s_f = s_g + W * GP;
    for (int k = threadIdx.x; k < groups * kGridGroup; k += BLOCK) {
        double f = s_g[k];
        for (int w = 1; w < W; ++w) f += s_g[w * GP + k];
        s_f[k] = f;
    }
    __syncthreads();
    if ((int)threadIdx.x < nrows) {
        double tot = 0.0;
        for (int w = 0; w < W; ++w) tot += s_red[w];
        const double lin = (double)n * (double)v - tot;
        s_ig[threadIdx.x] = (float)((double)d.g * (0.8 * grid_value(s_f, g0, v) + 0.2 * lin));
    }
}

// ---------------------------------------------------------------- all-to-all, each unordered pair once
// The pair term dV * f(dV) (Section 2.3.1, Algorithm 1) is odd in dV, and
// exactly so in floating point:
// the difference of (j, i) is minus that of (i, j), its square and the
// factor are the same, so its term is minus the other. An all-to-all
// network with one weight g therefore needs each unordered pair once.
// Cells form blocks of 64 (B blocks; the last one padded with kSentinel,
// whose terms against any cell are zero). The pairs of distinct blocks
// {J, J + k mod B}, 1 <= k <= B / 2 (k = B / 2 only for J < B / 2 when B is
// even, so that each block pair is taken once), belong to column block J.
// A workgroup of four waves takes sym_ki row blocks I = J + k in turn,
// lanes being I's cells, each wave with 16 of J's voltages in scalar
// registers: per pair one difference, square, exponential and two fused
// multiply-adds, one into the row's sum (the four waves' parts added in LDS,
// written for (I, k)) and one into the column's (added over the row blocks,
// then over the lanes). Each block's own 64 x 64 ordered pairs give its row
// sums directly. The step adds a cell's partial sums in a fixed order, so
// results do not depend on scheduling.

// Halving step of a lane-transposed sum: v[0 .. 2H) are sums of 2H
// consecutive columns over this lane; afterwards v[0 .. H) hold the sums over
// this lane and lane ^ H of the half of them selected by bit H of the lane.
// After H = 8, 4, 2, 1 a lane holds column (lane & 15)'s sum over the 16
// lanes that share its bits 4 and 5.
template <int H>
__device__ __forceinline__ void sym_halve(float* v, int lane) {
    const bool hi = (lane & H) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const float send = hi ? v[i] : v[i + H];
        const float keep = hi ? v[i + H] : v[i];
        v[i] = keep + __shfl_xor(send, H, 64);
    }
}

// One workgroup of four waves per (column block J, share s of its row
// blocks); wave w takes J's columns 16w .. 16w + 15 in scalar registers.
// Per row block the four waves' row sums meet in LDS and are added in wave
// order. vd: the network's Vd row; P: its partial sums.
static __global__ __launch_bounds__(256) void k_pairs_sym(const float* __restrict__ vd, int n, int ki,
                                                          float* __restrict__ P) {
    __shared__ float s_row[4][kSymMaxKi + 1][64];
    const int B = sym_blocks(n), K = sym_kmax(n), S = sym_shares(n, ki);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = blockIdx.x;
    if (g >= B * S) return;
    const int J = g / S, s = g - J * S;
    float* prow = P;                                   // [B][K][64]
    float* pcol = P + (int64_t)B * K * 64;             // [B][S][64]
    float* pdiag = pcol + (int64_t)B * S * 64;         // [B][64]
    double* bsum = reinterpret_cast<double*>(P + sym_vsum_off(n, ki));   // [B]
    const int cj = J * 64 + lane;
    const float vraw = cj < n ? vd[cj] : 0.0f;
    const float vc = cj < n ? vraw * kPreScale : kSentinel;
    float sc[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) sc[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vc), 16 * w + u));
    // row blocks J + k, k in [k0, k1], of this workgroup
    const int KJ = (B - 1) / 2 + ((B % 2 == 0 && J < B / 2) ? 1 : 0);
    const int k0 = 1 + s * ki, k1 = min(KJ, s * ki + ki);
    if (s == 0) {
        // the block's own pairs, ordered, row sums only (a cell's term with
        // itself is exactly zero); wave 0 also sums the block's voltages
        float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
        for (int u = 0; u < 16; u += 2) {
            const float d0 = vc - sc[u], d1 = vc - sc[u + 1];
            a0 = fmaf(d0, __builtin_amdgcn_exp2f(-(d0 * d0)), a0);
            a1 = fmaf(d1, __builtin_amdgcn_exp2f(-(d1 * d1)), a1);
        }
        s_row[w][kSymMaxKi][lane] = a0 + a1;
        if (w == 0) {
            double t = (double)vraw;
            for (int m = 32; m > 0; m >>= 1) t += __shfl_xor(t, m, 64);
            if (lane == 0) bsum[J] = t;
        }
    }
    float acol[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) acol[u] = 0.0f;
    auto row_v = [&](int k) {
        const int i = ((J + k) % B) * 64 + lane;
        return i < n ? vd[i] * kPreScale : kSentinel;
    };
    float vnext = k0 <= k1 ? row_v(k0) : 0.0f;
    for (int k = k0; k <= k1; ++k) {
        const float vi = vnext;
        if (k < k1) vnext = row_v(k + 1);
        float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
        for (int u = 0; u < 16; u += 2) {
            const float d0 = vi - sc[u], d1 = vi - sc[u + 1];
            const float e0 = __builtin_amdgcn_exp2f(-(d0 * d0)), e1 = __builtin_amdgcn_exp2f(-(d1 * d1));
            a0 = fmaf(d0, e0, a0);
            a1 = fmaf(d1, e1, a1);
            acol[u] = fmaf(-d0, e0, acol[u]);
            acol[u + 1] = fmaf(-d1, e1, acol[u + 1]);
        }
        s_row[w][k - k0][lane] = a0 + a1;
    }
    // column sums over the 64 lanes: lane l ends with column 16w + (l & 15)'s
    sym_halve<8>(acol, lane);
    sym_halve<4>(acol, lane);
    sym_halve<2>(acol, lane);
    sym_halve<1>(acol, lane);
    float c = acol[0];
    c += __shfl_xor(c, 16, 64);
    c += __shfl_xor(c, 32, 64);
    if (lane < 16) pcol[((int64_t)J * S + s) * 64 + 16 * w + lane] = c;
    __syncthreads();
    // row sums: the four waves' parts in wave order; wave w stores rows
    // blocks k0 + w, k0 + w + 4, .. (and wave 0 the block's own)
    for (int q = w; q <= k1 - k0; q += 4)
        prow[((int64_t)((J + k0 + q) % B) * K + (k0 + q - 1)) * 64 + lane] =
            ((s_row[0][q][lane] + s_row[1][q][lane]) + s_row[2][q][lane]) + s_row[3][q][lane];
    if (s == 0 && w == 0)
        pdiag[(int64_t)J * 64 + lane] = ((s_row[0][kSymMaxKi][lane] + s_row[1][kSymMaxKi][lane]) +
                                         s_row[2][kSymMaxKi][lane]) + s_row[3][kSymMaxKi][lane];
}

// One workgroup per kVsumCells cells: thread k adds voltages k, k + 256, ..
// in fp64, the lanes combine by a fixed butterfly and the waves in wave order,
// so the step's sum of the groups' sums is the same every step. The loads
// are all issued before the first add (one memory round trip per thread).
static __global__ __launch_bounds__(256) void k_vsum(const float* __restrict__ vd, int n,
                                                     double* __restrict__ out) {
    constexpr int kPer = kVsumCells / 256;
    __shared__ double s_w[4];
    const int base = blockIdx.x * kVsumCells;
    const int m = min(kVsumCells, n - base);
    float v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {   // past the last cell: load it again, add 0
        const int k = threadIdx.x + 256 * i;
        const float x = vd[base + min(k, m - 1)];
        v[i] = k < m ? x : 0.0f;
    }
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) s += (double)v[i];
    for (int h = 32; h > 0; h >>= 1) s += __shfl_xor(s, h, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
}

// ---------------------------------------------------------------- dense weights
// The weight matrix is read once per step, 4 bytes a pair, so the loads bound
// the tile and have to be in flight together. A tile takes kDenseRows rows;
// the workgroup's waves split the columns into stretches of 256 (four
// consecutive columns a lane, 16-byte loads; a row may start at any 4-byte
// boundary), kDenseSteps stretches of all rows loaded before the first is
// used, the voltages of a stretch loaded once for all rows. Columns past n
// (the last stretch only) load whatever follows the row (the weight array has
// kDenseSlack spare entries, the voltage row is followed by other state rows)
// and count as the row's own voltage, whose term is zero. Four rows and two
// stretches (ten 16-byte loads a lane in flight, 960 workgroups at 3,840
// cells): 74.8 -> 14.3 us per step there, where one row per wave with a
// 4-byte load per pair waited for each load in turn; eight rows 15.6 us, two
// rows 17.7, four stretches 15.5. The weights are read once per step, so they
// are loaded past the caches' reuse order (14.8 us without).
constexpr int kDenseRows = 4;
constexpr int kDenseSteps = 2;
constexpr int kDenseSlack = 4;

template <int BLOCK, bool SGJ>
__device__ __forceinline__ void gap_dense(const StepArgs& a, const InstDesc& d, const Tile& t,
                                          const float* __restrict__ vd, float* s_part, float* s_ig) {
    constexpr int W = BLOCK / 64;
    constexpr int R = kDenseRows, U = kDenseSteps;
    static_assert(W * R <= BLOCK, "a partial sum per wave and row");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = d.n;
    const int steps = (n + 255) / 256;                    // stretches of 256 columns
    const int per = (steps + W - 1) / W;                  // per wave
    const int s0 = min(steps, wave * per), s1 = min(steps, s0 + per);
    const float* w = a.w + d.w_off;
    for (int r0 = t.row0; r0 < t.row1; r0 += R) {
        float vi[R], acc[R];
        const float* wr[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = min(r0 + q, t.row1 - 1);
            vi[q] = vd[r];
            acc[q] = 0.0f;
            wr[q] = w + (int64_t)r * n;
        }
        for (int s = s0; s < s1; s += U) {
            f32x4u wv[U][R], v[U];
            // a step past the wave's last one loads the last one again
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = min(s + u, s1 - 1) * 256 + 4 * lane;
                v[u] = *reinterpret_cast<const f32x4u*>(vd + min(c, n - 1));
#pragma unroll
                for (int q = 0; q < R; ++q) wv[u][q] = __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(wr[q] + min(c, n - 1)));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (s + u >= s1) break;
                const int c = (s + u) * 256 + 4 * lane;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float vj = v[u][e];
                    const bool in = c + e < n;
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const float dv = in ? vi[q] - vj : 0.0f;
                        acc[q] = fmaf(wv[u][q][e], dv * pair_factor<SGJ, false>(dv), acc[q]);
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) acc[q] = wave_sum_xor(acc[q], 64);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < R; ++q) s_part[wave * R + q] = acc[q];
        __syncthreads();
        if ((int)threadIdx.x < R && r0 + (int)threadIdx.x < t.row1) {
            float tot = 0.0f;
            for (int k = 0; k < W; ++k) tot += s_part[k * R + threadIdx.x];
            s_ig[r0 + threadIdx.x - t.row0] = tot;
        }
        __syncthreads();
    }
}

template <int BLOCK, bool LDS, bool C16, bool HASW, bool SGJ>
__device__ __forceinline__ void gap_csr_impl(const StepArgs& a, const InstDesc& d, const Tile& t,
                                             const float* __restrict__ vd, const float* s_vd,
                                             float* s_part, float* s_ig) {
    // L lanes per row (4..BLOCK, power of two); a row wider than a wave
    // spans L/64 consecutive waves and is reduced through LDS.
    const int L = d.lanes_per_row;
    const int groups = BLOCK / L;
    const int grp = threadIdx.x / L;
    const int lig = threadIdx.x % L;
    const int64_t* rp = a.row_ptr + d.rp_off;
    const int32_t* c32 = a.col + d.w_off;
    const uint16_t* c16 = a.col16 + d.w_off;
    const float* wv = a.w + d.w_off;
    auto col_at = [&](int64_t k) -> int { return C16 ? (int)c16[k] : c32[k]; };
    // LDS: staged voltages are prescaled (gap_factor_ps), the row sum is
    // scaled back at the end
    auto v_at = [&](int j) -> float { return LDS ? s_vd[j] : vd[j]; };
    auto term = [&](float w, float vi, float vj) -> float {
        const float dv = vi - vj;
        const float f = pair_factor<SGJ, LDS>(dv);
        return HASW ? w * (dv * f) : dv * f;
    };
    const float back = LDS ? kInvPreScale : 1.0f;
    for (int r0 = t.row0; r0 < t.row1; r0 += groups) {
        const int r = r0 + grp;
        float acc0 = 0.0f, acc1 = 0.0f;
        if (r < t.row1) {
            const float vi = v_at(r);
            const int64_t e = rp[r + 1];
            int64_t k = rp[r] + lig;
            // batches of kBatch independent edges: all loads issue before use
            for (; k + (kBatch - 1) * L < e; k += kBatch * L) {
                int j[kBatch];
                float w[kBatch], v[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    j[u] = col_at(k + u * L);
                    w[u] = HASW ? wv[k + u * L] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) v[u] = v_at(j[u]);
#pragma unroll
                for (int u = 0; u < kBatch; u += 2) {
                    acc0 += term(w[u], vi, v[u]);
                    acc1 += term(w[u + 1], vi, v[u + 1]);
                }
            }
            // the remaining (< kBatch) edges of this lane as one masked
            // batch, so their loads are in flight together as well
            if (k < e) {
                int j[kBatch];
                float w[kBatch], v[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const bool ok = k + u * L < e;
                    j[u] = ok ? col_at(k + u * L) : r;      // the row itself: dV = 0
                    w[u] = HASW && ok ? wv[k + u * L] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) v[u] = v_at(j[u]);
#pragma unroll
                for (int u = 0; u < kBatch; u += 2) {
                    acc0 += term(w[u], vi, v[u]);
                    acc1 += term(w[u + 1], vi, v[u + 1]);
                }
            }
        }
        float acc = acc0 + acc1;
        if (L <= 64) {
            // all lanes of a group run the butterfly together
            acc = wave_sum_xor(acc, L) * back;
            if (r < t.row1 && lig == 0) s_ig[r - t.row0] = HASW ? acc : d.g * acc;
        } else {
            acc = wave_sum_xor(acc, 64);
            const int wave = threadIdx.x >> 6;
            if ((threadIdx.x & 63) == 0) s_part[wave] = acc;
            __syncthreads();
            if (lig == 0 && r < t.row1) {
                float tot = 0.0f;
                for (int w = 0; w < L / 64; ++w) tot += s_part[wave + w];
                tot *= back;
                s_ig[r - t.row0] = HASW ? tot : d.g * tot;
            }
            __syncthreads();
        }
    }
}

constexpr int kBlkPasses = 4;       // row passes per tile kept in registers

// ---------------------------------------------------------------- chunked CSR
// Column lists in 16-byte chunks of eight 16-bit columns, read with one
// vector load per lane per chunk: the L lanes of a row read consecutive
// chunks, so a row's 128-byte cache line is touched by one load instruction.
// Padding entries make a zero term (their voltage is the row's own, dV = 0).
constexpr int kChunkCols = 8;

__device__ __forceinline__ uint4 pad_chunk(uint32_t v) {
    const uint32_t w = v | (v << 16);
    return make_uint4(w, w, w, w);
}

// Sixteen edges of a row from two chunks: columns j, voltages from `src`
// (LDS, prescaled; or global), accumulated into acc0/acc1.
template <bool PS, bool HASW, bool SGJ>
__device__ __forceinline__ void chunk_pair_terms(const uint4 q0, const uint4 q1, const float4* w4,
                                                 const float* src, float vi, float& acc0, float& acc1) {
    const uint32_t wd[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
    float v[2 * kChunkCols];
#pragma unroll
    for (int e = 0; e < 2 * kChunkCols; ++e) {
        const uint32_t j = (e & 1) ? (wd[e >> 1] >> 16) : (wd[e >> 1] & 0xffffu);
        v[e] = src[j];
    }
#pragma unroll
    for (int e = 0; e < 2 * kChunkCols; e += 2) {
        const float d0 = vi - v[e], d1 = vi - v[e + 1];
        const float f0 = pair_factor<SGJ, PS>(d0);
        const float f1 = pair_factor<SGJ, PS>(d1);
        if (HASW) {
            const float4 wa = w4[e >> 2];
            const float w0 = (e & 3) == 0 ? wa.x : wa.z, w1 = (e & 3) == 0 ? wa.y : wa.w;
            acc0 = fmaf(w0, d0 * f0, acc0);
            acc1 = fmaf(w1, d1 * f1, acc1);
        } else {
            acc0 = fmaf(d0, f0, acc0);
            acc1 = fmaf(d1, f1, acc1);
        }
    }
}

// Byte offset 4*j of the 16-bit column j in the low or high half of w: one
// instruction (a shift reading one half-word of its operand), where the
// plain form takes an extract and a shift.
__device__ __forceinline__ uint32_t col_lo_bytes(uint32_t w) {
    uint32_t r;
    asm("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
        : "=v"(r) : "v"(w));
    return r;
}
__device__ __forceinline__ uint32_t col_hi_bytes(uint32_t w) {
    uint32_t r;
    asm("v_lshlrev_b32_sdwa %0, 2, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
        : "=v"(r) : "v"(w));
    return r;
}

typedef const __attribute__((address_space(3))) float lds_float;

// ---------------------------------------------------------------- chunked rows
// A tile's rows are one contiguous run of chunks (rows layout, padded with the
// row itself). Every thread takes chunks of the run, whatever row they belong
// to: no lane is idle on short rows, and the loads need no row pointers. A
// one-byte tag (row mod 256) names a chunk's row; its eight terms' sum goes to
// an LDS slot of its own, and the rows' owners (consecutive threads, as many
// as the tile's rows leave) add their row's slots in a fixed order. Vd of the
// whole network is staged in LDS (prescaled). kFlatChunks chunks per thread
// are in flight, the first ones while Vd is staged.
constexpr int kFlatChunks = 4;
constexpr int kFlatCells = 32768;       // networks up to this size (128 KB of Vd)

__host__ __device__ constexpr int flat_vd_floats(int n) { return (n + 3) & ~3; }

// Chunk, from the tile's first one on, that slot k of a tile of m chunks loads: its
// own, past the last one the last again. A tile whose rows have no connections
// loads one chunk all the same (a branch around the loads would keep them from
// overlapping the staging of Vd: three 4,096-cell networks 9.3 -> 9.5 us a step),
// so its first chunk is the network's first: its own may be one past the last of
// the arrays.
__host__ __device__ constexpr int flat_load(int k, int m) {
    const int last = k < m - 1 ? k : m - 1;
    return last > 0 ? last : 0;
}
__host__ __device__ constexpr int64_t flat_first(int64_t network, int base, int m) {
    return m > 0 ? network + base : network;
}

template <int BLOCK, bool HASW, bool SGJ, bool VD0>
__device__ __forceinline__ void gap_flat(const StepArgs& a, const InstDesc& d, const Tile& t,
                                         const float* __restrict__ vd, float* s_vd, float* s_ig) {
    constexpr int K = HASW ? kFlatChunks / 2 : kFlatChunks;
    const int m = t.chunks;
    const int nrows = t.row1 - t.row0;
    const uint4* ch = a.chk + t.chk0;
    const uint8_t* tag = a.rtag + t.chk0;
    const float4* cw = reinterpret_cast<const float4*>(a.chkw) + 2 * t.chk0;
    float* s_sums = s_vd + flat_vd_floats(t.n);
    const uint32_t vd_lds = VD0 ? 0u : (uint32_t)(size_t)(lds_float*)s_vd;   // VD0: Vd is first in LDS
    uint4 q[K];
    uint32_t tg[K];
    float4 w4[K][2];
    auto load = [&](int base) {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int i = flat_load(base + u * BLOCK + (int)threadIdx.x, m);
            q[u] = ch[i];
            tg[u] = tag[i];
            if (HASW) {
                w4[u][0] = cw[2 * (int64_t)i];
                w4[u][1] = cw[2 * (int64_t)i + 1];
            }
        }
    };
    load(0);
    // the owners of a row: OWN consecutive threads (a power of two, at most a wave)
    const int own = max(1, min(64, BLOCK >> (nrows <= 1 ? 0 : 32 - __builtin_clz(nrows - 1))));
    const int orow = threadIdx.x / own, oq = threadIdx.x & (own - 1);
    int lo = 0, hi = 0;
    if (orow < nrows) {
        lo = a.ca[t.row_chk + orow] - t.chk_base;
        hi = a.ca[t.row_chk + orow + 1] - t.chk_base;
    }
    // (up to three values past the last cell: the next state rows follow Vd)
    for (int k = 4 * threadIdx.x; k < t.n; k += 4 * BLOCK) {
        const f32x4u v = *reinterpret_cast<const f32x4u*>(vd + k);
        *reinterpret_cast<float4*>(s_vd + k) =
            make_float4(v[0] * kPreScale, v[1] * kPreScale, v[2] * kPreScale, v[3] * kPreScale);
    }
    __syncthreads();
    for (int base = 0; base < m; base += K * BLOCK) {
        if (base) load(base);
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int i = base + u * BLOCK + threadIdx.x;
            if (i < m) {
                const float vi = s_vd[t.row0 + (int)((tg[u] - (uint32_t)t.row0) & 255u)];
                const uint32_t wd[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
                float v[kChunkCols];
#pragma unroll
                for (int e = 0; e < kChunkCols; ++e)
                    v[e] = *(lds_float*)(size_t)(vd_lds + ((e & 1) ? col_hi_bytes(wd[e >> 1]) : col_lo_bytes(wd[e >> 1])));
                float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
                for (int e = 0; e < kChunkCols; e += 2) {
                    const float d0 = vi - v[e], d1 = vi - v[e + 1];
                    const float f0 = pair_factor<SGJ, true>(d0), f1 = pair_factor<SGJ, true>(d1);
                    if (HASW) {
                        const float4 wa = w4[u][e >> 2];
                        a0 = fmaf((e & 2) ? wa.z : wa.x, d0 * f0, a0);
                        a1 = fmaf((e & 2) ? wa.w : wa.y, d1 * f1, a1);
                    } else {
                        a0 = fmaf(d0, f0, a0);
                        a1 = fmaf(d1, f1, a1);
                    }
                }
                s_sums[i] = a0 + a1;
            }
        }
    }
    __syncthreads();
    float part = 0.0f;
    for (int c = lo + oq; c < hi; c += own) part += s_sums[c];
    for (int h = own >> 1; h > 0; h >>= 1) part += __shfl_xor(part, h, 64);
    if (orow < nrows && oq == 0) s_ig[orow] = (HASW ? 1.0f : d.g) * part * kInvPreScale;
}

// Chunked rows that are no flat tiles (networks beyond kFlatCells, tiles whose
// sums do not fit LDS, a surrogate's gap launch): L lanes per row, the
// neighbours' voltages gathered from global memory (from a copy in LDS they were
// no faster at any of 2,000 to 8,192 cells and degrees 50 to 500: 2,000 of 500
// 7.2 us, 7.8 from LDS). Row r's chunks [ca[r], ca[r + 1]), padded with r itself.
template <int BLOCK, bool HASW, bool SGJ>
__device__ __forceinline__ void gap_chunks(const StepArgs& a, const InstDesc& d, const Tile& t,
                                           const float* __restrict__ vd, float* s_part,
                                           float* s_ig) {
    const int L = d.lanes_per_row;
    const int groups = BLOCK / L;
    const int grp = threadIdx.x / L;
    const int lig = threadIdx.x % L;
    const int32_t* ca = a.ca + d.ca_off;
    const uint4* ch = a.chk + d.chk_off;
    const float4* cw = reinterpret_cast<const float4*>(a.chkw) + 2 * d.chk_off;
    for (int r0 = t.row0; r0 < t.row1; r0 += groups) {
        const int r = r0 + grp;
        float acc0 = 0.0f, acc1 = 0.0f;
        if (r < t.row1) {
            const float vi = vd[r];
            const uint4 padc = pad_chunk((uint32_t)r);
            const int ce = ca[r + 1];
            for (int c = ca[r] + lig; c < ce; c += 2 * L) {
                const bool ok1 = c + L < ce;
                const uint4 q0 = ch[c];
                const uint4 q1 = ok1 ? ch[c + L] : padc;
                float4 w4[4];
                if (HASW) {
                    w4[0] = cw[2 * (int64_t)c];
                    w4[1] = cw[2 * (int64_t)c + 1];
                    w4[2] = ok1 ? cw[2 * (int64_t)(c + L)] : make_float4(0.f, 0.f, 0.f, 0.f);
                    w4[3] = ok1 ? cw[2 * (int64_t)(c + L) + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
                chunk_pair_terms<false, HASW, SGJ>(q0, q1, w4, vd, vi, acc0, acc1);
            }
        }
        float acc = acc0 + acc1;
        if (L <= 64) {
            acc = wave_sum_xor(acc, L);
            if (r < t.row1 && lig == 0) s_ig[r - t.row0] = HASW ? acc : d.g * acc;
        } else {
            acc = wave_sum_xor(acc, 64);
            const int wave = threadIdx.x >> 6;
            if ((threadIdx.x & 63) == 0) s_part[wave] = acc;
            __syncthreads();
            if (lig == 0 && r < t.row1) {
                float tot = 0.0f;
                for (int w = 0; w < L / 64; ++w) tot += s_part[wave + w];
                s_ig[r - t.row0] = HASW ? tot : d.g * tot;
            }
            __syncthreads();
        }
    }
}

constexpr int kSelfSlots = 256;     // LDS slots after a column block: the tile rows' own voltages

// Column blocks with chunks: per row and block, the columns relative to the
// block start, padded with S + (r mod 256), S = min(n, C), the LDS slot
// holding row r's own (prescaled) voltage; LDS holds S + kSelfSlots floats.
template <int BLOCK, bool HASW, bool SGJ>
__device__ __forceinline__ void gap_chunks_blocked(const StepArgs& a, const InstDesc& d, const Tile& t,
                                                   const float* __restrict__ vd, float* s_vd, float* s_part,
                                                   float* s_ig) {
    const int L = d.lanes_per_row;
    const int groups = BLOCK / L;
    const int grp = threadIdx.x / L;
    const int lig = threadIdx.x % L;
    const int C = a.blk_cols;
    const int64_t n1 = d.n + 1;
    const int32_t* cb = a.cb + d.cb_off;   // [nblk][n + 1]: block-major chunk starts
    const uint4* ch = a.chk + d.chkb_off;
    const float4* cw = reinterpret_cast<const float4*>(a.chkw) + 2 * d.chkb_off;
    const int S = C;               // own-voltage slots follow the block's C slots
    for (int k = threadIdx.x; k < t.row1 - t.row0; k += BLOCK)
        s_vd[S + ((t.row0 + k) & (kSelfSlots - 1))] = vd[t.row0 + k] * kPreScale;
    float acc[kBlkPasses], vi[kBlkPasses];
#pragma unroll
    for (int q = 0; q < kBlkPasses; ++q) {
        acc[q] = 0.0f;
        const int r = t.row0 + q * groups + grp;
        vi[q] = r < t.row1 ? vd[r] * kPreScale : 0.0f;
    }
    for (int b = 0; b < d.nblk; ++b) {
        const int j0 = b * C;
        const int jn = min(C, d.n - j0);
        __syncthreads();
        for (int k = threadIdx.x; k < jn; k += BLOCK) s_vd[k] = vd[j0 + k] * kPreScale;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBlkPasses; ++q) {
            const int r = t.row0 + q * groups + grp;
            if (r >= t.row1) continue;
            const uint4 padc = pad_chunk((uint32_t)(S + (r & (kSelfSlots - 1))));
            const int ce = cb[b * n1 + r + 1];
            float a0 = 0.0f, a1 = 0.0f;
            for (int c = cb[b * n1 + r] + lig; c < ce; c += 2 * L) {
                const bool ok1 = c + L < ce;
                const uint4 q0 = ch[c];
                const uint4 q1 = ok1 ? ch[c + L] : padc;
                float4 w4[4];
                if (HASW) {
                    w4[0] = cw[2 * (int64_t)c];
                    w4[1] = cw[2 * (int64_t)c + 1];
                    w4[2] = ok1 ? cw[2 * (int64_t)(c + L)] : make_float4(0.f, 0.f, 0.f, 0.f);
                    w4[3] = ok1 ? cw[2 * (int64_t)(c + L) + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
                }
                chunk_pair_terms<true, HASW, SGJ>(q0, q1, w4, s_vd, vi[q], a0, a1);
            }
            acc[q] += a0 + a1;
        }
    }
#pragma unroll
    for (int q = 0; q < kBlkPasses; ++q) {
        const int r = t.row0 + q * groups + grp;
        float v = acc[q];
        if (L <= 64) {
            v = wave_sum_xor(v, L) * kInvPreScale;
            if (r < t.row1 && lig == 0) s_ig[r - t.row0] = HASW ? v : d.g * v;
        } else {
            v = wave_sum_xor(v, 64);
            const int wave = threadIdx.x >> 6;
            __syncthreads();
            if ((threadIdx.x & 63) == 0) s_part[wave] = v;
            __syncthreads();
            if (lig == 0 && r < t.row1) {
                float tot = 0.0f;
                for (int w = 0; w < L / 64; ++w) tot += s_part[wave + w];
                tot *= kInvPreScale;
                s_ig[r - t.row0] = HASW ? tot : d.g * tot;
            }
        }
    }
}

// ---------------------------------------------------------------- chunk stream
// Column blocks read as one flat stream per tile: in the block-major layout
// the chunks of the tile's rows in block b are one contiguous run
// [cb[b][row0], cb[b][row1]). A round is that run, cut at the network's
// round size (kStreamRound or half of it, as the tuner timed them); every
// wave takes a contiguous share of the round's 64-chunk
// sweeps (lane l the l-th chunk of a sweep: one coalesced 1 KB load), in
// pieces of kStreamSweeps sweeps. A one-byte tag per chunk (its row mod 256)
// selects the row's own voltage; the chunk's eight terms go to an LDS slot of
// their own. Waves run a round's pieces without synchronising; at the round's
// end the OWN threads owning each row (lanes of one quad) add that row's
// slots in a fixed order (bitwise reproducible). Two register sets alternate: while one piece is
// summed the next piece's loads are in flight, and the next block's voltages
// load during the current block. kStreamSets register sets rotate, so that
// the loads of kStreamSets - 1 pieces are in flight while one is summed.
constexpr int kStreamSweeps = 4;
constexpr int kStreamSets = 2;
constexpr int kStreamMaxBlocks = 8;    // column blocks whose chunk offsets a tile keeps in LDS
constexpr int kStreamCols = 16384;     // the column block (C) the stream is compiled for
constexpr int kStreamRound = 8192;     // largest round: chunk sums of two rounds fit in LDS
constexpr size_t kStaticLds = 8192;    // bound on k_step's static LDS (s_ig, s_part, s_red)

// LDS floats of a stream tile: block voltages, own voltages, chunk sums of
// two rounds, chunk offsets of every block ([nblk][kSelfSlots + 1] ints).
template <int BLOCK>
__host__ __device__ constexpr int stream_lds_floats(int C) {
    return C + kSelfSlots + 2 * kStreamRound + kStreamMaxBlocks * (kSelfSlots + 1);
}
// chunks the stream may load past a round's end (the arrays carry as many
// zeroed ones): a wave's share is rounded up to whole pieces
constexpr int kStreamSlack = (1024 / 64 + kStreamSweeps) * 64;

// One chunk's eight terms (voltages prescaled, staged in LDS). The staged
// block is the first thing in LDS (the stream variant of k_step has no
// static LDS; the runtime checks it before it offers the stream), so a
// column's LDS address is the column times four, with no base to add.
template <bool SGJ>
__device__ __forceinline__ float chunk_terms(const uint4 q, float vi) {
    const uint32_t wd[4] = {q.x, q.y, q.z, q.w};
    float v[kChunkCols];
#pragma unroll
    for (int e = 0; e < kChunkCols; ++e)
        v[e] = *(lds_float*)(size_t)((e & 1) ? col_hi_bytes(wd[e >> 1]) : col_lo_bytes(wd[e >> 1]));
    float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
    for (int e = 0; e < kChunkCols; e += 2) {
        const float d0 = vi - v[e], d1 = vi - v[e + 1];
        a0 = fmaf(d0, pair_factor<SGJ, true>(d0), a0);
        a1 = fmaf(d1, pair_factor<SGJ, true>(d1), a1);
    }
    return a0 + a1;
}

// One piece of a wave's share of a round: block b (whose run ends at re),
// round [r0, r1), the wave's first sweep s0 and its sweeps in this piece np
// (0..kStreamSweeps), the piece's index in the share and the pieces per
// share; b == nblk: none.
struct StreamPiece {
    int b, re, r0, r1, s0, np, j, npieces;
};

template <int BLOCK, bool SGJ>
__device__ __forceinline__ void gap_stream_blocked(const StepArgs& a, const InstDesc& d, const Tile& t,
                                                   const float* __restrict__ vd, float* s_vd, float* s_ig) {
    constexpr int W = BLOCK / 64;
    constexpr int OWN = BLOCK / kSelfSlots;               // threads owning one row
    constexpr int STAGE = kStreamCols / BLOCK;            // block voltages staged per thread (C = kStreamCols)
    constexpr int SW = kStreamSweeps;
    static_assert(OWN >= 1 && OWN <= 64, "owners per row");
    // chunks per round: the descriptor's (the tuner times kStreamRound and
    // half of it), else kStreamRound; the LDS holds two rounds of kStreamRound
    const int RND = (d.stream_round >= 64 && d.stream_round <= kStreamRound) ? d.stream_round : kStreamRound;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // descriptor fields in registers: read once, not again inside the loop
    // (a load there would wait for the chunk loads in flight)
    const int C = kStreamCols;
    const int n = d.n;
    const int nblk = d.nblk;
    const float g = d.g;
    float* s_self = s_vd + C;                   // row r's own voltage at C + (r mod 256)
    float* s_sums = s_self + kSelfSlots;        // per-chunk sums of a round, rounds alternating buffers
    int* s_off = reinterpret_cast<int*>(s_sums + 2 * kStreamRound);   // [b][i]: chunk start of row row0 + i
    const int64_t n1 = n + 1;
    const int32_t* cb = a.cb + d.cb_off;
    const uint4* ch = a.chk + d.chkb_off;
    const uint8_t* tag = a.rtag + d.chkb_off;
    const int nrows = t.row1 - t.row0;
    const int nr1 = nrows + 1;
    // the tables' loads first (so that storing them waits for them only)
    constexpr int TBL = (kStreamMaxBlocks * (kSelfSlots + 1) + BLOCK - 1) / BLOCK;
    const int ntab = nblk * nr1;
    const float selfv = vd[t.row0 + min((int)threadIdx.x, nrows - 1)];
    int offv[TBL];
#pragma unroll
    for (int u = 0; u < TBL; ++u) {
        const int k = min((int)threadIdx.x + u * BLOCK, ntab - 1);
        const int b = k / nr1, i = k - b * nr1;
        offv[u] = cb[b * n1 + t.row0 + i];
    }
    const int orow = threadIdx.x / OWN, oq = threadIdx.x % OWN;
    const bool owner = orow < nrows;
    float rowacc = 0.0f;

    // Piece bounds are the same in every lane of a wave (made scalar, so that
    // branches on them are scalar: the loads and stores of the pipeline stay
    // in straight-line code and wait only for what they use).
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto piece_of = [&](int b, int re, int r0, int r1, int j) {
        const int nsw = (r1 - r0 + 63) / 64;                 // sweeps of the round
        const int q = (nsw + W - 1) / W;                     // sweeps per wave
        const int s0 = min(nsw, wave * q + j * SW);
        const int np = min(SW, min(nsw, wave * q + q) - s0);
        return StreamPiece{b, re, r0, r1, s0, max(np, 0), j, (q + SW - 1) / SW};
    };
    auto first_round_from = [&](int b0) {    // the first piece of the first round of block b0 or later
        for (int b = b0; b < nblk; ++b) {
            const int r0 = uni(s_off[b * nr1]), re = uni(s_off[b * nr1 + nrows]);
            if (r0 < re) return piece_of(b, re, r0, min(re, r0 + RND), 0);
        }
        return StreamPiece{nblk, 0, 0, 0, 0, 0, 0, 1};
    };
    // within a block from registers only; LDS is read at block changes
    auto next_piece = [&](const StreamPiece& p) {
        if (p.j + 1 < p.npieces) return piece_of(p.b, p.re, p.r0, p.r1, p.j + 1);
        if (p.r1 < p.re) return piece_of(p.b, p.re, p.r1, min(p.re, p.r1 + RND), 0);
        return first_round_from(p.b + 1);
    };
    auto next_block = [&](int b) {     // the next block with chunks after b, nblk if none
        for (++b; b < nblk; ++b)
            if (uni(s_off[b * nr1]) < uni(s_off[b * nr1 + nrows])) return b;
        return nblk;
    };
    // every sweep slot of a piece loads (past its end, chunks the compute
    // skips: the arrays carry kStreamSlack chunks of slack), from one address
    auto load = [&](uint4 (&q)[SW], uint32_t (&tg)[SW], const StreamPiece& p) {
        const int c0 = p.r0 + p.s0 * 64 + lane;
        const uint4* qp = ch + c0;
        const uint8_t* tp = tag + c0;
#pragma unroll
        for (int i = 0; i < SW; ++i) {
            q[i] = qp[i * 64];
            tg[i] = tp[i * 64];
        }
    };
    auto compute = [&](const uint4 (&q)[SW], const uint32_t (&tg)[SW], const StreamPiece& p, float* sums) {
        const int slot = p.s0 * 64 + lane;                  // this lane's slot of sweep 0
        const int m = p.r1 - p.r0;
        float* dst = sums + slot;
        if (p.np == SW && (p.s0 + SW) * 64 <= m) {
            // whole sweeps only (all but a round's last piece): one basic
            // block, in which the scheduler overlaps two sweeps at a time
#pragma unroll
            for (int i = 0; i < SW; ++i) {
                dst[i * 64] = chunk_terms<SGJ>(q[i], s_self[tg[i]]);
                if (i & 1) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < SW; ++i) {
                if (i < p.np) {
                    const float sum = chunk_terms<SGJ>(q[i], s_self[tg[i]]);
                    if (slot + i * 64 < m) dst[i * 64] = sum;
                }
            }
        }
    };
    auto combine = [&](const StreamPiece& p, const float* sums) {
        float part = 0.0f;
        if (owner) {
            const int rlo = max(s_off[p.b * nr1 + orow], p.r0), rhi = min(s_off[p.b * nr1 + orow + 1], p.r1);
            for (int c = rlo + oq; c < rhi; c += OWN) part += sums[c - p.r0];
        }
        // the OWN owners of a row are the lanes of a quad (or half of one):
        // add them through DPP, in wave_sum_xor's order, without a trip to LDS
        static_assert(OWN == 2 || OWN == 4, "owners per row");
        if constexpr (OWN == 4)
            part += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(part), 0x4E, 0xF, 0xF, false));
        part += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(part), 0xB1, 0xF, 0xF, false));
        rowacc += part;
    };
    // all C slots are loaded and stored, past the network's last cell too:
    // the state buffer holds 14 rows of at least n > C / 2 cells after Vd,
    // and no column entry names a slot past the block's end
    // (four voltages per load and store: the network's Vd row starts on a
    // 16-byte boundary, which the runtime requires of stream networks)
    constexpr int STAGE4 = STAGE / 4;
    float4 sv[STAGE4];
    auto load_voltages = [&](int b) {
        const float4* src = reinterpret_cast<const float4*>(vd + b * C) + threadIdx.x;
#pragma unroll
        for (int u = 0; u < STAGE4; ++u) sv[u] = src[u * BLOCK];
    };
    auto store_voltages = [&]() {
        float4* dst = reinterpret_cast<float4*>(s_vd) + threadIdx.x;
#pragma unroll
        for (int u = 0; u < STAGE4; ++u)
            dst[u * BLOCK] = make_float4(sv[u].x * kPreScale, sv[u].y * kPreScale, sv[u].z * kPreScale,
                                         sv[u].w * kPreScale);
    };

    constexpr int NS = kStreamSets;
    uint4 q[NS][SW];
    uint32_t tg[NS][SW];
    StreamPiece prev{-1, 0, 0, 0, 0, 0, 0, 1};   // the round summed last (combined at the next round's start)
    int staged = -1;
    // the first piece when block 0 has chunks: its loads go out before the
    // tables are stored (the bounds from global memory; else after them)
    StreamPiece cur{nblk, 0, 0, 0, 0, 0, 0, 1};
    {
        const int g0 = uni(cb[t.row0]), g1 = uni(cb[t.row1]);
        if (nblk > 0 && g0 < g1) {
            cur = piece_of(0, g1, g0, min(g1, g0 + RND), 0);
            load_voltages(0);
            load(q[0], tg[0], cur);
        }
    }
    if (threadIdx.x < nrows) s_self[(t.row0 + threadIdx.x) & (kSelfSlots - 1)] = selfv * kPreScale;
#pragma unroll
    for (int u = 0; u < TBL; ++u)
        if ((int)threadIdx.x + u * BLOCK < ntab) s_off[threadIdx.x + u * BLOCK] = offv[u];
    __syncthreads();
    if (cur.b >= nblk) {
        cur = first_round_from(1);
        if (cur.b < nblk) {
            load_voltages(cur.b);
            load(q[0], tg[0], cur);
        }
    }
    StreamPiece ahead = cur;                     // the last piece whose loads are queued
#pragma unroll
    for (int k = 1; k < NS - 1; ++k) {
        const StreamPiece nx = ahead.b < nblk ? next_piece(ahead) : ahead;
        ahead = nx;
        if (ahead.b < nblk) load(q[k], tg[k], ahead);
    }
    int rb = 0;                                  // the sums buffer of the current round
    // Sum the piece in set u while set u - 1 (summed last) loads the piece
    // NS - 1 ahead. Every wave has the same pieces per round, so the barriers
    // at round starts match. Rounds alternate between two sums buffers: the
    // previous round's rows are added while the next block is staged.
    auto step = [&](uint4 (&qx)[SW], uint32_t (&tx)[SW], uint4 (&qz)[SW], uint32_t (&tz)[SW]) {
        if (ahead.b < nblk) {
            ahead = next_piece(ahead);
            if (ahead.b < nblk) load(qz, tz, ahead);
        }
        if (cur.j == 0) {
            __syncthreads();                    // the previous round is summed; its voltages are done with
            if (prev.b >= 0) {
                rb ^= 1;
                combine(prev, s_sums + (rb ^ 1) * kStreamRound);
            }
            if (staged != cur.b) {
                store_voltages();
                staged = cur.b;
                __syncthreads();                // the voltages are staged; the previous round's rows added
                const int nb = next_block(cur.b);   // its voltages load during this block
                if (nb < nblk) load_voltages(nb);
            }
        }
        compute(qx, tx, cur, s_sums + rb * kStreamRound);
        prev = cur;
        cur = next_piece(cur);
    };
    while (cur.b < nblk) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            if (cur.b < nblk) step(q[u], tg[u], q[(u + NS - 1) % NS], tg[(u + NS - 1) % NS]);
        }
    }
    __syncthreads();
    if (prev.b >= 0) combine(prev, s_sums + rb * kStreamRound);
    if (owner && oq == 0) s_ig[orow] = g * rowacc * kInvPreScale;
}

// f(std::true_type) for a network with per-edge weights when the launch
// compiles those paths (W), else f(std::false_type).
template <bool W, typename F>
__device__ __forceinline__ void by_weights(const InstDesc& d, F&& f) {
    if constexpr (W) {
        if (d.has_w) {
            f(std::true_type{});
            return;
        }
    }
    f(std::false_type{});
}

// CSR paths of one gap form (SGJ: simplified).
template <int BLOCK, bool SGJ, int VAR>
__device__ __forceinline__ void gap_csr_form(const StepArgs& a, const InstDesc& d, const Tile& t,
                                             const float* __restrict__ vd, float* s_vd, float* s_part,
                                             float* s_ig) {
    constexpr bool W = var_weights(VAR);
    if constexpr (!var_gathers(VAR)) {
        by_weights<W>(d, [&](auto hw) { gap_flat<BLOCK, decltype(hw)::value, SGJ, var_vd_first(VAR)>(a, d, t, vd, s_vd, s_ig); });
    } else {
        // column-blocked tiles run in the wide launch group only (512- or
        // 1024-thread workgroups; the runtime places them there); elsewhere the
        // same rows take the gathers below
        if constexpr (BLOCK >= 512) {
            if (d.blocked && d.cb_off >= 0) {
                by_weights<W>(d, [&](auto hw) {
                    gap_chunks_blocked<BLOCK, decltype(hw)::value, SGJ>(a, d, t, vd, s_vd, s_part, s_ig);
                });
                return;
            }
        }
        if (d.flat) {
            by_weights<W>(d, [&](auto hw) { gap_flat<BLOCK, decltype(hw)::value, SGJ, var_vd_first(VAR)>(a, d, t, vd, s_vd, s_ig); });
            return;
        }
        const bool chunks = d.chunked && d.ca_off >= 0;
        if (d.vd_lds && !chunks) {
            for (int k = threadIdx.x; k < d.n; k += BLOCK) s_vd[k] = vd[k] * kPreScale;
            __syncthreads();
        }
        by_weights<W>(d, [&](auto hw) {
            constexpr bool HW = decltype(hw)::value;
            if (chunks) {
                gap_chunks<BLOCK, HW, SGJ>(a, d, t, vd, s_part, s_ig);
            } else if (d.vd_lds) {
                if (d.col16) gap_csr_impl<BLOCK, true, true, HW, SGJ>(a, d, t, vd, s_vd, s_part, s_ig);
                else gap_csr_impl<BLOCK, true, false, HW, SGJ>(a, d, t, vd, s_vd, s_part, s_ig);
            } else {
                if (d.col16) gap_csr_impl<BLOCK, false, true, HW, SGJ>(a, d, t, vd, s_vd, s_part, s_ig);
                else gap_csr_impl<BLOCK, false, false, HW, SGJ>(a, d, t, vd, s_vd, s_part, s_ig);
            }
        });
    }
}

template <int BLOCK, int VAR>
__device__ __forceinline__ void gap_csr(const StepArgs& a, const InstDesc& d, const Tile& t,
                                        const float* __restrict__ vd, float* s_vd, float* s_part,
                                        float* s_ig) {
    if (d.sgj) gap_csr_form<BLOCK, true, VAR>(a, d, t, vd, s_vd, s_part, s_ig);
    else gap_csr_form<BLOCK, false, VAR>(a, d, t, vd, s_vd, s_part, s_ig);
}

// Bitmap words of a network: group gr (128 senders), row r (padded to a
// multiple of 16 rows), block p (senders gr*128 + 32p .. +31): word
// (gr * n_pad16 + r) * 4 + p, bit t = sender gr*128 + 32p + t. LDS holds a
// chunk of prescaled Vd, contiguous.
constexpr int kBitGroup = 128;
constexpr int kBitRows = 16;
constexpr int kBitChunkGroups = kChunk / kBitGroup;            // 64 groups per LDS chunk

__host__ __device__ __forceinline__ int bitmap_rows_pad(int n) { return (n + kBitRows - 1) / kBitRows * kBitRows; }

template <int BLOCK>
__device__ __forceinline__ void gap_bitmap(const StepArgs& a, const InstDesc& d, const Tile& t,
                                           const float* __restrict__ vd, float* s_v, float* s_part,
                                           float* s_ig) {
    // Lanes are senders, the tile's 16 rows are wave-uniform: row r's 64-bit
    // coupling word for 64 senders is a scalar load and masks the pair term
    // as the lane mask of one select.
    constexpr int W = BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = d.n;
    const int npad = bitmap_rows_pad(n);
    const int groups = (n + kBitGroup - 1) / kBitGroup;
    const int nrows = t.row1 - t.row0;
    float vis[kBitRows];
    float acc[kBitRows];
#pragma unroll
    for (int r = 0; r < kBitRows; ++r) {
        vis[r] = r < nrows ? vd[t.row0 + r] * kPreScale : 0.0f;
        acc[r] = 0.0f;
    }
    // words of the tile's rows in group gr: 16 rows x 4 words, contiguous
    const uint32_t* bits = a.bits + d.bits_off + (int64_t)t.row0 * 4;
    for (int g0 = 0; g0 < groups; g0 += kBitChunkGroups) {
        const int gc = min(kBitChunkGroups, groups - g0);
        __syncthreads();
        for (int k = threadIdx.x; k < gc * kBitGroup; k += BLOCK) {
            const int j = g0 * kBitGroup + k;
            s_v[k] = j < n ? vd[j] * kPreScale : kSentinel;
        }
        __syncthreads();
        const int per = (gc + W - 1) / W;
        const int gb = wave * per, ge = min(gc, gb + per);
        for (int gl = gb; gl < ge; ++gl) {
            // qword 2r + h: row r's senders (g0 + gl) * 128 + 64h + (0..63);
            // the bitmap is not written while a step runs, so it is read
            // through the constant address space (scalar loads)
            const auto wq = (const __attribute__((address_space(4))) uint64_t*)(
                bits + (int64_t)(g0 + gl) * npad * 4);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float vj = s_v[gl * kBitGroup + 64 * h + lane];
#pragma unroll
                for (int r = 0; r < kBitRows; ++r) {
                    const float dv = vis[r] - vj;
                    const float f = fmaf(0.8f, __builtin_amdgcn_exp2f(-(dv * dv)), 0.2f);
                    const float dm = __builtin_amdgcn_inverse_ballot_w64(wq[2 * r + h]) ? dv : 0.0f;
                    acc[r] = fmaf(dm, f, acc[r]);
                }
            }
        }
    }
    // Sum each row over the 64 lanes: four exchanges that halve the values
    // a lane holds (a lane with bit b of its index set keeps the upper half)
    // leave lane l with row (l & 15) summed over its 16-lane group; two
    // more add the four groups.
    float v8[8], v4[4], v2[2];
    {
        const bool up = lane & 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float keep = up ? acc[i + 8] : acc[i], send = up ? acc[i] : acc[i + 8];
            v8[i] = keep + __shfl_xor(send, 8, 64);
        }
    }
    {
        const bool up = lane & 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float keep = up ? v8[i + 4] : v8[i], send = up ? v8[i] : v8[i + 4];
            v4[i] = keep + __shfl_xor(send, 4, 64);
        }
    }
    {
        const bool up = lane & 2;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float keep = up ? v4[i + 2] : v4[i], send = up ? v4[i] : v4[i + 2];
            v2[i] = keep + __shfl_xor(send, 2, 64);
        }
    }
    float v1;
    {
        const bool up = lane & 1;
        const float keep = up ? v2[1] : v2[0], send = up ? v2[0] : v2[1];
        v1 = keep + __shfl_xor(send, 1, 64);
    }
    v1 += __shfl_xor(v1, 16, 64);
    v1 += __shfl_xor(v1, 32, 64);
    if (lane < kBitRows) s_part[wave * kBitRows + lane] = v1;
    __syncthreads();
    if (threadIdx.x < kBitRows && t.row0 + (int)threadIdx.x < t.row1) {
        float tot = 0.0f;
        for (int w = 0; w < W; ++w) tot += s_part[w * kBitRows + threadIdx.x];
        s_ig[threadIdx.x] = d.g * (tot * kInvPreScale);
    }
}

// Evoked input of a cell at a step, `iapp` its bias.
__device__ __forceinline__ float evoked_from(float iapp, const StepArgs& a, const InstDesc& d, int64_t step, int li) {
    if (step >= d.p0_n0 && step < d.p0_n1 && li >= d.p0_c0 && li < d.p0_c1) iapp += d.p0_amp;
    for (int k = 1; k < d.n_pulses; ++k) {
        const DevPulse pl = a.pulses[d.pulse_off + k];
        if (step >= pl.n0 && step < pl.n1 && li >= pl.c0 && li < pl.c1) iapp += pl.amp;
    }
    if (d.stream_off >= 0 && step >= 0 && step < d.stream_steps)
        iapp += a.i_stream[d.stream_off + step * (int64_t)d.n + li];
    return iapp;
}
__device__ __forceinline__ float evoked_input(const StepArgs& a, const InstDesc& d, int64_t step,
                                              int li, int64_t cell) {
    return evoked_from(a.bias[cell], a, d, step, li);
}

template <int BLOCK, int VAR>
__device__ __forceinline__ void step_body(const StepArgs& a, const float* __restrict__ xin, float* __restrict__ xout,
                                          int64_t step_arg, int32_t step_off, float* s_ig, float* s_part,
                                          double* s_red, float4* s_v4) {
    const Tile t = a.tiles[blockIdx.x];
    const InstDesc& d = a.inst[t.inst];
    const int64_t step = (a.d_step ? *a.d_step : step_arg) + step_off;
    const float* vd = xin + (int64_t)SV_VD * a.stride + t.cell_off;
    const int nrows = t.row1 - t.row0;

    // The compartment update of cell row0 + k: with at most 64 rows, lane k
    // of wave 0 advances its dendrite and axon and lane k of wave 1 its soma
    // (the update is Jacobi, so the parts are independent and their
    // arithmetic is cell_step's); else thread k advances the whole cell.
    // State loads are issued first so their latency overlaps the gap work.
    const bool split = nrows <= 64;
    const int k_own = split ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    const int part = split ? (int)(threadIdx.x >> 6) : 0;   // 0: dendrite + axon (or all), 1: soma
    const bool own = k_own < nrows && part < 2 && !a.gap_only;
    const int li = t.row0 + k_own;
    const int64_t cell = t.cell_off + li;
    float x[NSV];
    float iapp = 0.0f;
    if (own) {
#pragma unroll
        for (int v = 0; v < NSV; ++v) x[v] = xin[v * a.stride + cell];
        iapp = evoked_input(a, d, step, li, cell);
    }

    if constexpr (VAR == kVarStream) {
        if (d.sgj) gap_stream_blocked<BLOCK, true>(a, d, t, vd, reinterpret_cast<float*>(s_v4), s_ig);
        else gap_stream_blocked<BLOCK, false>(a, d, t, vd, reinterpret_cast<float*>(s_v4), s_ig);
    } else if constexpr (VAR == kVarNoGap) {
        for (int k = threadIdx.x; k < nrows; k += BLOCK) s_ig[k] = 0.0f;
    } else if constexpr (VAR == kVarDense) {
        if (d.conn != CONN_DENSE) {
            for (int k = threadIdx.x; k < nrows; k += BLOCK) s_ig[k] = 0.0f;
        } else if (d.sgj) {
            gap_dense<BLOCK, true>(a, d, t, vd, s_part, s_ig);
        } else {
            gap_dense<BLOCK, false>(a, d, t, vd, s_part, s_ig);
        }
    } else {
        switch (d.conn) {
            case CONN_UNIFORM:
                if (d.sgj && d.sym) {
                    gap_uniform_sum<BLOCK>(a, d, t, vd, s_ig, s_red);
                    break;
                }
                if constexpr (var_uniform(VAR)) {
                    if (d.grid) gap_uniform_grid<BLOCK>(a, d, t, vd, s_ig, s_part, s_red, reinterpret_cast<double*>(s_v4));
                    else gap_uniform<BLOCK>(a, d, t, vd, s_ig, s_v4, s_part, s_red);
                }
                break;
            case CONN_DENSE:
                if constexpr (VAR == kVarAll) {
                    if (d.sgj) gap_dense<BLOCK, true>(a, d, t, vd, s_part, s_ig);
                    else gap_dense<BLOCK, false>(a, d, t, vd, s_part, s_ig);
                }
                break;
            case CONN_CSR:
                if constexpr (var_gathers(VAR)) {
                    if (d.bitmap) {
                        gap_bitmap<BLOCK>(a, d, t, vd, reinterpret_cast<float*>(s_v4), s_part, s_ig);
                        break;
                    }
                }
                gap_csr<BLOCK, VAR>(a, d, t, vd, reinterpret_cast<float*>(s_v4), s_part, s_ig);
                break;
            default:
                for (int k = threadIdx.x; k < nrows; k += BLOCK) s_ig[k] = 0.0f;
                break;
        }
    }
    __syncthreads();

    if (a.gap_only) {
        for (int k = threadIdx.x; k < nrows; k += BLOCK) a.igap_out[t.cell_off + t.row0 + k] = s_ig[k];
        return;
    }
    // per-cell parameters exist in the var_cells variants only (the runtime
    // launches networks that have them with those)
    CellParams pc = d.p;
    if constexpr (var_cells(VAR)) {
        if (own) pc = cell_params_of(a, d, cell);
    }
    if (own && split) {
        float y[NSV];
        float chk = 0.0f;
        if (part == 0) {
            cell_step_dendrite(pc, x, s_ig[k_own], iapp, a.dt, y);
            cell_step_axon(pc, x, a.dt, y);
#pragma unroll
            for (int v : {SV_VD, SV_CA, SV_R, SV_S, SV_Q, SV_VA, SV_HA, SV_XA}) {
                xout[v * a.stride + cell] = y[v];
                chk += y[v];
            }
        } else {
            cell_step_soma(pc, x, a.dt, y);
#pragma unroll
            for (int v : {SV_VS, SV_K, SV_L, SV_H, SV_N, SV_X}) {
                xout[v * a.stride + cell] = y[v];
                chk += y[v];
            }
        }
        if (a.dry) return;
        if (!isfinite(chk)) atomicOr(a.flags, 1);
        if (part == 0 && a.out_slots) a.out_ring[out_slot(a, step) + cell] = y[SV_VA];
        // axon output (wave 0): upward 0 mV crossing, time interpolated within the step
        if (part == 0 && x[SV_VA] < 0.0f && y[SV_VA] >= 0.0f) {
            const int c = a.spike_count[cell];
            if (a.spike_cap > 0) {
                const float frac = (0.0f - x[SV_VA]) / (y[SV_VA] - x[SV_VA]);
                a.spike_times[cell * a.spike_cap + (c % a.spike_cap)] = ((float)step + frac) * a.dt;
            }
            a.spike_count[cell] = c + 1;
        }
    } else if (own) {
        float y[NSV];
        cell_step(pc, x, s_ig[k_own], iapp, a.dt, y);
        float chk = 0.0f;
#pragma unroll
        for (int v = 0; v < NSV; ++v) {
            xout[v * a.stride + cell] = y[v];
            chk += y[v];
        }
        if (a.dry) return;
        if (!isfinite(chk)) atomicOr(a.flags, 1);
        if (a.out_slots) a.out_ring[out_slot(a, step) + cell] = y[SV_VA];
        // axon output: upward 0 mV crossing, time interpolated within the step
        if (x[SV_VA] < 0.0f && y[SV_VA] >= 0.0f) {
            const int c = a.spike_count[cell];
            if (a.spike_cap > 0) {
                const float frac = (0.0f - x[SV_VA]) / (y[SV_VA] - x[SV_VA]);
                a.spike_times[cell * a.spike_cap + (c % a.spike_cap)] = ((float)step + frac) * a.dt;
            }
            a.spike_count[cell] = c + 1;
        }
    }
}

// The step. Vd staging in dynamic LDS, sized per launch: the largest
// all-to-all chunk (min(n, kChunk) + 8 per wave), the grid's sums, the largest
// flat tile or the largest LDS-staged CSR network. The chunk stream variant has no static LDS, so its staged
// voltages start at LDS address 0 (a gather's address is its column times
// four, with no base to add) and its row sums follow the stream's region; the
// same holds for the var_vd_first variants.
template <int BLOCK, int VAR = kVarAll>
__global__ __launch_bounds__(BLOCK, var_waves(VAR)) void k_step(StepArgs a, const float* __restrict__ xin,
                                                float* __restrict__ xout, int64_t step_arg,
                                                int32_t step_off) {
    extern __shared__ float4 s_v4[];
    if constexpr (VAR == kVarStream) {
        float* s_ig = reinterpret_cast<float*>(s_v4) + stream_lds_floats<BLOCK>(kStreamCols);
        step_body<BLOCK, VAR>(a, xin, xout, step_arg, step_off, s_ig, nullptr, nullptr, s_v4);
    } else if constexpr (var_vd_first(VAR)) {
        double* s_red = reinterpret_cast<double*>(reinterpret_cast<float*>(s_v4) + a.lds_floats);
        float* s_part = reinterpret_cast<float*>(s_red + BLOCK / 64);
        step_body<BLOCK, VAR>(a, xin, xout, step_arg, step_off, s_part + BLOCK, s_part, s_red, s_v4);
    } else {
        __shared__ float s_ig[kMaxTileRows];
        __shared__ float s_part[BLOCK];
        __shared__ double s_red[BLOCK / 64];
        step_body<BLOCK, VAR>(a, xin, xout, step_arg, step_off, s_ig, s_part, s_red, s_v4);
    }
}

static __global__ void k_set_step(int64_t* d_step, int64_t value) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *d_step = value;
}

}  // namespace infoli
