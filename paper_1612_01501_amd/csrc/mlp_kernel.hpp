// Learned surrogate of the cell update: an MLP 16 -> 128 -> 128 -> 16 (SiLU)
// that advances a cell by one macro step of four time steps. Weights are
// BF16 and every product runs on the matrix cores (v_mfma_f32_16x16x16_bf16)
// with FP32 accumulation, batched over cells so each layer is a GEMM.
//
// Layout: a wave owns 16 samples (cells). Activations are kept transposed,
// H^T [features x 16 samples], so the accumulator layout of one layer
// (lane j + 16*(i/4) holds rows i..i+3 of column j) is exactly the B-operand
// layout of the next (lane j + 16*(k/4) holds k..k+3 of column j): no data
// moves between layers. Weights W [out][in] are the A operand, read from LDS
// (row i at lane i%16, four consecutive k per lane).
//
// Parameter order (flat fp32): W1[128][16] b1[128] W2[128][128] b2[128]
// W3[16][128] b3[16].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace infoli {

constexpr int kIn = 16, kHid = 128, kOut = 16, kTargets = 14;
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kHid * kIn, kOffW2 = kOffB1 + kHid,
              kOffB2 = kOffW2 + kHid * kHid, kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kOut * kHid,
              kNumParams = kOffB3 + kOut;                    // 20,752
// LDS row strides (bf16 elements), padded against bank conflicts
constexpr int kS1 = kIn + 4, kS2 = kHid + 4, kS3 = kHid + 4;
constexpr int kLdsW1 = kHid * kS1, kLdsW2 = kHid * kS2, kLdsW3 = kOut * kS3;
constexpr int kMlpLdsElems = kLdsW1 + kLdsW2 + kLdsW3;     // bf16 elements (42 KB)

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// fp32 -> bf16 by the hardware conversion (v_cvt_pk_bf16_f32: round to
// nearest even, two values per instruction; NaN stays NaN)
typedef __bf16 hbf16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x4 pack_bf16(f32x4 v) {
    const hbf16x4 h = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
    return __builtin_bit_cast(bf16x4, h);
}

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

typedef short bf16x8s __attribute__((ext_vector_type(8)));
typedef __bf16 hbf16x8 __attribute__((ext_vector_type(8)));

// D += A B over 32 of K (v_mfma_f32_16x16x32_bf16, one instruction for two
// 16x16x16 products). Both operands hold, per lane, eight K slots that the
// instruction pairs up between A and B; the sum over K does not depend on
// which K each slot carries, so the slots take two 16-wide fragments side by
// side: (a0, b0) for K rows k0.. and (a1, b1) for K rows k0 + 16.. in the
// 16x16x16 layout. No activation moves between layers.
__device__ __forceinline__ f32x4 mfma32(bf16x4 a0, bf16x4 a1, bf16x4 b0, bf16x4 b1, f32x4 c) {
    const bf16x8s a = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
    const bf16x8s b = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(hbf16x8, a),
                                                   __builtin_bit_cast(hbf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ float sigmoid_f(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_f(z); }
__device__ __forceinline__ float silu_grad_f(float z) {
    const float s = sigmoid_f(z);
    return s * (1.0f + z * (1.0f - s));
}

struct MlpSmem {
    uint16_t* w1;   // [128][kS1]
    uint16_t* w2;   // [128][kS2]
    uint16_t* w3;   // [16][kS3]
};

__device__ __forceinline__ MlpSmem mlp_smem(uint16_t* base) {
    return MlpSmem{base, base + kLdsW1, base + kLdsW1 + kLdsW2};
}

// Copy the bf16 weights (dense [out][in] in global memory) into padded LDS,
// four weights (8 bytes) per access, eight loads in flight per thread before
// their stores. Every matrix offset and padded row start is a multiple of
// four weights.
template <int ROWS, int COLS, int S>
__device__ __forceinline__ void copy_matrix_lds(const uint16_t* __restrict__ src, uint16_t* dst) {
    constexpr int kChunks = ROWS * COLS / 4, kPerRow = COLS / 4, kUnroll = 8;
    const uint2* g = reinterpret_cast<const uint2*>(src);
    for (int e0 = threadIdx.x; e0 < kChunks; e0 += kUnroll * blockDim.x) {
        uint2 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = e0 + u * blockDim.x;
            if (e < kChunks) v[u] = g[e];
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int e = e0 + u * blockDim.x;
            if (e < kChunks) *reinterpret_cast<uint2*>(dst + (e / kPerRow) * S + 4 * (e % kPerRow)) = v[u];
        }
    }
}

__device__ __forceinline__ void load_weights_lds(const uint16_t* __restrict__ wb, MlpSmem s) {
    copy_matrix_lds<kHid, kIn, kS1>(wb + kOffW1, s.w1);
    copy_matrix_lds<kHid, kHid, kS2>(wb + kOffW2, s.w2);
    copy_matrix_lds<kOut, kHid, kS3>(wb + kOffW3, s.w3);
}

// A operand: rows rb*16 .. +15 of W (stride S), columns kb*16 + 4*(lane/16) .. +3
__device__ __forceinline__ bf16x4 a_rows(const uint16_t* w, int S, int rb, int kb) {
    const int l = threadIdx.x & 63;
    return *reinterpret_cast<const bf16x4*>(w + (rb * 16 + (l & 15)) * S + kb * 16 + 4 * (l >> 4));
}

// A operand of the transpose: A[i][k] = W[k][i] for rows ib*16.. of W^T
__device__ __forceinline__ bf16x4 a_cols(const uint16_t* w, int S, int ib, int kb) {
    const int l = threadIdx.x & 63;
    const int i = ib * 16 + (l & 15), k = kb * 16 + 4 * (l >> 4);
    bf16x4 r;
    r[0] = (short)w[(k + 0) * S + i];
    r[1] = (short)w[(k + 1) * S + i];
    r[2] = (short)w[(k + 2) * S + i];
    r[3] = (short)w[(k + 3) * S + i];
    return r;
}

// Bias of the four accumulator rows a lane holds in output block ob.
__device__ __forceinline__ f32x4 bias4(const float* b, int ob) {
    const int l = threadIdx.x & 63;
    return *reinterpret_cast<const f32x4*>(b + ob * 16 + 4 * (l >> 4));
}

// Forward pass of one wave. bx: B operand X^T (features 4*(lane/16).. of
// sample lane%16).
__device__ __forceinline__ f32x4 mlp_forward(MlpSmem s, const float* __restrict__ params, bf16x4 bx) {
    bf16x4 h1[8];
#pragma unroll
    for (int ob = 0; ob < 8; ++ob) {
        f32x4 z = mfma16(a_rows(s.w1, kS1, ob, 0), bx, bias4(params + kOffB1, ob));
        f32x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_f(z[e]);
        h1[ob] = pack_bf16(h);
    }
    bf16x4 h2[8];
#pragma unroll
    for (int ob = 0; ob < 8; ++ob) {
        f32x4 z = bias4(params + kOffB2, ob);
#pragma unroll
        for (int kb = 0; kb < 8; kb += 2)
            z = mfma32(a_rows(s.w2, kS2, ob, kb), a_rows(s.w2, kS2, ob, kb + 1), h1[kb], h1[kb + 1], z);
        f32x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_f(z[e]);
        h2[ob] = pack_bf16(h);
    }
    f32x4 y = bias4(params + kOffB3, 0);
#pragma unroll
    for (int kb = 0; kb < 8; kb += 2)
        y = mfma32(a_rows(s.w3, kS3, 0, kb), a_rows(s.w3, kS3, 0, kb + 1), h2[kb], h2[kb + 1], y);
    return y;   // lane holds outputs 4*(lane/16)..+3 of sample lane%16
}

// Weight copies for the matrix cores: bf16 of the fp32 masters.
static __global__ void k_mlp_to_bf16(const float* __restrict__ params, uint16_t* __restrict__ wb) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < kNumParams) wb[e] = to_bf16(params[e]);
}

// ---------------------------------------------------------------- training
// Transposed activations written by the forward/backward pass, read by the
// weight-gradient products: tiles of 16 features x 16 samples (512 contiguous
// bytes, sample fastest), a feature block's tiles in sample order, so that a
// wave of either kernel moves whole tiles.
struct TrainBufs {
    uint16_t* xT;     // [1][B/16][16][16]
    uint16_t* h1T;    // [8][B/16][16][16]
    uint16_t* h2T;    // [8]
    uint16_t* dyT;    // [1]
    uint16_t* dz2T;   // [8]
    uint16_t* dz1T;   // [8]
    float* loss_part; // [B/16] sums of squared errors of 16 samples
};

// Counter-based index draw: SplitMix64 finaliser (Steele, Lea, Flood 2014)
// of a key mixing the seed, the step and the position in the batch.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Forward, loss and back-propagation down to dz1, 16 samples at a time: the
// workgroup's eight waves take one block of 16 hidden features each, of every
// layer and both directions, and pass the activations on through LDS. The
// weights come from the fp32 masters, through LDS once; a wave keeps the
// operands of its feature block in registers for all its samples.
// Sample p of the batch is row idx(p) of the normalised data set (xn, tn:
// [N][16] fp32); idx(p) = p when seed == 0, else a hashed draw.
//
// Bound by latency: one read of the weights (82 KB from L2) and five dependent
// products. A wave that took 16 samples alone through all blocks left 3/4 of
// the waves' slots empty at a batch of 4,096 and needed the masters rounded by
// a kernel before (together 15.3 us; now 7.5).
constexpr int kFwdBwdBlock = 64 * (kHid / 16);

static __global__ __launch_bounds__(kFwdBwdBlock, 2) void k_mlp_fwd_bwd(const float* __restrict__ params,
                                                                 const float* __restrict__ xn,
                                                                 const float* __restrict__ tn, int64_t n_data,
                                                                 int batch, uint64_t seed, uint64_t step,
                                                                 TrainBufs buf) {
    __shared__ __align__(16) uint16_t s_w[kMlpLdsElems];
    __shared__ bf16x4 s_h1[8][64], s_h2[8][64], s_dz2[8][64];   // B operands by feature block
    const MlpSmem s = mlp_smem(s_w);
    const int l = threadIdx.x & 63;
    const int g = l >> 4;                       // feature group of this lane
    const int w = threadIdx.x >> 6;             // feature block of this wave
    const int nb = batch / 16;

    struct Sample {
        f32x4 x, t;
    };
    const auto load = [&](int sb) {
        const int p = sb * 16 + (l & 15);       // position in the batch
        const int64_t row = seed ? (int64_t)(mix64(seed ^ (step << 32) ^ (uint64_t)p) % (uint64_t)n_data) : p;
        return Sample{*reinterpret_cast<const f32x4*>(xn + row * 16 + 4 * g),
                      *reinterpret_cast<const f32x4*>(tn + row * 16 + 4 * g)};
    };

    // four weights per thread and access, all of them in flight
    constexpr int kPer2 = kHid * kHid / 4 / kFwdBwdBlock;
    static_assert(kHid * kIn / 4 == kFwdBwdBlock && kOut * kHid / 4 == kFwdBwdBlock, "one access per thread");
    const f32x4* m1 = reinterpret_cast<const f32x4*>(params + kOffW1);
    const f32x4* m2 = reinterpret_cast<const f32x4*>(params + kOffW2);
    const f32x4* m3 = reinterpret_cast<const f32x4*>(params + kOffW3);
    f32x4 v2[kPer2];
    const f32x4 v1 = m1[threadIdx.x], v3 = m3[threadIdx.x];
#pragma unroll
    for (int u = 0; u < kPer2; ++u) v2[u] = m2[threadIdx.x + u * kFwdBwdBlock];
    Sample cur = load(min((int)blockIdx.x, nb - 1));
    const f32x4 b1 = bias4(params + kOffB1, w), b2 = bias4(params + kOffB2, w), b3 = bias4(params + kOffB3, 0);
    const auto put_w = [&](uint16_t* dst, int S, int cols, int e, f32x4 v) {
        *reinterpret_cast<bf16x4*>(dst + (e / (cols / 4)) * S + 4 * (e % (cols / 4))) = pack_bf16(v);
    };
    put_w(s.w1, kS1, kIn, threadIdx.x, v1);
    put_w(s.w3, kS3, kHid, threadIdx.x, v3);
#pragma unroll
    for (int u = 0; u < kPer2; ++u) put_w(s.w2, kS2, kHid, threadIdx.x + u * kFwdBwdBlock, v2[u]);
    __syncthreads();

    const bf16x4 w1r = a_rows(s.w1, kS1, w, 0), w3c = a_cols(s.w3, kS3, w, 0);
    bf16x4 w2r[8], w2c[8], w3r[8];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
        w2r[kb] = a_rows(s.w2, kS2, w, kb);
        w3r[kb] = a_rows(s.w3, kS3, 0, kb);
        w2c[kb] = a_cols(s.w2, kS2, w, kb);
    }
    const float scale = 2.0f / (float)(batch * kTargets);

    // An exchange buffer is written again one barrier or more after every wave
    // has read it: its readers pass the next buffer's barrier first.
    for (int sb = blockIdx.x; sb < nb; sb += gridDim.x) {
        const auto put = [&](uint16_t* dst, int fb, bf16x4 v) {
            uint16_t* tile = dst + ((int64_t)fb * nb + sb) * 256 + 64 * g + (l & 15);
#pragma unroll
            for (int e = 0; e < 4; ++e) tile[16 * e] = (uint16_t)v[e];
        };
        const f32x4 tv = cur.t;
        const bf16x4 bx = pack_bf16(cur.x);
        if (sb + (int)gridDim.x < nb) cur = load(sb + gridDim.x);

        const f32x4 z1 = mfma16(w1r, bx, b1);
        f32x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_f(z1[e]);
        const bf16x4 h1 = pack_bf16(h);
        s_h1[w][l] = h1;
        __syncthreads();

        f32x4 z2 = b2;
#pragma unroll
        for (int kb = 0; kb < 8; kb += 2) z2 = mfma32(w2r[kb], w2r[kb + 1], s_h1[kb][l], s_h1[kb + 1][l], z2);
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_f(z2[e]);
        const bf16x4 h2 = pack_bf16(h);
        s_h2[w][l] = h2;
        put(buf.h1T, w, h1);
        __syncthreads();

        // every wave the outputs: each needs their errors
        f32x4 y = b3;
#pragma unroll
        for (int kb = 0; kb < 8; kb += 2) y = mfma32(w3r[kb], w3r[kb + 1], s_h2[kb][l], s_h2[kb + 1][l], y);
        // loss = mean over batch and the 14 targets of (y - t)^2
        f32x4 dy;
        float sq = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool on = 4 * g + e < kTargets;
            const float d = on ? y[e] - tv[e] : 0.0f;
            sq += d * d;
            dy[e] = d * scale;
        }
        const bf16x4 dyq = pack_bf16(dy);

        // dz2 = (W3^T dy) * silu'(z2)
        const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        f32x4 dh = mfma16(w3c, dyq, zero), dz;
#pragma unroll
        for (int e = 0; e < 4; ++e) dz[e] = dh[e] * silu_grad_f(z2[e]);
        const bf16x4 dz2 = pack_bf16(dz);
        s_dz2[w][l] = dz2;
        put(buf.h2T, w, h2);
        __syncthreads();

        // dz1 = (W2^T dz2) * silu'(z1)
        dh = zero;
#pragma unroll
        for (int kb = 0; kb < 8; kb += 2) dh = mfma32(w2c[kb], w2c[kb + 1], s_dz2[kb][l], s_dz2[kb + 1][l], dh);
#pragma unroll
        for (int e = 0; e < 4; ++e) dz[e] = dh[e] * silu_grad_f(z1[e]);
        put(buf.dz2T, w, dz2);
        put(buf.dz1T, w, pack_bf16(dz));
        if (w == 0) {
            put(buf.xT, 0, bx);
            for (int m = 32; m > 0; m >>= 1) sq += __shfl_xor(sq, m, 64);
            if (l == 0) buf.loss_part[sb] = sq;
        }
        if (w == 1) put(buf.dyT, 0, dyq);
    }
}

// Weight and bias gradients as products over the batch: one workgroup per
// 16x16 output tile (dW1 8, dW2 64, dW3 8), its sixteen waves a slice of the
// batch each (split K), whose sums it adds in slice order through LDS
// (deterministic). The workgroups of a bias row's first tile sum it as well, as
// a product with a ones vector. `splits` such workgroups per tile share a
// large batch; each then writes a partial gradient [splits][kNumParams], and
// the workgroups of a split are neighbours modulo eight, so that one XCD's L2
// holds its part of the activations for all tiles.
//
// Bound by what the XCDs read of the activations that others wrote (4,096
// samples: 1.6 MB each). The slices as workgroups of one wave, their partials
// added by a kernel of its own, took 13.7 us there (now 6.0), and 57 us at
// 32,768 (now 19).
constexpr int kGradTiles = 8 + 64 + 8;
constexpr int kGradWaves = 16;
constexpr int kGradLoads = 8;        // tiles of each operand in flight per wave

static __global__ __launch_bounds__(64 * kGradWaves, 8) void k_mlp_wgrad(TrainBufs buf, int batch, int splits,
                                                               float* __restrict__ grad_part,
                                                               float* __restrict__ loss_out) {
    __shared__ f32x4 s_acc[kGradWaves][64];
    __shared__ float s_bias[kGradWaves][16];
    const int t = blockIdx.x / splits;
    const int split = blockIdx.x % splits;
    float* grad = grad_part + (int64_t)split * kNumParams;
    const int l = threadIdx.x & 63;
    const int g = l >> 4;
    const int w = threadIdx.x >> 6;
    const int nb = batch / 16;
    const uint16_t *A, *Bm;      // feature blocks of [B/16] tiles
    int ib, jb, ncols, off, off_b;
    if (t < 8) {                 // dW1 = dz1^T x : [128][16]
        A = buf.dz1T; Bm = buf.xT; ib = t; jb = 0; ncols = kIn; off = kOffW1; off_b = kOffB1;
    } else if (t < 72) {         // dW2 = dz2^T h1 : [128][128]
        A = buf.dz2T; Bm = buf.h1T; ib = (t - 8) / 8; jb = (t - 8) % 8; ncols = kHid; off = kOffW2; off_b = kOffB2;
    } else {                     // dW3 = dy^T h2 : [16][128]
        A = buf.dyT; Bm = buf.h2T; ib = 0; jb = t - 72; ncols = kHid; off = kOffW3; off_b = kOffB3;
    }
    const bool bias = jb == 0;
    const bf16x4 ones = {(short)0x3f80, (short)0x3f80, (short)0x3f80, (short)0x3f80};
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, accb = acc;
    const uint16_t* at = A + (int64_t)ib * nb * 256 + (l & 15) * 16 + 4 * g;
    const uint16_t* bt = Bm + (int64_t)jb * nb * 256 + (l & 15) * 16 + 4 * g;
    const int64_t slices = (int64_t)splits * kGradWaves, slice = split * kGradWaves + w;
    const int k0 = (int)(slice * nb / slices), k1 = (int)((slice + 1) * nb / slices);
    for (int k = k0; k < k1; k += kGradLoads) {
        bf16x4 av[kGradLoads], bv[kGradLoads];
#pragma unroll
        for (int u = 0; u < kGradLoads; ++u) {
            const int64_t kk = min(k + u, k1 - 1);
            av[u] = *reinterpret_cast<const bf16x4*>(at + kk * 256);
            bv[u] = *reinterpret_cast<const bf16x4*>(bt + kk * 256);
        }
#pragma unroll
        for (int u = 0; u < kGradLoads; ++u)
            if (k + u < k1) {
                acc = mfma16(av[u], bv[u], acc);
                if (bias) accb = mfma16(av[u], ones, accb);
            }
    }
    // lane holds rows 4g + e of column l%16; the bias product has equal columns
    s_acc[w][l] = acc;
    if (bias && (l & 15) == 0)
#pragma unroll
        for (int e = 0; e < 4; ++e) s_bias[w][4 * g + e] = accb[e];
    __syncthreads();
    const int e = threadIdx.x;
    if (e < 256) {
        const int i = e >> 4, j = e & 15;
        float sum = s_acc[0][j + 16 * (i >> 2)][i & 3];
#pragma unroll
        for (int k = 1; k < kGradWaves; ++k) sum += s_acc[k][j + 16 * (i >> 2)][i & 3];
        grad[off + (ib * 16 + i) * ncols + jb * 16 + j] = sum;
    } else if (bias && e < 256 + 16) {
        float sum = s_bias[0][e - 256];
        for (int k = 1; k < kGradWaves; ++k) sum += s_bias[k][e - 256];
        grad[off_b + ib * 16 + e - 256] = sum;
    } else if (w == kGradWaves - 1 && blockIdx.x == (unsigned)splits && loss_out) {
        // whole wave: strided partial sums, fixed butterfly
        float sum = 0.0f;
        for (int k = l; k < nb; k += 64) sum += buf.loss_part[k];
        for (int m = 32; m > 0; m >>= 1) sum += __shfl_xor(sum, m, 64);
        if (l == 0) *loss_out = sum / (float)(batch * kTargets);
    }
}

// Workgroups per gradient tile: one each while another kernel that adds their
// partials costs more (8,192 samples: 10.4 us, with eight 8.3 and 4.0 for the
// sum), eight above (16,384: 20.5 us against 8.9 + 4.0, 32,768: 39.8 against
// 14.9 + 4.0).
constexpr int kGradSplits = 8;
inline int grad_splits(int batch) { return batch >= 12288 ? kGradSplits : 1; }

// Sum of the split-K partial gradients, in slice order.
__device__ __forceinline__ float grad_sum(const float* __restrict__ part, int splits, int e) {
    float gr = part[e];
    for (int sp = 1; sp < splits; ++sp) gr += part[(int64_t)sp * kNumParams + e];
    return gr;
}

static __global__ void k_grad_reduce(const float* __restrict__ part, int splits, float* __restrict__ grad) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < kNumParams) grad[e] = grad_sum(part, splits, e);
}

// Adam (Kingma and Ba, 2015) on the fp32 masters, then their bf16 copies;
// the gradient is the sum of `splits` partials [splits][kNumParams].
static __global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ grad, int splits, uint16_t* __restrict__ wb, float lr, float b1,
                       float b2, float eps, float corr1, float corr2) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= kNumParams) return;
    const float gr = grad_sum(grad, splits, e);
    const float mm = b1 * m[e] + (1.0f - b1) * gr;
    const float vv = b2 * v[e] + (1.0f - b2) * gr * gr;
    m[e] = mm;
    v[e] = vv;
    const float upd = lr * (mm / corr1) / (sqrtf(vv / corr2) + eps);
    const float nw = w[e] - upd;
    w[e] = nw;
    wb[e] = to_bf16(nw);
}

// Plain forward over a batch (x: [B][16] normalised) -> y [B][16].
static __global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ params,
                                                     const uint16_t* __restrict__ wb,
                                                     const float* __restrict__ x, int batch,
                                                     float* __restrict__ y) {
    __shared__ __align__(16) uint16_t s_w[kMlpLdsElems];
    const MlpSmem s = mlp_smem(s_w);
    load_weights_lds(wb, s);
    __syncthreads();
    const int l = threadIdx.x & 63;
    const int g = l >> 4;
    const int wave_g = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (wave_g * 16 >= batch) return;
    const int p = wave_g * 16 + (l & 15);
    const f32x4 xv = *reinterpret_cast<const f32x4*>(x + (int64_t)p * 16 + 4 * g);
    const f32x4 out = mlp_forward(s, params, pack_bf16(xv));
    *reinterpret_cast<f32x4*>(y + (int64_t)p * 16 + 4 * g) = out;
}

}  // namespace infoli
