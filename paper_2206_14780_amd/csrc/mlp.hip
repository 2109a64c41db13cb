// Per-particle MLP that gives the solver its initial guess: forward,
// backward and Adam on gfx950's BF16 matrix cores (v_mfma_f32_16x16x32_bf16)
// with FP32 accumulation.  Not part of the paper, which names better initial
// guesses as future work (Sections "Conclusions and future work" and
// "Implementation notes").
//
// Network (one sample = one fluid particle and one velocity component):
//   x[4] -> 64 -> 64 -> 64 -> o[3], ReLU on the hidden layers,
//   pred = o0 B0 + o1 B1 + o2 B2 with basis B = (b_c, u_c, (u - A u)_c) / U.
// All products run on MFMA, 16 samples per tile.  Weights enter every product
// as BF16; the inputs of the 64x64 products (activations and gradient signals)
// are rounded to BF16 as well, those of the 4->64 and 64->3 layers and of the
// gradient signal of the last hidden layer enter as sums of BF16 parts.
//
// MFMA fragment layout (lane l, g = l / 16, c = l % 16, r = 0..3): the
// output D[4g + r][c]; the operands of one 16x16x32 step carry 8 values of K
// per lane, A[c][k] and B[k][c] for the lane group's 8 slots.  The kernels
// assign slot i of group g to K index 16 (i / 4) + 4 g + i % 4 of the step:
// two 16-wide halves, each in the layout of a D output (rows 4g + r), so a
// product's output (or two tiles' worth of samples) becomes the next
// product's operand by concatenating two 4-value fragments, with no
// shuffle.  A and B use the same assignment, so the product is exact in it,
// and a fragment serves as either: with the operands swapped a product comes
// out transposed.
#include <algorithm>
#include <cmath>

#include "mlp.hpp"
#include "operator_kernels.hpp"

namespace sph {
namespace mlp {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16s8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The operand of one 16x16x32 step from two 4-value fragments (K slots
// 0..3 and 4..7 of the lane group).
__device__ inline bf16x8 cat8(bf16x4 lo, bf16x4 hi) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ inline f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr int kWaves = 4;             // waves per block
constexpr int kThreads = kWaves * kWave;

// What a wave writes to LDS in the tile loops is its own (wave_sync), so the
// waves of a block never wait for each other after the parameters are loaded.

__device__ inline uint16_t f2bf(float f) {  // nearest, ties to even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Two floats to packed BF16, nearest-even (the hardware conversion of
// gfx950; the same rounding as f2bf on finite values).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 hbf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pk_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, hbf16x2));
}
__device__ inline bf16x4 bf16x4_of(float v0, float v1, float v2, float v3) {
    return __builtin_bit_cast(bf16x4, u32x2{pk_bf16(v0, v1), pk_bf16(v2, v3)});
}
// The four values' BF16 parts: hi = nearest BF16, lo = BF16 of v - hi (the
// remainder v - hi is exact in FP32); rem receives v - hi - lo, exact too.
__device__ inline void bf16x4_split(const float (&v)[4], bf16x4& hi, bf16x4& lo, float (&rem)[4]) {
    hi = bf16x4_of(v[0], v[1], v[2], v[3]);
    for (int r = 0; r < 4; ++r) rem[r] = v[r] - bf2f((uint16_t)hi[r]);
    lo = bf16x4_of(rem[0], rem[1], rem[2], rem[3]);
    for (int r = 0; r < 4; ++r) rem[r] -= bf2f((uint16_t)lo[r]);
}
// Four values as the operand of one step, exactly: part g (g = 0, 1, 2) of
// value r in K slot 4g + r, to meet the same weight in all three.
__device__ inline bf16x8 parts_operand(const float (&v)[4], int g) {
    const bf16x4 z4 = {0, 0, 0, 0};
    bf16x4 hi, lo;
    float rem[4];
    bf16x4_split(v, hi, lo, rem);
    const bf16x4 last = bf16x4_of(rem[0], rem[1], rem[2], rem[3]);  // exact: at most 8 bits remain
    return cat8(g == 0 ? hi : (g == 1 ? lo : (g == 2 ? last : z4)), z4);
}

// A weight operand of one step: w(k) for the lane group's K indices, value i at
// k = 16 (i / 4) + 4g + i % 4.
template <typename F>
__device__ inline bf16x8 weight_frag(F&& w, int g) {
    return cat8(bf16x4_of(w(4 * g), w(4 * g + 1), w(4 * g + 2), w(4 * g + 3)),
                bf16x4_of(w(16 + 4 * g), w(17 + 4 * g), w(18 + 4 * g), w(19 + 4 * g)));
}

// Inference: out[s] = (o0, o1, o2, pred) for samples [0, n).  All four
// products run on MFMA, transposed, Z^T = W^T H^T, with the 16 samples of a
// tile on the MFMA N dimension: a product's output then sits in registers
// exactly as the next product's B operand (lane (g, c) holds features
// 16t + 4g + r of sample c), so no LDS transpose is needed; the weights of
// the 64x64 layers, as A operands, stay in registers for the whole launch,
// those of the first and last layers in LDS.  The 64x64 layers take BF16
// weights and BF16 layer inputs, as in the training kernel.  The first and
// last layers take their inputs as sums of BF16 parts against the same BF16
// weight: the features as three parts, which hold an FP32 value exactly (K
// slots 4g + r, g = 0, 1, 2, carry part g of feature r; the layer's output is
// rounded to BF16 next, where a less accurate input would flip roundings); the
// last hidden layer as two parts, to 2^-16 relative (one K step per part; the
// output is not rounded again).  The training kernel takes three there too.
struct alignas(16) InferSmem {
    alignas(16) float b1[kH];
    alignas(16) float b2[kH];
    alignas(16) float b3[kH];
    alignas(16) float b4[4];
    alignas(16) bf16x8 a1[4][kWave];  // A operands of layer 1 (tile t, lane)
    alignas(16) bf16x8 a4[2][kWave];  // A operands of layer 4 (K step s, lane)
    alignas(16) bf16x8 f2[8][kWave], f3[8][kWave];  // the 64x64 layers', [2 t + s]
};

// Bounded by the vector ALU (bias, ReLU, rounding: 200 instructions a tile, 20
// us of a launch of 985k samples), once the loads are out of its way: 68 -> 35
// us for that launch with the samples loaded ahead, the weights gathered once
// per block and no more waves than fit.  At most 128 registers, so that four
// waves share a SIMD.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_mlp_infer(const float* __restrict__ S, int64_t n,
                                                        const float* __restrict__ p, float* __restrict__ out) {
    __shared__ __align__(16) InferSmem sm;
    for (int i = threadIdx.x; i < kH; i += blockDim.x) {
        sm.b1[i] = p[kOB1 + i];
        sm.b2[i] = p[kOB2 + i];
        sm.b3[i] = p[kOB3 + i];
    }
    if (threadIdx.x < 4) sm.b4[threadIdx.x] = threadIdx.x < kOut ? p[kOB4 + threadIdx.x] : 0.f;
    // A operands: step s of output tile t holds W[in][16t + c] (W stored
    // [in][out]) for the lane group's K slots, in = 32s + 16 (i / 4) + 4g + i % 4.
    // The waves share their gathers: each by itself, as before, read all 128
    // values of a lane one by one, 19 us of a launch of 985k samples.
    const int lane = threadIdx.x % kWave, g = lane / 16, c = lane % 16;
    for (int q = threadIdx.x / kWave; q < 8; q += kWaves) {
        sm.f2[q][lane] = weight_frag([&](int k) { return p[kOW2 + (32 * (q % 2) + k) * kH + 16 * (q / 2) + c]; }, g);
        sm.f3[q][lane] = weight_frag([&](int k) { return p[kOW3 + (32 * (q % 2) + k) * kH + 16 * (q / 2) + c]; }, g);
    }
    // layer 1: K slot 4g + r (g = 0, 1, 2: the three parts) is feature r;
    // the other slots are zero.  Layer 4: output row c (< 3) of
    // W4^T, K = the 64 hidden units.  Both kept in LDS (one copy per lane
    // index, shared by the block's waves), read once per tile.
    const bf16x4 z4 = {0, 0, 0, 0};
    if (threadIdx.x < kWave) {
        for (int t = 0; t < 4; ++t) {
            bf16x4 w = z4;
            if (g < 3)
                for (int r = 0; r < 4; ++r) w[r] = (short)f2bf(p[kOW1 + r * kH + 16 * t + c]);
            sm.a1[t][lane] = cat8(w, z4);
        }
        for (int s = 0; s < 2; ++s)
            sm.a4[s][lane] = weight_frag([&](int k) { return c < kOut ? p[kOW4 + (32 * s + k) * kOut + c] : 0.f; }, g);
    }
    __syncthreads();
    bf16x8 a2[4][2], a3[4][2];
    for (int t = 0; t < 4; ++t)
        for (int s = 0; s < 2; ++s) {
            a2[t][s] = sm.f2[2 * t + s][lane];
            a3[t][s] = sm.f3[2 * t + s][lane];
        }
    // the next tile's features are loaded a tile ahead and the basis at the
    // tile's start: waiting for them in turn took half of the time
    const int64_t ntiles = ceil_div(n, (int64_t)16);
    const int64_t nw = (int64_t)gridDim.x * kWaves;
    const auto features = [&](int64_t tile) {
        const int64_t smp = tile * 16 + c;
        return smp < n ? *reinterpret_cast<const float4*>(S + smp * kSample) : float4{0.f, 0.f, 0.f, 0.f};
    };
    int64_t tile = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave;
    float4 x = features(tile);
    for (; tile < ntiles; tile += nw) {
        // re-read the small LDS tables every tile rather than keeping them
        // in registers (which would leave room for fewer waves per SIMD)
        __asm__ volatile("" ::: "memory");
        const int64_t smp = tile * 16 + c;
        const bool last = g == 0 && smp < n;  // the lanes that write
        float4 bs;
        if (last) bs = *reinterpret_cast<const float4*>(S + smp * kSample + 4);
        const bf16x8 b1 = parts_operand({x.x, x.y, x.z, x.w}, g);
        x = features(tile + nw);
        bf16x4 h[4];
        for (int t = 0; t < 4; ++t) {
            const f32x4 z = mfma32(sm.a1[t][lane], b1, f32x4{0.f, 0.f, 0.f, 0.f});
            const float4 b = *reinterpret_cast<const float4*>(&sm.b1[16 * t + 4 * g]);
            h[t] = bf16x4_of(fmaxf(z[0] + b.x, 0.f), fmaxf(z[1] + b.y, 0.f), fmaxf(z[2] + b.z, 0.f),
                             fmaxf(z[3] + b.w, 0.f));
        }
        // layer 2 on MFMA, bias, ReLU, BF16: the B operand of layer 3
        f32x4 acc[4];
        for (int t = 0; t < 4; ++t) {
            acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int s = 0; s < 2; ++s) acc[t] = mfma32(a2[t][s], cat8(h[2 * s], h[2 * s + 1]), acc[t]);
        }
        for (int t = 0; t < 4; ++t) {
            const float4 b = *reinterpret_cast<const float4*>(&sm.b2[16 * t + 4 * g]);
            const float bb[4] = {b.x, b.y, b.z, b.w};
            h[t] = bf16x4_of(fmaxf(acc[t][0] + bb[0], 0.f), fmaxf(acc[t][1] + bb[1], 0.f),
                             fmaxf(acc[t][2] + bb[2], 0.f), fmaxf(acc[t][3] + bb[3], 0.f));
        }
        // layer 3 on MFMA, bias, ReLU, split into BF16 parts: the B operands
        // of layer 4
        for (int t = 0; t < 4; ++t) {
            acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int s = 0; s < 2; ++s) acc[t] = mfma32(a3[t][s], cat8(h[2 * s], h[2 * s + 1]), acc[t]);
        }
        bf16x4 hh[4], hl[4];
        for (int t = 0; t < 4; ++t) {
            const float4 b = *reinterpret_cast<const float4*>(&sm.b3[16 * t + 4 * g]);
            const float v[4] = {fmaxf(acc[t][0] + b.x, 0.f), fmaxf(acc[t][1] + b.y, 0.f),
                                fmaxf(acc[t][2] + b.z, 0.f), fmaxf(acc[t][3] + b.w, 0.f)};
            float rem[4];
            bf16x4_split(v, hh[t], hl[t], rem);
        }
        // layer 4 on MFMA: rows 0-2 of the output tile (lanes of group 0)
        f32x4 o4 = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < 2; ++s) {
            const bf16x8 w4 = sm.a4[s][lane];
            o4 = mfma32(w4, cat8(hh[2 * s], hh[2 * s + 1]), o4);
            o4 = mfma32(w4, cat8(hl[2 * s], hl[2 * s + 1]), o4);
        }
        if (last) {
            const float o0 = o4[0] + sm.b4[0], o1 = o4[1] + sm.b4[1], o2 = o4[2] + sm.b4[2];
            float pred = o0 * bs.x;
            pred = __builtin_fmaf(o1, bs.y, pred);
            pred = __builtin_fmaf(o2, bs.z, pred);
            *reinterpret_cast<float4*>(out + smp * 4) = float4{o0, o1, o2, pred};
        }
    }
}

// Forward and backward of a batch (sample ids idx[0, batch)); every block
// writes its partial gradient (kNParam values) and its partial sum of squared
// errors, in FP64, to part[block][0 .. kNParam].
//
// Each product is taken twice with the operands swapped: transposed ("T": lane
// (g, c) holds features 16t + 4g + r of sample c), which is the next product's
// operand, and plain ("N": feature 16t + c of samples 4g + r), which is the
// operand of the weight gradients h^T dz, whose K is the samples.  Matrix
// instructions are cheaper here than the transposes through LDS that one of
// the two forms would need: they are idle nine tenths of the time.  Two tiles
// go together, for the 32 samples of a weight gradient's K step and because
// one wave per SIMD (the gradients of both 64x64 layers take 128 registers)
// has only its own instructions to overlap; the weights' fragments come from
// LDS in lane order, one 16-byte read for four products.  Layers 1 and 4 and
// the last layer's data gradient take their FP32 inputs as three BF16 parts,
// that is exactly; bias gradients and those of layers 1 and 4 are FP32 on the
// vector ALU.  The four waves' gradients are added in FP64 in the block.
// A step of 65,536 samples with the sum of its 256 partials (1024, one per wave,
// before): 82 -> 42 us; 38 with a block's sums rounded to FP32, whose gradient
// is further off.
// What bounds it is the vector ALU of a single wave (bias, ReLU, rounding and
// the small gradients: about 700 instructions a tile) and, at this size, the
// setup and the exchange at the end, about a third.
// Sums over the samples are FP32 within four tiles of a wave (the accumulators
// of the matrix cores) and FP64 from there on: the block adds its waves'
// values after every four tiles, so that a larger batch does not make the FP32
// chains longer, and hands the sum on unrounded.
struct alignas(16) TrainSmem {
    bf16x8 f2[8][kWave], f3[8][kWave];  // W[in][16t + c], K = in; [2 t + s]: tile t, K step s
    bf16x8 r2[8][kWave], r3[8][kWave];  // W[16t + c][out], K = out
    bf16x8 a1[4][kWave];                // layer 1: W[r][16t + c] in K slots 4g + r, g < 3
    bf16x8 a4[2][kWave];                // layer 4: W[in][c % 4], K = in (every lane group gets the outputs)
    bf16x8 r4[4][kWave];                // its data gradient: W[16t + c][r] in K slots 4g + r, g < 3
    float b1[kH], b2[kH], b3[kH], b4[4];
    float4 smp[kWaves][4][16][2];       // a wave's four tiles of samples
    float4 go[kWaves][2][16];           // output gradients of two tiles
};
constexpr int kExchange = 64;  // values per lane that the waves exchange at a time
struct TrainLds {
    TrainSmem p;
    float x[kWaves][kExchange][kWave];
};

__device__ inline void train_params(TrainSmem& sm, const float* __restrict__ p) {
    const bf16x4 z4 = {0, 0, 0, 0};
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, g = lane / 16, c = lane % 16;
    const auto frag = [&](auto w) { return weight_frag(w, g); };
#pragma unroll
    for (int q = wave; q < 8; q += kWaves) {
        const int o = 16 * (q / 2) + c, k0 = 32 * (q % 2);
        sm.f2[q][lane] = frag([&](int k) { return p[kOW2 + (k0 + k) * kH + o]; });
        sm.f3[q][lane] = frag([&](int k) { return p[kOW3 + (k0 + k) * kH + o]; });
        sm.r2[q][lane] = frag([&](int k) { return p[kOW2 + o * kH + k0 + k]; });
        sm.r3[q][lane] = frag([&](int k) { return p[kOW3 + o * kH + k0 + k]; });
    }
    {
        const int o = 16 * wave + c;
        const auto w1 = [&](int r) { return p[kOW1 + r * kH + o]; };
        const auto w4 = [&](int r) { return p[kOW4 + o * kOut + r]; };
        sm.a1[wave][lane] = cat8(g < 3 ? bf16x4_of(w1(0), w1(1), w1(2), w1(3)) : z4, z4);
        sm.r4[wave][lane] = cat8(g < 3 ? bf16x4_of(w4(0), w4(1), w4(2), 0.f) : z4, z4);
    }
    if (wave < 2) sm.a4[wave][lane] = frag([&](int k) { return c % 4 < kOut ? p[kOW4 + (32 * wave + k) * kOut + c % 4] : 0.f; });
    if (threadIdx.x < kH) {
        sm.b1[threadIdx.x] = p[kOB1 + threadIdx.x];
        sm.b2[threadIdx.x] = p[kOB2 + threadIdx.x];
        sm.b3[threadIdx.x] = p[kOB3 + threadIdx.x];
    }
    if (threadIdx.x < 4) sm.b4[threadIdx.x] = threadIdx.x < kOut ? p[kOB4 + threadIdx.x] : 0.f;
}

__device__ inline bf16x4 relu_bf16(f32x4 z) {
    return bf16x4_of(fmaxf(z[0], 0.f), fmaxf(z[1], 0.f), fmaxf(z[2], 0.f), fmaxf(z[3], 0.f));
}
// The gradient signal where the layer's output (BF16, never negative) is not 0.
__device__ inline f32x4 where_on(f32x4 d, bf16x4 h) {
    return f32x4{h[0] ? d[0] : 0.f, h[1] ? d[1] : 0.f, h[2] ? d[2] : 0.f, h[3] ? d[3] : 0.f};
}
__device__ inline bf16x4 to_bf16(f32x4 d) { return bf16x4_of(d[0], d[1], d[2], d[3]); }

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_mlp_train(
    const float* __restrict__ S, const int32_t* __restrict__ idx, int64_t batch, const float* __restrict__ params,
    double* __restrict__ part, int32_t tiles_per_wave) {
    __shared__ __align__(16) TrainLds lds;
    TrainSmem& sm = lds.p;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave, g = lane / 16, c = lane % 16;
    const int64_t tile0 = ((int64_t)blockIdx.x * kWaves + wave) * tiles_per_wave;
    const int64_t left = ceil_div(batch, (int64_t)16) - tile0;
    const int32_t mine = (int32_t)(left < 0 ? 0 : min(left, (int64_t)tiles_per_wave));
    // samples of four tiles at a time, lane (g, c) sample c of tile g; zeros
    // beyond the batch give no gradient
    float4 sx, sb;
    const auto load = [&](int32_t q) {
        const int64_t k = (tile0 + q + g) * 16 + c;
        sx = sb = float4{0.f, 0.f, 0.f, 0.f};
        if (q + g < mine && k < batch) {
            // (the caller's samples need not be aligned to 16 bytes)
            typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
            const f32x4u* v = reinterpret_cast<const f32x4u*>(S + (int64_t)idx[k] * kSample);
            sx = float4{v[0][0], v[0][1], v[0][2], v[0][3]};
            sb = float4{v[1][0], v[1][1], v[1][2], v[1][3]};
        }
    };
    load(0);
    train_params(sm, params);
    __syncthreads();
    const float inv_m = 2.0f / (float)batch;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    double* P = part + (int64_t)blockIdx.x * (kNParam + 1);
    // a layer's bias as the accumulator to start from, in both forms
    const auto biasT = [&](const float* b, int t) { return *reinterpret_cast<const f32x4*>(b + 16 * t + 4 * g); };
    const auto biasN = [&](const float* b, int t) {
        const float v = b[16 * t + c];
        return f32x4{v, v, v, v};
    };
    for (int32_t q = 0; q < tiles_per_wave; q += 4) {
        f32x4 gW2[4][4], gW3[4][4];
        for (int i = 0; i < 4; ++i)
            for (int j = 0; j < 4; ++j) gW2[i][j] = gW3[i][j] = z;
        float gW1[4][4] = {}, gW4[4][3] = {}, gb1[4] = {}, gb2[4] = {}, gb3[4] = {}, gb4[3] = {}, sse = 0.f;
        sm.smp[wave][g][c][0] = sx;
        sm.smp[wave][g][c][1] = sb;
        wave_sync();
        load(q + 4);
        for (int32_t pr = 0; pr < 2 && q + 2 * pr < mine; ++pr) {
            // re-read the tables for every pair rather than keeping them in registers
            __asm__ volatile("" ::: "memory");
            bf16x4 h1o[2][4], h1n[2][4], h2o[2][4], h2n[2][4], h3o[2][4];
            bf16x8 in[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 x = sm.smp[wave][2 * pr + u][c][0];
                in[u] = parts_operand({x.x, x.y, x.z, x.w}, g);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 w = sm.a1[t][lane];
                const f32x4 bT = biasT(sm.b1, t), bN = biasN(sm.b1, t);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    h1o[u][t] = relu_bf16(mfma32(w, in[u], bT));
                    h1n[u][t] = relu_bf16(mfma32(in[u], w, bN));
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 w0 = sm.f2[2 * t][lane], w1 = sm.f2[2 * t + 1][lane];
                const f32x4 bT = biasT(sm.b2, t), bN = biasN(sm.b2, t);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bf16x8 v0 = cat8(h1o[u][0], h1o[u][1]), v1 = cat8(h1o[u][2], h1o[u][3]);
                    h2o[u][t] = relu_bf16(mfma32(w1, v1, mfma32(w0, v0, bT)));
                    h2n[u][t] = relu_bf16(mfma32(v1, w1, mfma32(v0, w0, bN)));
                }
            }
            // layer 3, whose output layer 4 takes as three BF16 parts
            f32x4 h3n[2][4], o4[2];
            bf16x4 h3m[2][4], h3l[2][4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 w0 = sm.f3[2 * t][lane], w1 = sm.f3[2 * t + 1][lane];
                const f32x4 bT = biasT(sm.b3, t), bN = biasN(sm.b3, t);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bf16x8 v0 = cat8(h2o[u][0], h2o[u][1]), v1 = cat8(h2o[u][2], h2o[u][3]);
                    const f32x4 zT = mfma32(w1, v1, mfma32(w0, v0, bT));
                    const float v[4] = {fmaxf(zT[0], 0.f), fmaxf(zT[1], 0.f), fmaxf(zT[2], 0.f), fmaxf(zT[3], 0.f)};
                    float rem[4];
                    bf16x4_split(v, h3o[u][t], h3m[u][t], rem);
                    h3l[u][t] = bf16x4_of(rem[0], rem[1], rem[2], rem[3]);
                    h3n[u][t] = mfma32(v1, w1, mfma32(v0, w0, bN));
#pragma unroll
                    for (int r = 0; r < 4; ++r) h3n[u][t][r] = fmaxf(h3n[u][t][r], 0.f);
                }
            }
            o4[0] = o4[1] = *reinterpret_cast<const f32x4*>(sm.b4);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 w = sm.a4[s][lane];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    o4[u] = mfma32(w, cat8(h3l[u][2 * s], h3l[u][2 * s + 1]), o4[u]);
                    o4[u] = mfma32(w, cat8(h3m[u][2 * s], h3m[u][2 * s + 1]), o4[u]);
                    o4[u] = mfma32(w, cat8(h3o[u][2 * s], h3o[u][2 * s + 1]), o4[u]);
                }
            }
            // output gradient g_o = (2/m) (pred - t) B of sample c
            bf16x8 gin[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 bs = sm.smp[wave][2 * pr + u][c][1];
                float pred = o4[u][0] * bs.x;
                pred = __builtin_fmaf(o4[u][1], bs.y, pred);
                pred = __builtin_fmaf(o4[u][2], bs.z, pred);
                const float err = pred - bs.w;
                const float go[4] = {inv_m * err * bs.x, inv_m * err * bs.y, inv_m * err * bs.z, 0.f};
                if (g == 0) {
                    sse = __builtin_fmaf(err, err, sse);
                    for (int k = 0; k < 3; ++k) gb4[k] += go[k];
                    sm.go[wave][u][c] = float4{go[0], go[1], go[2], 0.f};
                }
                gin[u] = parts_operand(go, g);
            }
            wave_sync();
            // layer 4: weight gradient h3^T g_o, and the signal of layer 3
            bf16x4 dzo[2][4], dzn[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float4 o = sm.go[wave][u][4 * g + r];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        gW4[t][0] = __builtin_fmaf(h3n[u][t][r], o.x, gW4[t][0]);
                        gW4[t][1] = __builtin_fmaf(h3n[u][t][r], o.y, gW4[t][1]);
                        gW4[t][2] = __builtin_fmaf(h3n[u][t][r], o.z, gW4[t][2]);
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 w = sm.r4[t][lane];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    dzo[u][t] = to_bf16(where_on(mfma32(w, gin[u], z), h3o[u][t]));
                    f32x4 d = mfma32(gin[u], w, z);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        d[r] = h3n[u][t][r] > 0.f ? d[r] : 0.f;
                        gb3[t] += d[r];
                    }
                    dzn[u][t] = to_bf16(d);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    gW3[mt][nt] = mfma32(cat8(h2n[0][mt], h2n[1][mt]), cat8(dzn[0][nt], dzn[1][nt]), gW3[mt][nt]);
            // layer 2: signal dz3 W3^T where h2 > 0
            bf16x4 ezo[2][4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x8 w0 = sm.r3[2 * t][lane], w1 = sm.r3[2 * t + 1][lane];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bf16x8 v0 = cat8(dzo[u][0], dzo[u][1]), v1 = cat8(dzo[u][2], dzo[u][3]);
                    ezo[u][t] = to_bf16(where_on(mfma32(w1, v1, mfma32(w0, v0, z)), h2o[u][t]));
                    const f32x4 d = where_on(mfma32(v1, w1, mfma32(v0, w0, z)), h2n[u][t]);
                    gb2[t] += (d[0] + d[1]) + (d[2] + d[3]);
                    dzn[u][t] = to_bf16(d);
                }
            }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    gW2[mt][nt] = mfma32(cat8(h1n[0][mt], h1n[1][mt]), cat8(dzn[0][nt], dzn[1][nt]), gW2[mt][nt]);
            // layer 1
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const bf16x8 v0 = cat8(ezo[u][0], ezo[u][1]), v1 = cat8(ezo[u][2], ezo[u][3]);
                f32x4 d[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    d[t] = where_on(mfma32(v1, sm.r2[2 * t + 1][lane], mfma32(v0, sm.r2[2 * t][lane], z)), h1n[u][t]);
                    gb1[t] += (d[t][0] + d[t][1]) + (d[t][2] + d[t][3]);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float4 x = sm.smp[wave][2 * pr + u][4 * g + r][0];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        gW1[0][t] = __builtin_fmaf(x.x, d[t][r], gW1[0][t]);
                        gW1[1][t] = __builtin_fmaf(x.y, d[t][r], gW1[1][t]);
                        gW1[2][t] = __builtin_fmaf(x.z, d[t][r], gW1[2][t]);
                        gW1[3][t] = __builtin_fmaf(x.w, d[t][r], gW1[3][t]);
                    }
                }
            }
            wave_sync();
        }
        // The block's sums of these four tiles: the waves' values side by side
        // in LDS, 64 per lane at a time, added by all threads (P[at] by the
        // same one every time).
        const auto put = [&](int at, double s) { P[at] = q == 0 ? s : P[at] + s; };
        const auto exchange = [&](const f32x4 (&gW)[4][4], int off) {
            __syncthreads();
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) lds.x[wave][(4 * mt + nt) * 4 + r][lane] = gW[mt][nt][r];
            __syncthreads();
            for (int v = wave; v < kExchange; v += kWaves) {
                double s = 0.0;
                for (int w = 0; w < kWaves; ++w) s += (double)lds.x[w][v][lane];
                put(off + (16 * (v / 16) + 4 * g + v % 4) * kH + 16 * (v / 4 % 4) + c, s);
            }
        };
        exchange(gW2, kOW2);
        exchange(gW3, kOW3);
        __syncthreads();
        constexpr int kSmall = 10;  // per tile t: four rows of W1, three biases, three columns of W4
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            for (int f = 0; f < 4; ++f) lds.x[wave][kSmall * t + f][lane] = gW1[f][t];
            lds.x[wave][kSmall * t + 4][lane] = gb1[t];
            lds.x[wave][kSmall * t + 5][lane] = gb2[t];
            lds.x[wave][kSmall * t + 6][lane] = gb3[t];
            for (int k = 0; k < 3; ++k) lds.x[wave][kSmall * t + 7 + k][lane] = gW4[t][k];
        }
        for (int k = 0; k < 3; ++k) lds.x[wave][4 * kSmall + k][lane] = gb4[k];
        lds.x[wave][4 * kSmall + 3][lane] = sse;
        __syncthreads();
        // features 16t + c: over the waves and their lane groups
        for (int e = threadIdx.x; e < 4 * kSmall * 16; e += kThreads) {
            const int v = e / 16, t = v / kSmall, k = v % kSmall, o = 16 * t + e % 16;
            double s = 0.0;
            for (int w = 0; w < kWaves; ++w)
                for (int l = e % 16; l < kWave; l += 16) s += (double)lds.x[w][v][l];
            const int at = k < 4 ? kOW1 + k * kH + o : k == 4 ? kOB1 + o : k == 5 ? kOB2 + o : k == 6 ? kOB3 + o
                                                                                              : kOW4 + o * kOut + k - 7;
            put(at, s);
        }
        // output biases and squared error: a wave each, over the waves' lanes of group 0
        double s = 0.0;
        if (lane < 16)
            for (int w = 0; w < kWaves; ++w) s += (double)lds.x[w][4 * kSmall + wave][lane];
        for (int off = 1; off < 16; off <<= 1) s += __shfl_xor(s, off, kWave);
        if (lane == 0) put(wave < 3 ? kOB4 + wave : kNParam, s);
    }
}
static_assert(kWaves == 4, "the four values beside the tiles: a wave each");

// Sums the blocks' partials in a fixed order.  With Adam (step > 0) it
// updates the FP32 master weights (Kingma & Ba, bias-corrected); otherwise it
// writes the gradient to `grad`.  out[0] = mean squared error of the batch.
// One lane per parameter, kRedWaves waves per block: wave
// w adds the partials w, w + kRedWaves, ... in that order, then the first
// wave adds the waves' sums in wave order, so the result depends only on
// the number of partials, not on timing.
constexpr int kRedWaves = 16;
__global__ __launch_bounds__(kRedWaves * kWave) void k_mlp_reduce(const double* __restrict__ part, int32_t nparts,
                                                                  int64_t batch, float* __restrict__ params,
                                                                  float* __restrict__ m, float* __restrict__ v,
                                                                  float* __restrict__ grad, int32_t step,
                                                                  double lr, double* __restrict__ out) {
    __shared__ double lds[kRedWaves][kWave];
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int p = blockIdx.x * kWave + lane;
    double sw = 0.0;
    if (p <= kNParam) {
#pragma unroll 8
        for (int q = w; q < nparts; q += kRedWaves) sw += part[(int64_t)q * (kNParam + 1) + p];
    }
    lds[w][lane] = sw;
    __syncthreads();
    if (w != 0 || p > kNParam) return;
    double s = 0.0;
    for (int k = 0; k < kRedWaves; ++k) s += lds[k][lane];
    if (p == kNParam) {
        out[0] = s / (double)batch;
        return;
    }
    if (step <= 0) {
        grad[p] = (float)s;
        return;
    }
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    const double mm = b1 * (double)m[p] + (1.0 - b1) * s;
    const double vv = b2 * (double)v[p] + (1.0 - b2) * s * s;
    const double mh = mm / (1.0 - pow(b1, (double)step));
    const double vh = vv / (1.0 - pow(b2, (double)step));
    params[p] = (float)((double)params[p] - lr * mh / (sqrt(vh) + eps));
    m[p] = (float)mm;
    v[p] = (float)vv;
}

}  // namespace mlp
}  // namespace sph

using namespace sph;
using namespace sph::mlp;

// Tiles per wave of the training kernel and its blocks: a block per CU (its
// registers leave room for one), and pairs of tiles.
static int32_t tiles_per_wave(int64_t n, int32_t* grid) {
    const int64_t tiles = ceil_div(n, (int64_t)16);
    const int64_t blocks = std::min<int64_t>(ceil_div(tiles, (int64_t)(2 * kWaves)), 256);
    *grid = (int32_t)blocks;
    const int64_t per = ceil_div(tiles, blocks * kWaves);
    return (int32_t)((per + 1) / 2 * 2);
}

sph_status sph::mlp::forward(sph_ctx* ctx, const float* samples, int64_t n, const float* params, float* out) {
    if (n == 0) return SPH_OK;
    // several tiles per wave, which loads its 32 weight fragments once, and
    // no more waves than the chip holds at a time (four per SIMD)
    const int64_t waves = std::min<int64_t>(ceil_div(ceil_div(n, (int64_t)16), 4), 4096);
    const int32_t grid = (int32_t)std::max<int64_t>(ceil_div(waves, (int64_t)kWaves), 1);
    hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(kThreads), 0, ctx->stream, samples, n, params, out);
    SPH_LAUNCHED("k_mlp_infer");
    return SPH_OK;
}

extern "C" sph_status sph_mlp_forward(sph_ctx* ctx, const float* samples, int64_t n, const float* params,
                                      float* out) {
    if (!ctx) return SPH_E_ARG;
    if (!samples || !params || !out || n < 0) return ctx->fail(SPH_E_ARG, "mlp_forward: bad argument");
    if (reinterpret_cast<uintptr_t>(samples) % 16 || reinterpret_cast<uintptr_t>(out) % 16)
        return ctx->fail(SPH_E_ARG, "mlp_forward: samples and out must be 16-byte aligned");
    return sph::mlp::forward(ctx, samples, n, params, out);
}

static sph_status train_or_grad(sph_ctx* ctx, const float* samples, const int32_t* idx, int64_t batch,
                                float* params, float* m, float* v, float* grad, int32_t step, double lr,
                                double* loss) {
    int32_t grid = 0;
    const int32_t tpw = tiles_per_wave(batch, &grid);
    const int64_t nparts = grid;
    double* part = nullptr;
    double* out = nullptr;
    SPH_TRY(ctx->ensure_t(kMlpPart, (size_t)nparts * (kNParam + 1), &part));
    SPH_TRY(ctx->ensure_t(kMlpOut, 1, &out));
    hipLaunchKernelGGL(k_mlp_train, dim3(grid), dim3(kThreads), 0, ctx->stream, samples, idx, batch, params, part,
                       tpw);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((unsigned)ceil_div(kNParam + 1, kWave)), dim3(kRedWaves * kWave), 0,
                       ctx->stream, part,
                       (int32_t)nparts, batch, params, m, v, grad, step, lr, out);
    SPH_LAUNCHED("k_mlp_train/k_mlp_reduce");
    if (loss) {
        SPH_HIP(hipMemcpyAsync(loss, out, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
        SPH_HIP(hipStreamSynchronize(ctx->stream));
    }
    return SPH_OK;
}

extern "C" sph_status sph_mlp_grad(sph_ctx* ctx, const float* samples, const int32_t* idx, int64_t batch,
                                   const float* params, float* grad, double* loss) {
    if (!ctx) return SPH_E_ARG;
    if (!samples || !idx || !params || !grad || batch < 1) return ctx->fail(SPH_E_ARG, "mlp_grad: bad argument");
    return train_or_grad(ctx, samples, idx, batch, const_cast<float*>(params), nullptr, nullptr, grad, 0, 0.0, loss);
}

extern "C" sph_status sph_mlp_train_step(sph_ctx* ctx, const float* samples, const int32_t* idx, int64_t batch,
                                         float* params, float* adam_m, float* adam_v, int32_t step, double lr,
                                         double* loss) {
    if (!ctx) return SPH_E_ARG;
    if (!samples || !idx || !params || !adam_m || !adam_v || batch < 1 || step < 1 || !(lr > 0.0))
        return ctx->fail(SPH_E_ARG, "mlp_train_step: bad argument");
    return train_or_grad(ctx, samples, idx, batch, params, adam_m, adam_v, nullptr, step, lr, loss);
}
