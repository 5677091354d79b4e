// Training of the MLP decoder (gfx950): Eq. 9 cross-entropy against code
// index labels (or the uncertainty-weighted loss of Eqs. 10-12), gradients by
// the chain rule, and the fused Adam update of Sec. 4 (Adam, betas (0.9,
// 0.999)) used for both the decoder and the per-Gaussian parameters.
//
// Every contraction runs on v_mfma_f32_32x32x16_bf16 with float32 accumulation:
//   k_mlp_train  per 32-pixel tile and wave: the inference forward (so training
//                sees exactly the activations inference produces), softmax, CE,
//                dz3 = (p - onehot) w_p, then the backward through the layers
//                (dh2 = W3^T dz3, dz2 = dh2 [h2 > 0], dh1 = W2^T dz2, dz1 =
//                dh1 [h1 > 0], and the input gradient W1^T dz1) with the
//                upstream gradient split into two bf16 parts (hi + lo, 16
//                significant bits) and the W^T fragments in LDS next to the
//                forward ones; straight through the bf16 roundings. The weight
//                gradients dW_l = sum_p dz_l h_(l-1)^T contract over the
//                pixels, which lie along the lanes: both operands are turned
//                by MFMAs against the identity (exact) and the products
//                accumulate in registers over all of a wave's tiles; the bias
//                sums accumulate in LDS in float32.
//   k_mlp_reduce the sum of the workgroups' partial results.
// One pass over the inputs, nothing per pixel in memory but the outputs.
// Writing the layer inputs and dz to memory for a second kernel that contracts
// them (1.3 KB a pixel each way, then float atomics) took 740 us for the
// semantic loss of 1080 x 720 pixels at K = 128 and 163 us for a decoder step
// of 65,536; this takes 240 and 45.
// Workspace: the partial results, 53 KB a workgroup at K = 128.
#include <algorithm>

#include "legs_internal.h"
#include "legs_decode_internal.h"

namespace {

typedef legs_f32x16 f32x16;
typedef legs_bf16x8 bf16x8;

constexpr int MH = LEGS_MLP_H;                     // 64 hidden units

// Per-pixel weighting of the cross-entropy. ru == NULL: the mean over the
// batch (Eq. 9). Otherwise the uncertainty-weighted loss of Eqs. 10-12:
// pixel p's CE is weighted by lce (1 - ru[p]) inv_hw, the loss gains
// lu ru[p] inv_hw, and d_ru[p] = (lu - lce CE_p) inv_hw.
struct CeWeights {
    const float *ru;
    float *d_ru;
    float lce, lu, inv_hw;
};

// Input gradient request: d_feat (NULL: none) receives dL/d(feature) at
// d_feat[c * dcs + p * dps]; with NORM the decoder input was f / |f| and its
// Jacobian (I - u u^T) / |f| (u = f / |f|) is applied, straight through the
// bf16 rounding of the input.
struct InputGrad {
    float *d_feat;
    int64_t dcs, dps;
};

// W^T fragments of the backward: (block, k-step, lane, e) = row 32 block +
// lane % 32 of W^T (a unit of the layer below), column legs_khid(k-step,
// lane / 32, e) (a unit of the layer above).
template <int KB>
struct MlpBwdLds {
    bf16x8 t3[2 * 2 * KB * 64];     // W3^T: 64 rows x K
    bf16x8 t2[2 * 4 * 64];          // W2^T: 64 x 64
    bf16x8 t1[4 * 64];              // W1^T: 8 rows (block padded to 32) x 64
};

template <int KB, int NT>
__device__ __forceinline__ void mlp_stage_bwd(const float *__restrict__ params, MlpBwdLds<KB> &T)
{
    const float *W1 = params + LEGS_MLP_OFF_W1, *W2 = params + LEGS_MLP_OFF_W2, *W3 = params + LEGS_MLP_OFF_W3;
    constexpr int S3 = 2 * KB;
    legs_stage_frags<2 * S3 * 64, NT, 4>(T.t3, [&](int i) {
        const int l = i & 63, ks = (i >> 6) % S3, mb = (i >> 6) / S3;
        bf16x8 f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = (__bf16)W3[legs_khid(ks, l >> 5, e) * MH + 32 * mb + (l & 31)];
        return f;
    });
    legs_stage_frags<2 * 4 * 64, NT, 2>(T.t2, [&](int i) {
        const int l = i & 63, ks = (i >> 6) & 3, mb = i >> 8;
        bf16x8 f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = (__bf16)W2[legs_khid(ks, l >> 5, e) * MH + 32 * mb + (l & 31)];
        return f;
    });
    legs_stage_frags<4 * 64, NT, 1>(T.t1, [&](int i) {
        const int l = i & 63, ks = i >> 6, row = l & 31;
        bf16x8 f;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            f[e] = row < LEGS_MLP_IN ? (__bf16)W1[legs_khid(ks, l >> 5, e) * LEGS_MLP_IN + row] : (__bf16)0.0f;
        return f;
    });
}

__device__ __forceinline__ void split8(const f32x16 &z, int first, bf16x8 &hi, bf16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 a = (__bf16)z[first + e];
        hi[e] = a;
        lo[e] = (__bf16)(z[first + e] - (float)a);
    }
}

using legs_turn::i32x4;

// Blocks turned for the weight gradients (legs_turn::turn). EXACT: byte by byte, any
// bit pattern. Otherwise by a bf16 identity, half of the MFMAs and a third of the
// VALU work, where an infinity or a NaN of a pixel spreads over its block's units:
// only for the last layer, whose gradient is NaN throughout at a pixel where it or
// its input is not finite. In the layers below a ReLU may stand between (a NaN
// feature beside closed units). (The semantic loss of 1080 x 720 pixels at K = 128
// takes 224 us with the bf16 identity in all layers, 240 so, 251 byte by byte in all.)
// bf: the bf16 identity's two k-steps; i8: the low bytes', the high ones' one up.
struct TurnId {
    const bf16x8 *bf;
    const i32x4 *i8;
};

__device__ __forceinline__ bf16x8 cvt8(const f32x16 &z, int first)
{
    bf16x8 f;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = (__bf16)z[first + e];
    return f;
}

__device__ __forceinline__ auto byte_identity(const TurnId &id)
{
    return [i8 = id.i8](int k) { return k < 2 ? i8[k * LEGS_WAVE] : i8[(k - 2) * LEGS_WAVE] << 8; };
}

template <bool EXACT>
__device__ __forceinline__ void turn_block(const bf16x8 &f0, const bf16x8 &f1, const TurnId &id, bf16x8 (&out)[2])
{
    if constexpr (EXACT) {
        legs_turn::turn(f0, f1, byte_identity(id), out);
    } else {
        const f32x16 t = legs_mfma(f1, id.bf[LEGS_WAVE], legs_mfma(f0, id.bf[0], (f32x16){}));
        out[0] = cvt8(t, 0);
        out[1] = cvt8(t, 8);
    }
}

// A turned block (lane = row, 2 x 8 pixels each half) as two operands of the
// 16 x 16 x 32 MFMA: rows 0 .. 15 and 16 .. 31, all 32 pixels.
__device__ __forceinline__ void halves(const bf16x8 (&f)[2], bf16x8 (&out)[2])
{
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    const u32x4 a = __builtin_bit_cast(u32x4, f[0]), b = __builtin_bit_cast(u32x4, f[1]);
    u32x4 x, y;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const auto r = __builtin_amdgcn_permlane16_swap(a[q], b[q], false, false);
        x[q] = r[0];
        y[q] = r[1];
    }
    out[0] = __builtin_bit_cast(bf16x8, x);
    out[1] = __builtin_bit_cast(bf16x8, y);
}

// Accumulators of the weight gradients, 32 x 32 blocks (row = unit of the
// layer, column = its input). Layer 1 has 8 inputs and the bias, four blocks of 16
// units x 16 columns in the registers of one: inputs 0 .. 3 in columns 0 .. 3, the
// bias in 4, inputs 4 .. 7 in 8 .. 11 (the order of the identity's rows). Units of
// two blocks never share a row: zeros do not mask a gradient that is not finite.
template <int KB>
struct MlpGrad {
    f32x16 w3[KB][2], w2[2][2], w1;
};

// dW block += dz (hi + lo parts) times the transposed layer input, over the
// tile's 32 pixels.
template <bool EXACT, int NB>
__device__ __forceinline__ void wgrad_block(const bf16x8 (&hi)[2], const bf16x8 (&lo)[2], const bf16x8 (&in)[NB][2],
                                            const TurnId &id, f32x16 *acc)
{
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        bf16x8 a[2];
        if (part) turn_block<EXACT>(lo[0], lo[1], id, a);
        else turn_block<EXACT>(hi[0], hi[1], id, a);
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[n] = legs_mfma(a[g], in[n][g], acc[n]);
    }
    __builtin_amdgcn_sched_barrier(0);   // one block's operands live at a time
}

// dW1 and db1 of the 32 units of block b: in holds the turned inputs and ones.
__device__ __forceinline__ void wgrad_input(const bf16x8 (&hi)[2], const bf16x8 (&lo)[2], const bf16x8 &in,
                                            const TurnId &id, int b, f32x16 &acc)
{
    typedef __attribute__((ext_vector_type(4))) float f32x4;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        bf16x8 t[2], a[2];
        if (part) turn_block<true>(lo[0], lo[1], id, t);
        else turn_block<true>(hi[0], hi[1], id, t);
        halves(t, a);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int o = 4 * (2 * b + k);
            f32x4 c = {acc[o], acc[o + 1], acc[o + 2], acc[o + 3]};
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k], in, c, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[o + r] = c[r];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Bias sums of a dz block: each lane adds its 16 values to its own words of LDS
// (read, add and write back: LDS float atomics took 600 cycles a wave here).
__device__ __forceinline__ void bias_add(float4 *bias, const f32x16 &z)
{
    float4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = bias[q * LEGS_WAVE];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        bias[q * LEGS_WAVE] = make_float4(v[q].x + z[4 * q], v[q].y + z[4 * q + 1], v[q].z + z[4 * q + 2],
                                          v[q].w + z[4 * q + 3]);
}

// A workgroup's partial result: the weight-gradient accumulators in register
// order, [16-value block][4 float4][lane], then the biases of layers 3 and 2,
// then the loss.
constexpr int mlp_acc_blocks(int KB) { return LEGS_MLP_PART_BLOCKS(KB); }
constexpr int mlp_part_floats(int KB) { return LEGS_MLP_PART_FLOATS(KB); }

template <int KB>
__device__ __forceinline__ f32x16 &mlp_acc(MlpGrad<KB> &G, int i)
{
    return i < 2 * KB ? G.w3[i / 2][i % 2] : i < 2 * KB + 4 ? G.w2[(i - 2 * KB) / 2][(i - 2 * KB) % 2] : G.w1;
}

// Parameter that word i of a partial result adds to (np: the loss, -1: none).
template <int KB>
__device__ __forceinline__ int mlp_part_param(int i)
{
    constexpr int NA = mlp_acc_blocks(KB) * 1024;
    if (i >= NA) {
        const int u = i - NA;
        return u < 32 * KB ? LEGS_MLP_OFF_B3(KB) + u
                           : u < 32 * (KB + 2) ? LEGS_MLP_OFF_B2 + u - 32 * KB : (int)LEGS_MLP_NPARAMS(KB);
    }
    const int blk = i >> 10, q = (i >> 8) & 3, lane = (i >> 2) & 63, col = lane & 31;
    const int row = legs_drow(4 * q + (i & 3), lane >> 5);
    if (blk < 2 * KB) return LEGS_MLP_OFF_W3 + (32 * (blk >> 1) + row) * MH + 32 * (blk & 1) + col;
    if (blk < 2 * KB + 4) {
        const int k = blk - 2 * KB;
        return LEGS_MLP_OFF_W2 + (32 * (k >> 1) + row) * MH + 32 * (k & 1) + col;
    }
    // 16 x 16 blocks: register r of lane l is row 4 (l / 16) + r, column l % 16
    const int unit = 16 * q + 4 * (lane >> 4) + (i & 3), c = lane & 15;
    if (c == 4) return LEGS_MLP_OFF_B1 + unit;
    return (c & 7) < 4 ? LEGS_MLP_OFF_W1 + unit * LEGS_MLP_IN + (c & 3) + 4 * (c >> 3) : -1;
}

// Forward, loss, backward and parameter gradient of 32-pixel tiles, one wave
// each (see the top of the file). Bound by the matrix unit and the VALU work
// between the layers, so nothing but the features, labels and input gradients
// touches memory: the weight gradients accumulate in registers over all of a
// wave's tiles (13 blocks of 32 x 32 at K = 128), which takes one wave per
// SIMD; the bias sums accumulate in LDS. part: the workgroups' partial results.
template <int KB, bool NORM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_mlp_train(const float *__restrict__ feat, int64_t B, int64_t cs, int64_t ps, const int32_t *__restrict__ labels,
            const float *__restrict__ params, float *__restrict__ part, CeWeights cw, InputGrad ig)
{
    constexpr int NACC = mlp_acc_blocks(KB);
    __shared__ struct { MlpLds L; MlpBwdLds<KB> T; bf16x8 id[2 * 64]; i32x4 id8[2 * 64]; float4 bias[4][(KB + 2) * 4 * 64]; } S;
    static_assert(sizeof(S) <= 163840 && sizeof(S) >= 3 * NACC * 4096, "the gradient sums reuse the LDS");
    MlpLds &L = S.L;
    MlpBwdLds<KB> &T = S.T;
    mlp_stage_weights<KB, 256>(params, L);
    mlp_stage_bwd<KB, 256>(params, T);
    const int lane = __lane_id(), wave = threadIdx.x / LEGS_WAVE, h = lane >> 5;
    {
        const i32x4 low = legs_turn::identity(wave & 1, lane);      // ones, as bytes
        if (wave < 2) S.id8[wave * 64 + lane] = low;
        else S.id[(wave - 2) * 64 + lane] = __builtin_bit_cast(bf16x8, low * 0x3f80);   // as bf16
    }
    float4 *bias = &S.bias[wave][lane];
#pragma unroll
    for (int i = 0; i < (KB + 2) * 4; ++i) bias[i * 64] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
    const int64_t tiles = (B + 31) / 32;
    const int64_t stride = (int64_t)gridDim.x * 4;
    const float invB = 1.0f / (float)B;
    MlpGrad<KB> G = {};
    float lsum = 0.0f;
    // a pixel's inputs, read one tile ahead: the features (lower lane half), the
    // four that this half's input gradients belong to, the label and R_u
    struct Inputs {
        float v[LEGS_MLP_IN], f[4], ru;
        int y;
    };
    const auto load = [&](int64_t tile) {
        Inputs in;
        const int64_t p = tile * 32 + (lane & 31);
        const bool valid = p < B;
#pragma unroll
        for (int e = 0; e < LEGS_MLP_IN; ++e) in.v[e] = (h == 0 && valid) ? legs_ldfeat(feat, p, e, cs, ps) : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            in.f[r] = (NORM && ig.d_feat && valid) ? legs_ldfeat(feat, p, 4 * h + r, cs, ps) : 0.0f;
        in.y = valid ? labels[p] : -1;
        in.ru = cw.ru && valid ? cw.ru[p] : 0.0f;
        return in;
    };
    int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    Inputs next = load(tile);   // (past the last tile: nothing is read)
    for (; tile < tiles; tile += stride) {
        int off = 0;
        asm volatile("" : "+s"(off));   // fragments are re-read from LDS every tile
        const int ln = lane + off;
        const TurnId id = {S.id + ln, S.id8 + ln};
        const int64_t p = tile * 32 + (lane & 31);
        const bool valid = p < B;
        const Inputs in = next;
        next = load(tile + stride);
        MlpTile<KB> F;
        mlp_tile_forward<KB, NORM>(L, in.v, F, off);
        // softmax over the pixel's K logits (this lane and its partner)
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, F.z3[b][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, LEGS_WAVE));
        // register (b, r) of this lane holds class 32 b + drow(r, 0) + 4 h
        const int y = in.y, yh = y - 4 * h;
        float sum = 0.0f, zy = 0.0f;   // zy: the label's logit, in the lane that holds it
#pragma unroll
        for (int b = 0; b < KB; ++b) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                zy = yh == 32 * b + legs_drow(r, 0) ? F.z3[b][r] : zy;
                F.z3[b][r] = __expf(F.z3[b][r] - mx);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) sum += F.z3[b][r];
        }
        sum += __shfl_xor(sum, 32, LEGS_WAVE);
        const float inv = 1.0f / sum;
        float wpx = valid ? invB : 0.0f;
        if (cw.ru && valid) {
            const float ru = in.ru;
            wpx = cw.lce * (1.0f - ru) * cw.inv_hw;
            if (h == 0) lsum += cw.lu * ru * cw.inv_hw;
        }
        if (y >= 0 && y < 32 * KB && h == ((y >> 2) & 1)) {
            const float ce = mx + __logf(sum) - zy;
            lsum += ce * wpx;
            if (cw.ru) cw.d_ru[p] = (cw.lu - cw.lce * ce) * cw.inv_hw;
        }
        __builtin_amdgcn_sched_barrier(0);
        const float pw = inv * wpx;
        f32x16 dxa = {};
        // the layer inputs transposed: columns of the weight gradients
        bf16x8 h2t[2][2];
#pragma unroll
        for (int n = 0; n < 2; ++n) turn_block<false>(F.h2[2 * n], F.h2[2 * n + 1], id, h2t[n]);
        // dz3 = (p - onehot) w_p; dh2 = W3^T dz3, dW3 = dz3 h2^T
        int yh2 = yh;
        asm volatile("" : "+v"(yh2));   // the compares are made again: 64 masks kept from above would be spilled
        f32x16 dh[2] = {};
#pragma unroll
        for (int b = 0; b < KB; ++b) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                F.z3[b][r] = fmaf(F.z3[b][r], pw, yh2 == 32 * b + legs_drow(r, 0) ? -wpx : 0.0f);
            bias_add(bias + b * 4 * LEGS_WAVE, F.z3[b]);
            bf16x8 hi[2], lo[2];
            split8(F.z3[b], 0, hi[0], lo[0]);
            split8(F.z3[b], 8, hi[1], lo[1]);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const bf16x8 a = T.t3[(mb * 2 * KB + 2 * b + q) * 64 + ln];
                    dh[mb] = legs_mfma(a, lo[q], legs_mfma(a, hi[q], dh[mb]));
                }
            __builtin_amdgcn_sched_barrier(0);
            wgrad_block<false, 2>(hi, lo, h2t, id, G.w3[b]);
        }
        // dz2 = dh2 gated by h2 > 0; dh1 = W2^T dz2, dW2 = dz2 h1^T
        bf16x8 h1t[2][2];
#pragma unroll
        for (int n = 0; n < 2; ++n) turn_block<true>(F.h1[2 * n], F.h1[2 * n + 1], id, h1t[n]);
        f32x16 dg[2] = {};
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!((float)F.h2[2 * b + (r >> 3)][r & 7] > 0.0f)) dh[b][r] = 0.0f;
            bias_add(bias + (KB + b) * 4 * LEGS_WAVE, dh[b]);
            bf16x8 hi[2], lo[2];
            split8(dh[b], 0, hi[0], lo[0]);
            split8(dh[b], 8, hi[1], lo[1]);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const bf16x8 a = T.t2[(mb * 4 + 2 * b + q) * 64 + ln];
                    dg[mb] = legs_mfma(a, lo[q], legs_mfma(a, hi[q], dg[mb]));
                }
            __builtin_amdgcn_sched_barrier(0);
            wgrad_block<true, 2>(hi, lo, h1t, id, G.w2[b]);
        }
        bf16x8 xt[2], xh[2];
        legs_turn::turn(F.x, byte_identity(id), xt);
        halves(xt, xh);                               // xh[0]: columns 0 .. 15
        // dz1 = dh1 gated by h1 > 0; dW1 and db1 against the input and its bias one
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (!((float)F.h1[2 * b + (r >> 3)][r & 7] > 0.0f)) dg[b][r] = 0.0f;
            bf16x8 hi[2], lo[2];
            split8(dg[b], 0, hi[0], lo[0]);
            split8(dg[b], 8, hi[1], lo[1]);
            if (ig.d_feat) {
                // dx = W1^T dz1: inputs 4 h + r in registers r = 0..3
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const bf16x8 a = T.t1[(2 * b + q) * 64 + ln];
                    dxa = legs_mfma(a, lo[q], legs_mfma(a, hi[q], dxa));
                }
            }
            wgrad_input(hi, lo, xh[0], id, b, G.w1);
        }
        if (ig.d_feat) {
            float dx[4] = {dxa[0], dxa[1], dxa[2], dxa[3]};
            if constexpr (NORM) {
                const float (&f)[4] = in.f;
                float ss = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) ss = fmaf(f[r], f[r], ss);
                ss += __shfl_xor(ss, 32, LEGS_WAVE);
                const float nrm = sqrtf(ss);
                const float iv = nrm > 0.0f ? 1.0f / nrm : 0.0f;
                float ud = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) ud += f[r] * iv * dx[r];
                ud += __shfl_xor(ud, 32, LEGS_WAVE);
#pragma unroll
                for (int r = 0; r < 4; ++r) dx[r] = (dx[r] - ud * (f[r] * iv)) * iv;
            }
            if (valid) {
#pragma unroll
                for (int r = 0; r < 4; ++r) ig.d_feat[(int64_t)(4 * h + r) * ig.dcs + p * ig.dps] = dx[r];
            }
        }
    }
    // the workgroup's sums over its lanes and waves
    float *dst = part + (int64_t)blockIdx.x * mlp_part_floats(KB);
    float *s_loss = reinterpret_cast<float *>(S.id);   // the last tile's fragments are read
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, LEGS_WAVE);
    __syncthreads();
    if (lane == 0) s_loss[wave] = lsum;
    __syncthreads();
    for (int u = threadIdx.x; u < (KB + 2) * 32; u += 256) {
        const int b = u >> 5, q = u & 31;   // unit q of block b: register 4 (q / 8) + q % 4, lane half (q / 4) % 2
        float s = 0.0f;
        for (int w = 0; w < 4; ++w) {
            const float *src = reinterpret_cast<const float *>(&S.bias[w][(b * 4 + (q >> 3)) * 64 + 32 * ((q >> 2) & 1)]);
#pragma unroll 8
            for (int i = 0; i < 32; ++i) s += src[4 * ((i + u) & 31) + (q & 3)];
        }
        dst[NACC * 1024 + u] = s;
    }
    if (threadIdx.x == 0)
        dst[NACC * 1024 + (KB + 2) * 32] = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
    __syncthreads();
    float4 *sum = reinterpret_cast<float4 *>(&S) + lane;
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < NACC; ++i) {
            const f32x16 &z = mlp_acc<KB>(G, i);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                sum[((wave - 1) * NACC + i) * 256 + q * 64] = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
        }
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int i = 0; i < NACC; ++i) {
            const f32x16 &z = mlp_acc<KB>(G, i);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4 v = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
#pragma unroll
                for (int w = 0; w < 3; ++w) {
                    const float4 o = sum[(w * NACC + i) * 256 + q * 64];
                    v.x += o.x;
                    v.y += o.y;
                    v.z += o.z;
                    v.w += o.w;
                }
                float *d = dst + i * 1024 + q * 256 + 4 * lane;   // 4-byte aligned rows
                d[0] = v.x;
                d[1] = v.y;
                d[2] = v.z;
                d[3] = v.w;
            }
        }
    }
}

// Sums the nwg partial results: a wave per 16 words, its four lane groups
// taking every fourth workgroup. ADD: added to grad and loss with atomics
// (calls on several streams may share them), otherwise stored.
template <int KB, bool ADD>
__global__ void __launch_bounds__(256)
k_mlp_reduce(const float *__restrict__ part, int nwg, float *__restrict__ grad, float *__restrict__ loss)
{
    constexpr int n = mlp_part_floats(KB);
    const int lane = __lane_id(), wave = threadIdx.x / LEGS_WAVE;
    const int i = (blockIdx.x * 4 + wave) * 16 + (lane & 15);
    const int param = i < n ? mlp_part_param<KB>(i) : -1;
    float s = 0.0f;
    if (param >= 0) {
#pragma unroll 8
        for (int g = lane >> 4; g < nwg; g += 4) s += part[(int64_t)g * n + i];
    }
    s += __shfl_xor(s, 16, LEGS_WAVE);
    s += __shfl_xor(s, 32, LEGS_WAVE);
    if (param >= 0 && lane < 16) {
        float *dst = param < (int)LEGS_MLP_NPARAMS(KB) ? grad + param : loss;
        if constexpr (ADD) atomicAdd(dst, s);
        else *dst = s;
    }
}

__global__ void __launch_bounds__(256)
k_zero_f32(float *__restrict__ p, int64_t n, float *__restrict__ q)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        p[i] = 0.0f;
    if (blockIdx.x == 0 && threadIdx.x == 0) *q = 0.0f;
}

} // namespace

// Workgroups of the training kernel for B pixels, at most.
static int64_t mlp_parts(int64_t B) { return std::min<int64_t>((B + 127) / 128, LEGS_MLP_MAX_PARTS); }

int64_t legs_mlp_workspace_floats(int64_t B, int32_t K) { return mlp_parts(B) * LEGS_MLP_PART_FLOATS(K / 32); }

namespace {

// The training kernel, then the sum of its partial results: added to grad and
// loss, or stored there.
int32_t mlp_train_kernels(legs_ctx *ctx, const float *feat, int64_t B, int64_t cs, int64_t ps,
                          const int32_t *labels, int32_t K, int32_t mlp_flags, const float *params,
                          float *workspace, float *grad, float *loss, const CeWeights &cw,
                          const InputGrad &ig, bool add, hipStream_t s)
{
    if (B == 0) {
        if (!add)
            hipLaunchKernelGGL(k_zero_f32, dim3(64), dim3(256), 0, s, grad, (int64_t)LEGS_MLP_NPARAMS(K / 32), loss);
        LEGS_CHECK_LAUNCH(ctx);
        return LEGS_OK;
    }
    // one workgroup per CU (one wave per SIMD), each with at least one tile per wave
    // but the last
    const int64_t g = std::min<int64_t>(mlp_parts(B), ctx->num_cus);
    const bool norm = (mlp_flags & LEGS_MLP_NORMALIZE_INPUT) != 0;
#define LEGS_MLP_TRAIN(KBV)                                                                                          \
    {                                                                                                                \
        if (norm)                                                                                                    \
            hipLaunchKernelGGL((k_mlp_train<KBV, true>), dim3((unsigned)g), dim3(256), 0, s, feat, B, cs, ps,        \
                               labels, params, workspace, cw, ig);                                                   \
        else                                                                                                         \
            hipLaunchKernelGGL((k_mlp_train<KBV, false>), dim3((unsigned)g), dim3(256), 0, s, feat, B, cs, ps,       \
                               labels, params, workspace, cw, ig);                                                   \
        const dim3 gr((mlp_part_floats(KBV) + 63) / 64);                                                             \
        if (add)                                                                                                     \
            hipLaunchKernelGGL((k_mlp_reduce<KBV, true>), gr, dim3(256), 0, s, workspace, (int)g, grad, loss);       \
        else                                                                                                         \
            hipLaunchKernelGGL((k_mlp_reduce<KBV, false>), gr, dim3(256), 0, s, workspace, (int)g, grad, loss);      \
    }
    switch (K) {
    case 32: LEGS_MLP_TRAIN(1) break;
    case 64: LEGS_MLP_TRAIN(2) break;
    case 128: LEGS_MLP_TRAIN(4) break;
    default: return legs_set_error(ctx, LEGS_ERR_ARG, "K must be 32, 64 or 128");
    }
#undef LEGS_MLP_TRAIN
    LEGS_CHECK_LAUNCH(ctx);
    return LEGS_OK;
}

} // namespace

int32_t legs_launch_mlp_grad(legs_ctx *ctx, const float *feat, int64_t B, int64_t cs, int64_t ps,
                             const int32_t *labels, int32_t K, int32_t mlp_flags, const float *params,
                             float *workspace, float *grad, float *loss, hipStream_t s)
{
    const CeWeights cw = {nullptr, nullptr, 1.0f, 0.0f, 0.0f};
    const InputGrad ig = {nullptr, 0, 0};
    return mlp_train_kernels(ctx, feat, B, cs, ps, labels, K, mlp_flags, params, workspace, grad, loss, cw, ig, false,
                             s);
}

int32_t legs_launch_semantic_loss_grad(legs_ctx *ctx, const float *feat, const float *ru, int64_t P,
                                       int64_t cs, int64_t ps, const int32_t *labels, int32_t K,
                                       int32_t mlp_flags, const float *params, float lambda_ce,
                                       float lambda_u, float inv_hw, float *workspace, float *grad,
                                       float *d_feat, int64_t dcs, int64_t dps, float *d_ru,
                                       float *loss, hipStream_t s)
{
    const CeWeights cw = {ru, d_ru, lambda_ce, lambda_u, inv_hw};
    const InputGrad ig = {d_feat, dcs, dps};
    return mlp_train_kernels(ctx, feat, P, cs, ps, labels, K, mlp_flags, params, workspace, grad, loss, cw, ig, true,
                             s);
}

// ---- fused Adam over parameter groups -------------------------------------------

namespace {

// Elements per workgroup of k_adam: four neighbouring floats per thread, four times.
constexpr int ADAM_CHUNK = 256 * 4 * 4;

struct AdamArgs {
    legs_adam_group g[LEGS_ADAM_MAX_GROUPS];
    int64_t bstart[LEGS_ADAM_MAX_GROUPS + 1];   // first workgroup of each group
    int vec[LEGS_ADAM_MAX_GROUPS];              // the group's four arrays are 16-byte aligned
    int n_groups;
    // omb = 1 - b rounded once from double (1 - 0.999f would be 1.3e-5 off
    // 0.001); c1 = 1 / (1 - b1^t), c2 = 1 / (1 - b2^t)
    float lr, b1, b2, omb1, omb2, eps, c1, c2;
};

__device__ __forceinline__ float adam_one(const AdamArgs &A, float p, float g, float &m, float &v)
{
    m = A.b1 * m + A.omb1 * g;
    v = A.b2 * v + A.omb2 * g * g;
    return p - A.lr * (m * A.c1) / (sqrtf(v * A.c2) + A.eps);
}

// Each workgroup updates one ADAM_CHUNK of one group, the group found by a
// wave-uniform walk over the workgroup counts (so its pointers are scalars);
// float4 access where the group is aligned, and the clamp test takes one
// remainder per four elements.
__global__ void __launch_bounds__(256)
k_adam(AdamArgs A)
{
    int k = 0;
    while (k + 1 < A.n_groups && (int64_t)blockIdx.x >= A.bstart[k + 1]) ++k;
    const legs_adam_group &G = A.g[k];
    const int64_t c0 = ((int64_t)blockIdx.x - A.bstart[k]) * ADAM_CHUNK;
    const int64_t c1 = c0 + ADAM_CHUNK < G.n ? c0 + ADAM_CHUNK : G.n;
    const int64_t ce = G.clamp_every;
    int64_t j0 = c0;
    if (A.vec[k]) {
        const int64_t q1 = c1 / 4;
        for (int64_t q = c0 / 4 + threadIdx.x; q < q1; q += 256) {
            float4 p = reinterpret_cast<const float4 *>(G.param)[q];
            const float4 g = reinterpret_cast<const float4 *>(G.grad)[q];
            float4 m = reinterpret_cast<const float4 *>(G.m)[q];
            float4 v = reinterpret_cast<const float4 *>(G.v)[q];
            p.x = adam_one(A, p.x, g.x, m.x, v.x);
            p.y = adam_one(A, p.y, g.y, m.y, v.y);
            p.z = adam_one(A, p.z, g.z, m.z, v.z);
            p.w = adam_one(A, p.w, g.w, m.w, v.w);
            if (ce > 0) {
                const int64_t r0 = (4 * q) % ce;
                const int64_t r1 = r0 + 1 == ce ? 0 : r0 + 1, r2 = r1 + 1 == ce ? 0 : r1 + 1,
                              r3 = r2 + 1 == ce ? 0 : r2 + 1;
                const float lo = G.clamp_lo, hi = G.clamp_hi;
                const int64_t off = G.clamp_offset;
                if (r0 == off) p.x = fminf(fmaxf(p.x, lo), hi);
                if (r1 == off) p.y = fminf(fmaxf(p.y, lo), hi);
                if (r2 == off) p.z = fminf(fmaxf(p.z, lo), hi);
                if (r3 == off) p.w = fminf(fmaxf(p.w, lo), hi);
            }
            reinterpret_cast<float4 *>(G.m)[q] = m;
            reinterpret_cast<float4 *>(G.v)[q] = v;
            reinterpret_cast<float4 *>(G.param)[q] = p;
        }
        j0 = 4 * q1;
    }
    for (int64_t j = j0 + threadIdx.x; j < c1; j += 256) {
        float m = G.m[j], v = G.v[j];
        float p = adam_one(A, G.param[j], G.grad[j], m, v);
        G.m[j] = m;
        G.v[j] = v;
        if (ce > 0 && (j % ce) == G.clamp_offset) p = fminf(fmaxf(p, G.clamp_lo), G.clamp_hi);
        G.param[j] = p;
    }
}

} // namespace

int32_t legs_launch_adam(legs_ctx *ctx, const legs_adam_group *groups, int32_t n_groups,
                         int32_t step, float lr, double beta1, double beta2, float eps, hipStream_t s)
{
    AdamArgs A;
    A.n_groups = n_groups;
    A.bstart[0] = 0;
    for (int k = 0; k < n_groups; ++k) {
        const legs_adam_group &G = groups[k];
        A.g[k] = G;
        A.bstart[k + 1] = A.bstart[k] + (G.n + ADAM_CHUNK - 1) / ADAM_CHUNK;
        A.vec[k] = ((reinterpret_cast<uintptr_t>(G.param) | reinterpret_cast<uintptr_t>(G.grad) |
                     reinterpret_cast<uintptr_t>(G.m) | reinterpret_cast<uintptr_t>(G.v)) & 15) == 0;
    }
    A.lr = lr; A.eps = eps;
    A.b1 = (float)beta1; A.b2 = (float)beta2;
    A.omb1 = (float)(1.0 - beta1); A.omb2 = (float)(1.0 - beta2);
    A.c1 = (float)(1.0 / (1.0 - pow(beta1, (double)step)));
    A.c2 = (float)(1.0 / (1.0 - pow(beta2, (double)step)));
    const int64_t blocks = A.bstart[n_groups];
    if (blocks == 0) return LEGS_OK;
    hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), dim3(256), 0, s, A);
    LEGS_CHECK_LAUNCH(ctx);
    return LEGS_OK;
}
