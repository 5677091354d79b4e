// Adaptive spatial smoothing (Sec. 3.4.2, Eqs. 13-14; PE and MLP of Table 4),
// gfx950.
//
//   s_MLP = MLP(PE(p)), PE of configuration 0 (the position itself), MLP
//   3 -> 128 -> 128 -> 128 -> 8 with ReLU after the first three layers;
//   L_smo = mean_g [ |s_MLP - s_G*| + max(u_G*, w_s) |s_MLP* - s_G| ]
//   (* = stop gradient): the first term trains the MLP, the second pulls s_G
//   towards the smoothed feature; u and the position receive nothing.
//
// BF16 weights and hidden activations, FP32 accumulation on
// v_mfma_f32_32x32x16_bf16, every layer transposed (units x Gaussians) as in
// the decoders. The position enters the first layer unrounded: each
// coordinate is split into three bf16 parts (hi + mid + lo = the float32
// value exactly), so the first layer computes bf16(W1) p + b1 with p in
// float32. Backward through the layers on the same MFMAs with the upstream
// gradient split into two bf16 parts (hi + lo, 16 significant bits): W^T
// fragments stay in LDS next to the forward ones (153 KB in all).
//
//  k_smooth_fwd_bwd  per 32-Gaussian tile (two per wave): forward, loss,
//                    dL/ds_G (accumulated into the channel gradient), and
//                    dz of every layer; writes the bf16 hidden activations and
//                    dz (as its two bf16 parts) into the workspace planes in
//                    the weight gradient's operand order, each block turned by
//                    the matrix unit so that a wave stores 1 KB contiguous.
//                    Bound by its stores, 2.4 KB a Gaussian (without them it
//                    takes 0.13 ms for 1M): plane after plane and past the
//                    caches, 0.64 ms.
//  k_smooth_wgrad    dW_l = sum_g dz_l h_(l-1)^T and db_l = sum_g dz_l: the
//                    Gaussians are the MFMA contraction, each operand one
//                    16-byte load (a wave's load of a 128-row plane is 1 KB
//                    contiguous); whole products per wave, so that the planes
//                    are read once, past the caches, and a third of the atomics
//                    are left. Bound by the reads: 0.41 ms
//                    for 1M, a row block per wave and 245 chunks 0.56.
#include "legs_internal.h"
#include "legs_decode_internal.h"
#include "lane_transpose.h"

namespace {

typedef legs_f32x16 f32x16;
typedef legs_bf16x8 bf16x8;

constexpr int SH = LEGS_SMOOTH_H;         // 128 hidden units
constexpr int SB = SH / 32;               // 4 blocks
constexpr int SK = SH / 16;               // 8 k-steps
constexpr int SNT = 2;                    // tiles per wave

struct SmoothLds {
    bf16x8 w1[SB * 64];
    bf16x8 w2[SB * SK * 64], bb2[SB * 64];
    bf16x8 w3[SB * SK * 64], bb3[SB * 64];
    bf16x8 w4[SK * 64], bb4[64];
    bf16x8 t4[SB * 64];                   // W4^T
    bf16x8 t3[SB * SK * 64], t2[SB * SK * 64];
};

__device__ __forceinline__ void smooth_stage(const float *__restrict__ P, SmoothLds &L)
{
    constexpr int NT = 256;
    const float *W1 = P + LEGS_SMOOTH_OFF_W1, *b1 = P + LEGS_SMOOTH_OFF_B1;
    const float *W2 = P + LEGS_SMOOTH_OFF_W2, *b2 = P + LEGS_SMOOTH_OFF_B2;
    const float *W3 = P + LEGS_SMOOTH_OFF_W3, *b3 = P + LEGS_SMOOTH_OFF_B3;
    const float *W4 = P + LEGS_SMOOTH_OFF_W4, *b4 = P + LEGS_SMOOTH_OFF_B4;
    // hidden layers and their transposes: fragment (block, k-step, lane, e)
    // = row 32 block + lane % 32, column legs_khid(k-step, lane / 32, e)
    auto rows = [](const float *W) {
        return [W](int i) {
            const int l = i & 63, ks = (i >> 6) % SK, mb = (i >> 6) / SK;
            return legs_frag_row(W + (32 * mb + (l & 31)) * SH, ks, l >> 5);
        };
    };
    auto columns = [](const float *W) {
        return [W](int i) {
            const int l = i & 63, ks = (i >> 6) % SK, mb = (i >> 6) / SK;
            bf16x8 f;
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = (__bf16)W[legs_khid(ks, l >> 5, e) * SH + 32 * mb + (l & 31)];
            return f;
        };
    };
    legs_stage_frags<SB * SK * 64, NT, 4>(L.w2, rows(W2));
    legs_stage_frags<SB * SK * 64, NT, 4>(L.w3, rows(W3));
    legs_stage_frags<SB * SK * 64, NT, 4>(L.t3, columns(W3));
    legs_stage_frags<SB * SK * 64, NT, 4>(L.t2, columns(W2));
    legs_stage_frags<SK * 64, NT, 2>(L.w4, [&](int i) {      // W4: rows 8..31 zero
        const int l = i & 63, row = l & 31;
        return row < LEGS_SMOOTH_OUT ? legs_frag_row(W4 + row * SH, i >> 6, l >> 5) : (bf16x8){};
    });
    // layer 1: lower half [wx wy wz wx wy wz wx wy], upper half [wz b_hi b_mid b_lo 0 0 0 0]
    legs_stage_frags<SB * 64, NT, 1>(L.w1, [&](int i) {
        const int row = 32 * (i >> 6) + (i & 31);
        const __bf16 x = (__bf16)W1[row * 3], y = (__bf16)W1[row * 3 + 1], z = (__bf16)W1[row * 3 + 2];
        __bf16 p[3];
        legs_split3(b1[row], p[0], p[1], p[2]);
        const __bf16 o = (__bf16)0.0f;
        const bf16x8 lower = {x, y, z, x, y, z, x, y}, upper = {z, p[0], p[1], p[2], o, o, o, o};
        return (i >> 5) & 1 ? upper : lower;
    });
    // W4^T: k-slot e of half h is output legs_khid(0, h, e) (outputs 0..7
    // sit in slots 0..3 of both halves)
    legs_stage_frags<SB * 64, NT, 1>(L.t4, [&](int i) {
        const int l = i & 63, mb = i >> 6;
        bf16x8 f = {};
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = (__bf16)W4[legs_khid(0, l >> 5, e) * SH + 32 * mb + (l & 31)];
        return f;
    });
    legs_stage_frags<SB * 64, NT, 1>(L.bb2, [&](int i) { return legs_frag_bias(b2[32 * (i >> 6) + (i & 31)], (i >> 5) & 1); });
    legs_stage_frags<SB * 64, NT, 1>(L.bb3, [&](int i) { return legs_frag_bias(b3[32 * (i >> 6) + (i & 31)], (i >> 5) & 1); });
    legs_stage_frags<64, NT, 1>(L.bb4, [&](int i) {
        return legs_frag_bias((i & 31) < LEGS_SMOOTH_OUT ? b4[i & 31] : 0.0f, (i >> 5) & 1);
    });
}

// bf16 split of 8 accumulator values (first .. first + 7): hi = bf16(z),
// lo = bf16(z - hi)
__device__ __forceinline__ void split_bf16x8(const f32x16 &z, int first, bf16x8 &hi, bf16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 a = (__bf16)z[first + e];
        hi[e] = a;
        lo[e] = (__bf16)(z[first + e] - (float)a);
    }
}

// Workspace planes are kept in the operand order of the weight-gradient
// MFMAs (legs_lt::frag_at with the Gaussians as the columns), so a forward
// store is one 16-byte fragment and a weight-gradient load of a 128-row plane
// is 1 KB contiguous per wave.
using legs_lt::frag_at;

struct SmoothArgs {
    const float *mean, *ch;
    int32_t C, sem, uch;
    int64_t n, Gp;
    const float *params;
    float w_s, inv_n;             // inv_n = lambda_smo / n
    float *d_ch, *loss;
    __bf16 *X, *H1, *H2, *H3;     // 16 and 128 (x 3) rows, fragment order (frag_at)
    __bf16 *D1, *D2, *D3, *D4;    // dz: hi plane then lo plane, 128 (x 3) and 8 rows
};

// Hidden-layer step: acc of block mb from B fragments x[NT][KS] and A
// fragments a(mb, ks) in LDS.
template <int KS>
__device__ __forceinline__ void layer_block(const bf16x8 *__restrict__ wA, const bf16x8 *__restrict__ bias,
                                            int mb, int lane, const bf16x8 (&x)[SNT][KS], f32x16 (&z)[SNT])
{
    const f32x16 cb = bias ? legs_mfma(bias[mb * 64 + lane], mlp_bias_ones(__lane_id() >> 5), (f32x16){}) : (f32x16){};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a = wA[(mb * KS + ks) * 64 + lane];
#pragma unroll
        for (int t = 0; t < SNT; ++t) z[t] = legs_mfma(a, x[t][ks], ks == 0 ? cb : z[t]);
    }
}

// Lanes and Gaussians of a tile: lane l holds Gaussian l % 32 with bits 2 and 3
// swapped, so that the 16 rows of a lane half in an MFMA result are two runs of
// 8 Gaussians in order (rows legs_drow(r, h): Gaussians 8 h + r and, from r = 8,
// 16 more), the two 16-byte fragments of the planes.
__device__ __forceinline__ int swap23(int x) { return (x & ~12) | ((x & 4) << 1) | ((x & 8) >> 1); }

using legs_turn::i32x4;

// A block of 32 units x the tile's 32 Gaussians turned (legs_turn::turn). id: this
// lane's identity fragments, [low, high byte][k-step].
__device__ __forceinline__ void turn(const bf16x8 &f0, const bf16x8 &f1, const i32x4 *id, bf16x8 (&out)[2])
{
    legs_turn::turn(f0, f1, [&](int k) { return id[k * LEGS_WAVE]; }, out);
}

// Row block mb of a 128-row plane: 1 KB contiguous per fragment.
__device__ __forceinline__ void store_block(__bf16 *__restrict__ plane, int64_t g0, int mb, const bf16x8 &f0,
                                            const bf16x8 &f1, const i32x4 *id, int lane)
{
    bf16x8 f[2];
    turn(f0, f1, id, f);
    __bf16 *p = plane + frag_at(g0, SH, 32 * mb) + 8 * lane;
    __builtin_nontemporal_store(f[0], reinterpret_cast<bf16x8 *>(p));
    __builtin_nontemporal_store(f[1], reinterpret_cast<bf16x8 *>(p + SB * 64 * 8));
    __builtin_amdgcn_sched_barrier(0);          // one block's registers at a time
}

// A plane of R <= 16 rows from one fragment; lane column n holds row row(n).
template <int R, typename RowOf>
__device__ __forceinline__ void store_narrow(__bf16 *__restrict__ plane, int64_t g0, const bf16x8 &v, const i32x4 *id,
                                             int lane, RowOf row_of)
{
    bf16x8 f[2];
    turn(v, (bf16x8){}, id, f);
    if ((lane & 31) >= R) return;
    __bf16 *p = plane + frag_at(g0, R, row_of(lane & 31)) + R * 8 * (lane >> 5);
    *reinterpret_cast<bf16x8 *>(p) = f[0];
    *reinterpret_cast<bf16x8 *>(p + 2 * R * 8) = f[1];
}

__global__ void __launch_bounds__(256)
k_smooth_fwd_bwd(SmoothArgs A)
{
    __shared__ SmoothLds L;
    __shared__ i32x4 ident[4 * 64];        // the identity in accumulator order (turn)
    __shared__ float s_loss[4];
    smooth_stage(A.params, L);
    const int lane = __lane_id(), wave = threadIdx.x / LEGS_WAVE, h = lane >> 5;
    ident[wave * LEGS_WAVE + lane] = legs_turn::identity(wave, lane);
    __syncthreads();
    const int64_t groups = (A.n + 32 * SNT - 1) / (32 * SNT);
    const int64_t stride = (int64_t)gridDim.x * 4;
    float lsum = 0.0f;
    for (int64_t grp = (int64_t)blockIdx.x * 4 + wave; grp < groups; grp += stride) {
        int off = 0;
        asm volatile("" : "+s"(off));     // fragments are re-read from LDS every group
        const int ln = lane + off;
        const i32x4 *id = ident + ln;
        int64_t gi[SNT];
        bool valid[SNT];
        bf16x8 x[SNT][1];
#pragma unroll
        for (int t = 0; t < SNT; ++t) {
            gi[t] = (grp * SNT + t) * 32 + swap23(lane & 31);
            valid[t] = gi[t] < A.n;
            float p[3] = {0.0f, 0.0f, 0.0f};
            if (valid[t]) {
                p[0] = A.mean[3 * gi[t] + 0];
                p[1] = A.mean[3 * gi[t] + 1];
                p[2] = A.mean[3 * gi[t] + 2];
            }
            __bf16 s[3][3];
#pragma unroll
            for (int c = 0; c < 3; ++c) legs_split3(p[c], s[c][0], s[c][1], s[c][2]);
            // lower half: x_hi y_hi z_hi x_mid y_mid z_mid x_lo y_lo; upper: z_lo 1 1 1 0...
            bf16x8 v;
            if (h == 0) {
                v[0] = s[0][0]; v[1] = s[1][0]; v[2] = s[2][0];
                v[3] = s[0][1]; v[4] = s[1][1]; v[5] = s[2][1];
                v[6] = s[0][2]; v[7] = s[1][2];
            } else {
                v[0] = s[2][2]; v[1] = (__bf16)1.0f; v[2] = (__bf16)1.0f; v[3] = (__bf16)1.0f;
                v[4] = v[5] = v[6] = v[7] = (__bf16)0.0f;
            }
            x[t][0] = v;
        }
        // forward
        bf16x8 h1[SNT][SK], h2[SNT][SK], h3[SNT][SK];
#pragma unroll
        for (int mb = 0; mb < SB; ++mb) {
            f32x16 z[SNT];
            layer_block<1>(L.w1, nullptr, mb, ln, x, z);
#pragma unroll
            for (int t = 0; t < SNT; ++t) {
                h1[t][2 * mb] = relu_bf16x8(z[t], 0);
                h1[t][2 * mb + 1] = relu_bf16x8(z[t], 8);
            }
        }
#pragma unroll
        for (int mb = 0; mb < SB; ++mb) {
            f32x16 z[SNT];
            layer_block<SK>(L.w2, L.bb2, mb, ln, h1, z);
#pragma unroll
            for (int t = 0; t < SNT; ++t) {
                h2[t][2 * mb] = relu_bf16x8(z[t], 0);
                h2[t][2 * mb + 1] = relu_bf16x8(z[t], 8);
            }
        }
#pragma unroll
        for (int mb = 0; mb < SB; ++mb) {
            f32x16 z[SNT];
            layer_block<SK>(L.w3, L.bb3, mb, ln, h2, z);
#pragma unroll
            for (int t = 0; t < SNT; ++t) {
                h3[t][2 * mb] = relu_bf16x8(z[t], 0);
                h3[t][2 * mb + 1] = relu_bf16x8(z[t], 8);
            }
        }
        f32x16 s4[SNT];
        layer_block<SK>(L.w4, L.bb4, 0, ln, h3, s4);
        // inputs and hidden activations to the workspace (zero for padding
        // Gaussians). Input rows 0..8: the split coordinates (part-major), row 9
        // ones, rows 10..15 zero; lane half h holds rows 8 h .. 8 h + 7
        if (h == 1) {
#pragma unroll
            for (int t = 0; t < SNT; ++t) x[t][0][2] = x[t][0][3] = (__bf16)0.0f;
        }
        if (legs_ballot(valid[0] && valid[1]) != ~0ull) {
#pragma unroll
            for (int t = 0; t < SNT; ++t) {
                if (valid[t]) continue;
                x[t][0] = (bf16x8){};
#pragma unroll
                for (int ks = 0; ks < SK; ++ks) h1[t][ks] = h2[t][ks] = h3[t][ks] = (bf16x8){};
            }
        }
#pragma unroll
        for (int t = 0; t < SNT; ++t) {
            const int64_t g0 = (grp * SNT + t) * 32;
            store_narrow<16>(A.X, g0, x[t][0], id, lane, [](int n) { return swap23(n); });
#pragma unroll
            for (int mb = 0; mb < SB; ++mb) store_block(A.H1, g0, mb, h1[t][2 * mb], h1[t][2 * mb + 1], id, lane);
#pragma unroll
            for (int mb = 0; mb < SB; ++mb) store_block(A.H2, g0, mb, h2[t][2 * mb], h2[t][2 * mb + 1], id, lane);
#pragma unroll
            for (int mb = 0; mb < SB; ++mb) store_block(A.H3, g0, mb, h3[t][2 * mb], h3[t][2 * mb + 1], id, lane);
        }
        // loss and dz4: outputs 4 h + r in registers r = 0..3
        f32x16 dz4[SNT];
#pragma unroll
        for (int t = 0; t < SNT; ++t) {
            dz4[t] = (f32x16){};
            float sg[4] = {0.0f, 0.0f, 0.0f, 0.0f}, u = 0.0f;
            if (valid[t]) {
                const float *row = A.ch + gi[t] * A.C;
#pragma unroll
                for (int r = 0; r < 4; ++r) sg[r] = row[A.sem + 4 * h + r];
                u = row[A.uch];
            }
            float diff[4], ss = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                diff[r] = s4[t][r] - sg[r];
                ss = fmaf(diff[r], diff[r], ss);
            }
            ss += __shfl_xor(ss, 32, LEGS_WAVE);
            const float nrm = sqrtf(ss);
            const float wgt = fmaxf(u, A.w_s);
            if (!valid[t] || !(nrm > 0.0f)) continue;
            if (h == 0) lsum += nrm * (1.0f + wgt) * A.inv_n;
            const float inv = A.inv_n / nrm;
            float *drow = A.d_ch + gi[t] * A.C + A.sem + 4 * h;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                dz4[t][r] = diff[r] * inv;
                drow[r] += -wgt * diff[r] * inv;
            }
        }
        // backward through the layers: dz_l split into hi and lo bf16 parts,
        // which are also what the planes keep (hi plane, then lo plane). dz is
        // exactly zero for padding Gaussians (dz4 is, and every lower dz is a
        // product with it), so the planes hold zeros there.
        // dh3 = W4^T dz4 (one k-step: outputs 0..7 in slots 0..3 of both halves)
        bf16x8 bh[SNT][SK], bl[SNT][SK];
        f32x16 dz[SNT][SB];
#pragma unroll
        for (int t = 0; t < SNT; ++t) split_bf16x8(dz4[t], 0, bh[t][0], bl[t][0]);
#pragma unroll
        for (int mb = 0; mb < SB; ++mb) {
            const bf16x8 a = L.t4[mb * 64 + ln];
#pragma unroll
            for (int t = 0; t < SNT; ++t)
                dz[t][mb] = legs_mfma(a, bl[t][0], legs_mfma(a, bh[t][0], (f32x16){}));
        }
#pragma unroll
        for (int t = 0; t < SNT; ++t)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const bf16x8 &f = p ? bl[t][0] : bh[t][0];
                __bf16 *plane = A.D4 + p * LEGS_SMOOTH_OUT * A.Gp;
                // outputs 4 h + i for i < 4: column n of the turned block is output n
                store_narrow<LEGS_SMOOTH_OUT>(plane, (grp * SNT + t) * 32, f, id, lane, [](int n) { return n; });
            }
        // ReLU gates from the stored activations (positive exactly where z > 0)
        auto gate = [&](const bf16x8 (&hf)[SNT][SK]) {
#pragma unroll
            for (int t = 0; t < SNT; ++t)
#pragma unroll
                for (int mb = 0; mb < SB; ++mb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (!((float)hf[t][2 * mb + (r >> 3)][r & 7] > 0.0f)) dz[t][mb][r] = 0.0f;
        };
        auto back = [&](const bf16x8 *__restrict__ T, __bf16 *plane) {
#pragma unroll
            for (int t = 0; t < SNT; ++t)
#pragma unroll
                for (int mb = 0; mb < SB; ++mb) {
                    split_bf16x8(dz[t][mb], 0, bh[t][2 * mb], bl[t][2 * mb]);
                    split_bf16x8(dz[t][mb], 8, bh[t][2 * mb + 1], bl[t][2 * mb + 1]);
                }
#pragma unroll
            for (int t = 0; t < SNT; ++t)
#pragma unroll
                for (int mb = 0; mb < SB; ++mb) {
                    const int64_t g0 = (grp * SNT + t) * 32;
                    store_block(plane, g0, mb, bh[t][2 * mb], bh[t][2 * mb + 1], id, lane);
                }
#pragma unroll
            for (int t = 0; t < SNT; ++t)
#pragma unroll
                for (int mb = 0; mb < SB; ++mb)
                    store_block(plane + SH * A.Gp, (grp * SNT + t) * 32, mb, bl[t][2 * mb], bl[t][2 * mb + 1], id, lane);
            if (!T) return;
#pragma unroll
            for (int mb = 0; mb < SB; ++mb) {
                f32x16 acc[SNT];
#pragma unroll
                for (int t = 0; t < SNT; ++t) acc[t] = (f32x16){};
#pragma unroll
                for (int ks = 0; ks < SK; ++ks) {
                    const bf16x8 a = T[(mb * SK + ks) * 64 + ln];
#pragma unroll
                    for (int t = 0; t < SNT; ++t) acc[t] = legs_mfma(a, bl[t][ks], legs_mfma(a, bh[t][ks], acc[t]));
                }
#pragma unroll
                for (int t = 0; t < SNT; ++t) dz[t][mb] = acc[t];
            }
        };
        gate(h3);
        back(L.t3, A.D3);     // dz3 stored; dh2 = W3^T dz3
        gate(h2);
        back(L.t2, A.D2);     // dz2 stored; dh1 = W2^T dz2
        gate(h1);
        back(nullptr, A.D1);  // dz1 stored
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, LEGS_WAVE);
    if (lane == 0) s_loss[wave] = lsum;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float v = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
        if (v != 0.0f) atomicAdd(A.loss, v);
    }
}

// dW[m][k] += sum_g (Dhi + Dlo)[m][g] B[k][g], db[m] += sum_g (Dhi + Dlo)[m][g].
// Three kinds of workgroups (blockIdx.y), of about 12.5 KB per 16 Gaussians each:
// 0: D2 x H1 -> W2, b2;  1: D3 x H2 -> W3, b3;  2: D1 x X (rows 0..8 = split
// coordinates, row 9 = ones) -> W1 [128][3], b1, and D4 (8 rows) x H3 -> W4, b4.
// A wave owns whole products, all 16 blocks of a 128 x 128 one, for its steps of
// 16 Gaussians, so that every fragment is read once (with a row block per wave,
// B was read four times and the L2 was the limit), and has WG_AHEAD steps in
// flight; the waves of a workgroup sum in LDS before the atomics.
constexpr int WG_AHEAD = 3;

// The 1 KB fragments of one step: DN of D hi and of D lo, BN of B; rows past a
// plane's (DR, BR < 32) read its row 0 and count as zero.
template <int DR, int BR>
struct SmoothStep {
    static constexpr int DN = (DR + 31) / 32, BN = (BR + 31) / 32;
    bf16x8 hi[DN], lo[DN], b[BN];
    __device__ __forceinline__ void load(const __bf16 *D, const __bf16 *B, int64_t Gp, int64_t g, int lane)
    {
        const int r = lane & 31, h = lane >> 5;
        const int64_t gl = g + 8 * h;
#pragma unroll
        for (int k = 0; k < DN; ++k) {
            const int64_t o = frag_at(gl, DR, DR >= 32 || r < DR ? 32 * k + r : 0);
            hi[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(D + o));
            lo[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(D + DR * Gp + o));
        }
#pragma unroll
        for (int k = 0; k < BN; ++k)
            b[k] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(B + frag_at(gl, BR, BR >= 32 || r < BR ? 32 * k + r : 0)));
    }
    __device__ __forceinline__ void add(f32x16 (&acc)[DN][BN], float (&db)[DN], bool bias, int lane)
    {
        const int r = lane & 31;
        const bf16x8 zero = {};
        if constexpr (DR < 32) {
            hi[0] = r < DR ? hi[0] : zero;
            lo[0] = r < DR ? lo[0] : zero;
        }
        if constexpr (BR < 32) b[0] = r < BR ? b[0] : zero;
#pragma unroll
        for (int m = 0; m < DN; ++m)
#pragma unroll
            for (int k = 0; k < BN; ++k) acc[m][k] = legs_mfma(lo[m], b[k], legs_mfma(hi[m], b[k], acc[m][k]));
        if (bias) {
#pragma unroll
            for (int m = 0; m < DN; ++m)
#pragma unroll
                for (int e = 0; e < 8; ++e) db[m] += (float)hi[m][e] + (float)lo[m][e];
        }
    }
};

// Sum of z over the workgroup's waves, in wave 0's order (plain reads and
// writes of LDS, one wave after the other).
template <int N>
__device__ __forceinline__ void block_sum(f32x16 (&z)[N], float4 *lds, int lane, int wave)
{
    for (int w = 3; w >= 0; --w) {
        if (wave == w) {
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float4 &x = lds[(n * 4 + q) * LEGS_WAVE + lane];
                    float4 v = make_float4(z[n][4 * q], z[n][4 * q + 1], z[n][4 * q + 2], z[n][4 * q + 3]);
                    if (w < 3) {
                        const float4 y = x;
                        v = make_float4(v.x + y.x, v.y + y.y, v.z + y.z, v.w + y.w);
                    }
                    x = v;
                }
        }
        __syncthreads();
    }
}

// One product over the workgroup's steps; W(row, col, v) takes its elements.
template <int DR, int BR, bool BIAS, typename W>
__device__ __forceinline__ void smooth_product(const SmoothArgs &A, const __bf16 *D, const __bf16 *B, float4 *lds,
                                               float *__restrict__ db_out, W add)
{
    using Step = SmoothStep<DR, BR>;
    const int lane = __lane_id(), wave = threadIdx.x / LEGS_WAVE, h = lane >> 5;
    const int64_t steps = A.Gp / 16, stride = (int64_t)gridDim.x * 4;
    const int64_t s0 = (int64_t)blockIdx.x * 4 + wave;
    f32x16 acc[Step::DN][Step::BN] = {};
    float db[Step::DN] = {};
    Step ring[WG_AHEAD];
    auto at = [&](int64_t s) { return 16 * min(s, steps - 1); };
#pragma unroll
    for (int k = 0; k < WG_AHEAD; ++k) ring[k].load(D, B, A.Gp, at(s0 + k * stride), lane);
#pragma unroll 1
    for (int64_t s = s0; s < steps; s += WG_AHEAD * stride) {
#pragma unroll
        for (int k = 0; k < WG_AHEAD; ++k) {
            if (s + k * stride < steps) ring[k].add(acc, db, BIAS, lane);
            ring[k].load(D, B, A.Gp, at(s + (k + WG_AHEAD) * stride), lane);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (BIAS) {
#pragma unroll
        for (int m = 0; m < Step::DN; ++m) {
            const float v = db[m] + __shfl_xor(db[m], 32, LEGS_WAVE);
            if (h == 0 && 32 * m + lane < DR && v != 0.0f) atomicAdd(db_out + 32 * m + lane, v);
        }
    }
    block_sum(reinterpret_cast<f32x16(&)[Step::DN * Step::BN]>(acc), lds, lane, wave);
    for (int n = wave; n < Step::DN * Step::BN; n += 4)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = lds[(n * 4 + q) * LEGS_WAVE + lane];
            const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int row = 32 * (n / Step::BN) + legs_drow(4 * q + u, h), col = 32 * (n % Step::BN) + (lane & 31);
                if (row < DR && col < BR && v[u] != 0.0f) add(row, col, v[u]);
            }
        }
    __syncthreads();
}

__global__ void __launch_bounds__(256)
k_smooth_wgrad(SmoothArgs A, float *__restrict__ grad)
{
    __shared__ float4 lds[SB * SB * 4 * LEGS_WAVE];
    if (blockIdx.y < 2) {
        const int off = blockIdx.y ? LEGS_SMOOTH_OFF_W3 : LEGS_SMOOTH_OFF_W2;
        smooth_product<SH, SH, true>(A, blockIdx.y ? A.D3 : A.D2, blockIdx.y ? A.H2 : A.H1, lds,
                                     grad + (blockIdx.y ? LEGS_SMOOTH_OFF_B3 : LEGS_SMOOTH_OFF_B2),
                                     [=](int row, int col, float v) { atomicAdd(grad + off + row * SH + col, v); });
    } else {
        smooth_product<SH, 16, false>(A, A.D1, A.X, lds, nullptr, [=](int row, int col, float v) {
            if (col < 9) atomicAdd(grad + LEGS_SMOOTH_OFF_W1 + row * 3 + col % 3, v);
            else if (col == 9) atomicAdd(grad + LEGS_SMOOTH_OFF_B1 + row, v);
        });
        smooth_product<LEGS_SMOOTH_OUT, SH, true>(A, A.D4, A.H3, lds, grad + LEGS_SMOOTH_OFF_B4,
                                                  [=](int row, int col, float v) {
                                                      atomicAdd(grad + LEGS_SMOOTH_OFF_W4 + row * SH + col, v);
                                                  });
    }
}

struct SmoothLayout {
    int64_t Gp, X, H1, H2, H3, D1, D2, D3, D4, total;
};

SmoothLayout smooth_layout(int64_t n)
{
    SmoothLayout L;
    L.Gp = (n + 63) / 64 * 64;
    const int64_t plane = L.Gp * 2;       // one bf16 row
    int64_t o = 0;
    L.X = o;  o += 16 * plane;
    L.H1 = o; o += SH * plane;
    L.H2 = o; o += SH * plane;
    L.H3 = o; o += SH * plane;
    L.D1 = o; o += 2 * SH * plane;            // hi and lo bf16 planes
    L.D2 = o; o += 2 * SH * plane;
    L.D3 = o; o += 2 * SH * plane;
    L.D4 = o; o += 2 * LEGS_SMOOTH_OUT * plane;
    L.total = o;
    return L;
}

} // namespace

int64_t legs_smooth_workspace_bytes(int64_t n) { return smooth_layout(n).total; }

int32_t legs_launch_smooth(legs_ctx *ctx, const float *mean, const float *channels, int32_t C, int32_t sem,
                           int32_t uch, int64_t n, const float *params, float w_s, float lambda_smo,
                           void *workspace, float *grad, float *d_channels, float *loss, hipStream_t s)
{
    if (n == 0) return LEGS_OK;
    const SmoothLayout Lw = smooth_layout(n);
    char *ws = static_cast<char *>(workspace);
    SmoothArgs A;
    A.mean = mean;
    A.ch = channels;
    A.C = C;
    A.sem = sem;
    A.uch = uch;
    A.n = n;
    A.Gp = Lw.Gp;
    A.params = params;
    A.w_s = w_s;
    A.inv_n = lambda_smo / (float)n;
    A.d_ch = d_channels;
    A.loss = loss;
    A.X = reinterpret_cast<__bf16 *>(ws + Lw.X);
    A.H1 = reinterpret_cast<__bf16 *>(ws + Lw.H1);
    A.H2 = reinterpret_cast<__bf16 *>(ws + Lw.H2);
    A.H3 = reinterpret_cast<__bf16 *>(ws + Lw.H3);
    A.D1 = reinterpret_cast<__bf16 *>(ws + Lw.D1);
    A.D2 = reinterpret_cast<__bf16 *>(ws + Lw.D2);
    A.D3 = reinterpret_cast<__bf16 *>(ws + Lw.D3);
    A.D4 = reinterpret_cast<__bf16 *>(ws + Lw.D4);
    int64_t blocks = (Lw.Gp + 32 * SNT * 4 - 1) / (32 * SNT * 4);
    if (blocks > ctx->num_cus) blocks = ctx->num_cus;
    hipLaunchKernelGGL(k_smooth_fwd_bwd, dim3((unsigned)blocks), dim3(256), 0, s, A);
    // one workgroup per CU over the three kinds
    int64_t gx = (Lw.Gp / 16 + 3) / 4;
    if (gx > ctx->num_cus / 3) gx = ctx->num_cus / 3 > 0 ? ctx->num_cus / 3 : 1;
    const dim3 gw((unsigned)gx, 3);
    hipLaunchKernelGGL(k_smooth_wgrad, gw, dim3(256), 0, s, A, grad);
    LEGS_CHECK_LAUNCH(ctx);
    return LEGS_OK;
}
