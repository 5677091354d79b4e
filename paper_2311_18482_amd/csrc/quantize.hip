// Quantisation of hybrid language features into the discrete feature space
// (Sec. 3.3, Eqs. 4-7, and the supplementary load-balancing loss), gfx950.
//
// Features F [K][d] are IEEE half (CLIP dimensions [0, d_clip), DINO the
// rest), the feature space S [N][d] float32, rounded to half for every use
// (dot products and norms), so the cosines are those of the half-precision
// vectors; products are exact in float32 and accumulate in float32 on
// v_mfma_f32_32x32x16_f16.
//
//  k_quant_prep      S once per call into the LDS image of each 128-dimension
//                    chunk (A-operand fragments, code rows x dimensions),
//                    1 / |S_j| of both parts, and the sums and the gradient
//                    cleared.
//  k_quant_pass      one workgroup of 8 waves per CU, 32 features per wave: the
//                    codebook image of each 128-dimension chunk streams into
//                    one of two LDS buffers (global_load_lds, no registers) and
//                    each wave's feature fragments into registers one chunk
//                    ahead, across the rounds as well, so that loads are in
//                    flight during the softmax. The 32 x N dot products of a
//                    wave stay in registers (transposed: codes x features); at
//                    the end of the CLIP part they become its cosines. The
//                    feature norms are summed from the same fragments. Then per
//                    feature the distance D_j = cos^C_j + lambda cos^D_j, its
//                    argmax (first maximum) and its softmax: index, histogram
//                    of the indices, sum of the softmax (the mean selection
//                    probability), cosine loss and, for the gradient, 1 / |F_i|
//                    and the cosines of both parts in register order (1 KB
//                    contiguous per store).
//                    Bound by memory latency (one 8 KB chunk in flight per
//                    wave; two need 30 registers more than there are and
//                    spill, 1.36 ms a call instead of 1.21). 1M features x 896
//                    dimensions at N = 128: 640 us with the cosines' 1 GB,
//                    where four waves of 32 features with the features through
//                    LDS too and a drain per round took 695 without them.
//  k_quant_weights   dL_q/dD_ij with the final histogram from the stored
//                    cosines, in place, as half weights (scaled by 2^10 K) in
//                    the weight gradient's MFMA operand order (one 16-byte
//                    fragment per lane after an 8 x 8 lane transpose), and the
//                    sums over i of dL/dD_ij cos_ij. Reading 1 GB back takes
//                    274 us where a second pass over the features took 876.
//  k_quant_wgrad     sum_i W_ij F_ic / |F_i| for every code j and dimension c:
//                    FP16 MFMA with the features as the contraction (the
//                    weight fragments 1 KB contiguous per wave), the unit
//                    feature rows staged through LDS transposed
//                    (dimension-major) in steps of 64, split over feature
//                    ranges (x) and groups of two 128-dimension chunks (y: the
//                    weights are read once per group), float atomics into the
//                    gradient. Two workgroups per CU, one round of them: 632 us
//                    at the size above, with its weights of both parts and a
//                    chunk per group 660; one workgroup per CU makes the call
//                    35 % slower, four 9 %, one chunk per group 19 %.
//  k_quant_finish    the column-sum term, the losses, r and p.
#include <algorithm>

#include "legs_internal.h"
#include "legs_decode_internal.h"
#include "wave_reduce.h"
#include "lane_transpose.h"

namespace {

typedef legs_f32x16 f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

constexpr int QCH = 128;           // dimensions per chunk
// The gradient's half weights are 2^10 K dL/dD (at most 2^10 (lambda_cos +
// lambda_lb) in magnitude): the scale keeps the small terms of the
// load-balancing loss out of the half-precision subnormal range.
constexpr float WSCALE = 1024.0f;
constexpr int QTHREADS = 512;      // 8 waves, two per SIMD
constexpr int QGROUP = 256;        // features per workgroup round (the cosines and weights are padded to it)
static_assert(QTHREADS / LEGS_WAVE * 32 == QGROUP, "a workgroup's round is one padding group");

// s_waitcnt vmcnt(N) (expcnt and lgkmcnt not waited for).
template <int N>
__device__ __forceinline__ void vm_wait()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Workgroup barrier for the double-buffered chunks: this wave's LDS reads
// are complete (lgkmcnt 0) and the compiler keeps memory operations on their
// side of it, but the next chunk's loads in flight are not waited for (the
// fence of a __syncthreads() would wait for every load). Each wave waits for
// its own loads of a buffer (vm_wait) before the barrier that precedes the
// buffer's reads.
__device__ __forceinline__ void ring_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0); vmcnt, expcnt not waited for
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// 16 bytes per lane from global memory straight into LDS (gfx950
// global_load_lds_dwordx4): lane l's bytes land at lds + 16 l; lds is the
// same for the whole wave. Completion: s_waitcnt vmcnt(0) of this wave, then
// a barrier for the other waves' reads.
__device__ __forceinline__ void global_to_lds(const void *src, void *lds)
{
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}

// Two floats as a word of halves (round to nearest), a in the low half.
__device__ __forceinline__ uint32_t pack_half2(float a, float b)
{
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
    const f16x2 v = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ f32x16 mfma16(f16x8 a, f16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Image of chunk ch: fragment (mb, ks, lane) holds code 32 mb + lane % 32,
// dimensions 128 ch + 16 ks + 8 (lane / 32) + [0, 8).
template <int KB>
__global__ void __launch_bounds__(256)
k_quant_prep(const float *__restrict__ S, int d, int dC, f16x8 *__restrict__ img, float *__restrict__ invS,
             uint32_t *__restrict__ counts, uint32_t *__restrict__ sums, int nsums, float *__restrict__ grad)
{
    constexpr int NF = KB * 8 * 64;
    const int nch = d / QCH;
    const int t0 = blockIdx.x * 256 + threadIdx.x;
    for (int q = t0; q < 32 * KB; q += gridDim.x * 256) counts[q] = 0u;
    for (int q = t0; q < nsums; q += gridDim.x * 256) sums[q] = 0u;
    if (grad)
        for (int q = t0; q < 32 * KB * d; q += gridDim.x * 256) grad[q] = 0.0f;
    for (int q = blockIdx.x * 256 + threadIdx.x; q < nch * NF; q += gridDim.x * 256) {
        const int ch = q / NF, f = q % NF;
        const int l = f & 63, ks = (f >> 6) & 7, mb = f >> 9;
        const float *row = S + (int64_t)(32 * mb + (l & 31)) * d + ch * QCH + 16 * ks + 8 * (l >> 5);
        f16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (_Float16)row[e];
        img[q] = v;
    }
    // 1 / |S_j| per part (0 for a zero part): one wave per code
    constexpr int N = 32 * KB;
    const int wave = (blockIdx.x * 256 + threadIdx.x) / LEGS_WAVE, lane = __lane_id();
    for (int j = wave; j < N; j += gridDim.x * 4) {
        float sc = 0.0f, sd = 0.0f;
        for (int c = lane; c < d; c += LEGS_WAVE) {
            const float v = (float)(_Float16)S[(int64_t)j * d + c];
            if (c < dC) sc = fmaf(v, v, sc);
            else sd = fmaf(v, v, sd);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            sc += __shfl_xor(sc, o, LEGS_WAVE);
            sd += __shfl_xor(sd, o, LEGS_WAVE);
        }
        if (lane == 0) {
            invS[j] = sc > 0.0f ? 1.0f / sqrtf(sc) : 0.0f;
            invS[N + j] = sd > 0.0f ? 1.0f / sqrtf(sd) : 0.0f;
        }
    }
}

struct QuantArgs {
    const _Float16 *F;
    int64_t K, Kp;              // the launch's features, and padded to whole rounds
    int64_t Kall;               // the call's
    int d, dC;
    const f16x8 *img;
    const float *invS;          // [2][N]
    float lam_d, lam_cos, lam_lb;
    int32_t *index;             // [K]
    uint32_t *counts;           // [N]
    float *psum;                // [N] sum of softmax over features
    double *lsum;               // [1] cosine-loss sum
    f32x4 *cos;                 // [Kp / 32][2 parts][N / 8][64 lanes] cosines (codes 8 q + 4 h .. + 3 of feature l % 32)
    float *invF;                // [2][Kp] 1 / |F_i| of both parts (0 past K)
    float *col;                 // [2][N] sum_i dL/dD_ij cos_ij (lambda dL/dD for DINO)
};

// Half weights 2^10 K dL/dD of the 32 features from i (a multiple of 32) in
// the place of their cosines: the first quarter of it, in MFMA operand order
// (legs_lt::frag_at, codes as rows, features as columns).
__device__ __forceinline__ _Float16 *quant_weights(void *cos, int N, int64_t i)
{
    return reinterpret_cast<_Float16 *>(static_cast<char *>(cos) + (i >> 5) * (256 * (int64_t)N));
}

// Adds the sums of v over the 32 features of each lane half to this lane's
// shares: legs_tr::final_k slots, one code each (src_index names it).
template <int V>
__device__ __forceinline__ void half_wave_sums(float (&v)[V], float (&sum)[legs_tr::final_k(V, 5)], int lane)
{
    legs_tr::run<4, V, V>(v, lane);
#pragma unroll
    for (int k = 0; k < legs_tr::final_k(V, 5); ++k) sum[k] += v[k];
}

// A workgroup's shares of half_wave_sums, wave after wave, into dst (LDS; code
// order). Plain reads and writes: LDS float atomics take hundreds of cycles.
template <int V, int WAVES>
__device__ __forceinline__ void block_sums(const float (&sum)[legs_tr::final_k(V, 5)], float *dst, int lane, int wave)
{
    for (int w = 0; w < WAVES; ++w) {
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int k = 0; k < legs_tr::final_k(V, 5); ++k) {
                const int ix = legs_tr::src_index<4, V>(k, lane);
                if (ix < 0) continue;
                const int j = 32 * (ix >> 4) + legs_drow(ix & 15, lane >> 5);
                dst[j] = w == 0 ? sum[k] : dst[j] + sum[k];
            }
        }
    }
    __syncthreads();
}

template <int KB, bool KEEP>
__global__ void __launch_bounds__(QTHREADS)
k_quant_pass(QuantArgs A)
{
    constexpr int N = 32 * KB, NF = KB * 8 * 64;
    // two LDS buffers for the codebook image of a chunk; distinct arrays, so that
    // the compiler can tell the reads of one from the loads landing in the other
    __shared__ f16x8 frag0[NF], frag1[NF];
    __shared__ float s_inv[2][N];
    __shared__ uint32_t s_cnt[N];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int j = tid; j < N; j += QTHREADS) {
        s_inv[0][j] = A.invS[j];
        s_inv[1][j] = A.invS[N + j];
        s_cnt[j] = 0u;
    }
    float lcos = 0.0f;
    float psum[legs_tr::final_k(KB * 16, 5)] = {};
    const int nch = A.d / QCH, nchC = A.dC / QCH;
    const int64_t groups = A.Kp / QGROUP;   // (every column of invF below Kp is written)
    auto issue = [&](int ch, f16x8 *fg) {    // codebook image of chunk ch, 1 KB pieces over the waves
        for (int p = wave; p < NF / LEGS_WAVE; p += QTHREADS / LEGS_WAVE)
            global_to_lds(A.img + (int64_t)ch * NF + p * LEGS_WAVE + lane, fg + p * LEGS_WAVE);
    };
    // nothing requested later moves above the codebook pieces (the waits count)
    auto issue_end = [] {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // this lane's feature of round g; rows past K read row K - 1
    auto row_of = [&](int64_t g) {
        const int64_t i = g * QGROUP + wave * 32 + (lane & 31);
        return A.F + (i < A.K ? i : A.K - 1) * (int64_t)A.d + 8 * h;
    };
    f16x8 fb[8];                             // feature fragments of the next chunk, a k-step each
    const _Float16 *row = nullptr;
    if ((int64_t)blockIdx.x < groups) {
        row = row_of(blockIdx.x);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) fb[ks] = *reinterpret_cast<const f16x8 *>(row + 16 * ks);
        issue(0, frag0);
    }
    vm_wait<0>();
    __syncthreads();
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
        const int64_t gn = g + gridDim.x < groups ? g + gridDim.x : g;   // the round after (or this one again)
        const _Float16 *nrow = row_of(gn);
        f32x16 acc[KB], D[KB];
        float ss = 0.0f, inv0 = 0.0f;
#pragma unroll
        for (int mb = 0; mb < KB; ++mb) {
            acc[mb] = (f32x16){};
            D[mb] = (f32x16){};
        }
        auto norm = [&]() {                  // 1 / |F_i| of the part just summed
            const float s2 = ss + __shfl_xor(ss, 32, LEGS_WAVE);
            return s2 > 0.0f ? 1.0f / sqrtf(s2) : 0.0f;
        };
        // the CLIP dot products become cosines at the end of the part
        auto part_end = [&]() {
            inv0 = norm();
            ss = 0.0f;
#pragma unroll
            for (int mb = 0; mb < KB; ++mb) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    D[mb][r] = acc[mb][r] * inv0 * s_inv[0][32 * mb + legs_drow(r, h)];
                acc[mb] = (f32x16){};
            }
        };
        auto chunk = [&](const f16x8 *fr, int ch) {
            // the fragments of k-step ks + 1 are read while the MFMAs of ks run, and
            // the next chunk's feature fragments are requested in their place
            f16x8 a[KB];
#pragma unroll
            for (int mb = 0; mb < KB; ++mb) a[mb] = fr[mb * 8 * 64 + lane];
            const _Float16 *src = ch + 1 == nch ? nrow : row + (ch + 1) * QCH;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                f16x8 an[KB];
                if (ks + 1 < 8) {
#pragma unroll
                    for (int mb = 0; mb < KB; ++mb) an[mb] = fr[(mb * 8 + ks + 1) * 64 + lane];
                }
                const f16x8 b = fb[ks];
#pragma unroll
                for (int mb = 0; mb < KB; ++mb) acc[mb] = mfma16(a[mb], b, acc[mb]);
#pragma unroll
                for (int e = 0; e < 8; ++e) ss = fmaf((float)b[e], (float)b[e], ss);
                // a row's 128-byte line at a time: spread over the steps, the line
                // left the L1 between them (1.28 ms a call instead of 1.21)
                if ((ks & 3) == 3) {
#pragma unroll
                    for (int k = ks - 3; k <= ks; ++k) fb[k] = *reinterpret_cast<const f16x8 *>(src + 16 * k);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (ks + 1 < 8) {
#pragma unroll
                    for (int mb = 0; mb < KB; ++mb) a[mb] = an[mb];
                }
            }
        };
        // Chunk ch + 1's codebook loads while chunk ch computes. The waits count
        // what was requested after the codebook pieces that they wait for: the 8
        // feature fragments of the chunk before, or, at a round's start, the
        // cosines' stores (without them, whatever there is; the first round's
        // loads were waited for above).
        constexpr int FL = 8, ST = KEEP ? 8 * KB : 0;
#pragma unroll 1
        for (int ch = 0; ch < nch; ch += 2) {
            if (ch == nchC) part_end();
            if (ch) vm_wait<FL>();
            else vm_wait<ST>();
            ring_barrier();
            if (ch + 1 < nch) issue(ch + 1, frag1);
            issue_end();
            chunk(frag0, ch);
            if (ch + 1 < nch) {
                if (ch + 1 == nchC) part_end();
                vm_wait<FL>();
                ring_barrier();
                if (ch + 2 < nch) issue(ch + 2, frag0);
                issue_end();
                chunk(frag1, ch + 1);
            }
        }
        if (nchC == nch) part_end();         // no DINO chunks: their dot products are zero
        ring_barrier();                      // every wave is done with the codebook buffers
        issue(0, frag0);                     // the next round's first chunk, during the softmax
        issue_end();
        float sv[KB * 16];
        {
            const int64_t i = g * QGROUP + wave * 32 + (lane & 31);
            const bool vt = i < A.K;
            const float inv1 = nchC == nch ? 0.0f : norm();
            if (KEEP && h == 0) {
                A.invF[i] = vt ? inv0 : 0.0f;
                A.invF[A.Kp + i] = vt ? inv1 : 0.0f;
            }
            // distance, argmax (first maximum)
            float best = -INFINITY;
            int bidx = 0x7fffffff;
            f32x4 *pc = KEEP ? A.cos + (i >> 5) * (N / 4 * LEGS_WAVE) + lane : nullptr;
#pragma unroll
            for (int mb = 0; mb < KB; ++mb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 e;
                    const f32x4 c = {D[mb][4 * q], D[mb][4 * q + 1], D[mb][4 * q + 2], D[mb][4 * q + 3]};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int r = 4 * q + u;
                        e[u] = acc[mb][r] * inv1 * s_inv[1][32 * mb + legs_drow(r, h)];
                        const float Dv = D[mb][r] + A.lam_d * e[u];
                        D[mb][r] = Dv;
                        // (the half's offset 4 h, the same for every code, is added below)
                        if (Dv > best) { best = Dv; bidx = 32 * mb + legs_drow(r, 0); }
                    }
                    if (KEEP) {              // past the caches: a call's cosines outgrow them
                        __builtin_nontemporal_store(c, pc + (4 * mb + q) * LEGS_WAVE);
                        __builtin_nontemporal_store(e, pc + (N / 8 + 4 * mb + q) * LEGS_WAVE);
                    }
                }
            if (best > -INFINITY) bidx += 4 * h;
            {
                const float ob = __shfl_xor(best, 32, LEGS_WAVE);
                const int oi = __shfl_xor(bidx, 32, LEGS_WAVE);
                if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
                if (bidx >= N) bidx = 0;                  // no comparison held (NaN input)
            }
            float sum = 0.0f;
#pragma unroll
            for (int mb = 0; mb < KB; ++mb) {
#pragma unroll
                for (int r = 0; r < 16; ++r) D[mb][r] = __expf(D[mb][r] - best);
#pragma unroll
                for (int r = 0; r < 16; ++r) sum += D[mb][r];
            }
            sum += __shfl_xor(sum, 32, LEGS_WAVE);
            const float isum = 1.0f / sum;
#pragma unroll
            for (int mb = 0; mb < KB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) sv[16 * mb + r] = vt ? D[mb][r] * isum : 0.0f;
            // the cosine loss of the assigned code: (1 - cos^C) + lambda (1 - cos^D)
            // = (1 + lambda) - D at the maximum, which is best
            if (vt && h == 0) {
                lcos += (1.0f + A.lam_d) - best;
                A.index[i] = bidx;
                atomicAdd(&s_cnt[bidx], 1u);
            }
        }
        half_wave_sums(sv, psum, lane);
        row = nrow;
    }
    // the workgroup's sums (the softmax's in the codebook's place)
    vm_wait<0>();                            // the loads of the round that does not come
    float *s_p = reinterpret_cast<float *>(frag1);
    block_sums<KB * 16, QTHREADS / LEGS_WAVE>(psum, s_p, lane, wave);
    // (one addition per workgroup to the one loss, in float64)
    __shared__ double s_loss[QTHREADS / LEGS_WAVE];
    double lsum = lcos;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, LEGS_WAVE);
    if (lane == 0) s_loss[wave] = lsum;
    __syncthreads();
    if (tid == 0) {
        lsum = 0.0;
        for (int w = 0; w < QTHREADS / LEGS_WAVE; ++w) lsum += s_loss[w];
        if (lsum != 0.0) atomicAdd(A.lsum, lsum);
    }
    for (int j = tid; j < N; j += QTHREADS) {
        if (s_p[j] != 0.0f) atomicAdd(A.psum + j, s_p[j]);
        if (s_cnt[j]) atomicAdd(A.counts + j, s_cnt[j]);
    }
}

// dL_q/dD of 32 features per wave from their cosines, as half weights in their
// place (a wave reads its 256 N bytes before it writes the first quarter of
// them), and the sums over the features of its products with the cosines.
// Bound by memory: 10 N bytes a feature. (At N = 128 a lane's 128 cosines and their
// sums take all 256 registers and 13 more values are spilled.)
template <int KB>
__global__ void __launch_bounds__(256, 2)
k_quant_weights(QuantArgs A)
{
    constexpr int N = 32 * KB;
    __shared__ float s_r[N], s_col[2][N];
    const int lane = __lane_id(), h = lane >> 5;
    const int wave = threadIdx.x / LEGS_WAVE;
    const int i8 = lane & 7;
    const bool b1 = (lane & 2) != 0;
    const uint32_t psel = (lane & 1) ? 0x03020706u : 0x05040100u;
    const float invK = 1.0f / (float)A.Kall;
    for (int j = threadIdx.x; j < N; j += 256) s_r[j] = (float)A.counts[j] * invK;
    __syncthreads();
    const float scale = (float)A.Kall * WSCALE;
    float col[2][legs_tr::final_k(KB * 16, 5)] = {};
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wave; tile < A.Kp / 32; tile += (int64_t)gridDim.x * 4) {
        const int64_t i = 32 * tile + (lane & 31);
        const bool vt = i < A.K;
        const f32x4 *pc = A.cos + tile * (N / 4 * LEGS_WAVE) + lane;
        float c[KB * 16], e[KB * 16];
#pragma unroll
        for (int k = 0; k < KB * 4; ++k) {
            const f32x4 x = __builtin_nontemporal_load(pc + k * LEGS_WAVE);
            const f32x4 y = __builtin_nontemporal_load(pc + (N / 8 + k) * LEGS_WAVE);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[4 * k + u] = x[u];
                e[4 * k + u] = y[u];
            }
        }
        const int m = vt ? A.index[i] : -1;
        float best = -INFINITY, sum = 0.0f, rs = 0.0f;
#pragma unroll
        for (int k = 0; k < KB * 16; ++k) best = fmaxf(best, c[k] + A.lam_d * e[k]);
        best = fmaxf(best, __shfl_xor(best, 32, LEGS_WAVE));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < KB * 16; ++k) {
            const float x = __expf(c[k] + A.lam_d * e[k] - best);
            sum += x;
            rs += s_r[8 * (k >> 2) + 4 * h + (k & 3)] * x;
        }
        sum += __shfl_xor(sum, 32, LEGS_WAVE);
        rs += __shfl_xor(rs, 32, LEGS_WAVE);
        const float isum = 1.0f / sum;
        rs *= isum;
        __builtin_amdgcn_sched_barrier(0);
        // the 8 codes r = 8 k .. 8 k + 7 of block mb of this lane's feature,
        // transposed across its group of 8 lanes (8 consecutive features), are one
        // 16-byte fragment per lane
        _Float16 *W = quant_weights(A.cos, N, 32 * tile);
#pragma unroll
        for (int mb = 0; mb < KB; ++mb)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float gv[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int r = 8 * k + 2 * q + u, x = 16 * mb + r;
                        const float sm = __expf(c[x] + A.lam_d * e[x] - best) * isum;
                        float gj = A.lam_lb * invK * sm * (s_r[32 * mb + legs_drow(r, h)] - rs);
                        if (32 * mb + legs_drow(r, 0) == m - 4 * h) gj -= A.lam_cos * invK;
                        if (!vt) gj = 0.0f;
                        c[x] *= gj;                        // column-sum terms, in place
                        e[x] *= A.lam_d * gj;
                        gv[u] = gj;
                    }
                    w[q] = pack_half2(scale * gv[0], scale * gv[1]);
                }
                legs_lt::oct_transpose(w, b1, psel);
                // lane i8 now holds code 32 mb + drow(8 k + i8, h) of its group's 8 features
                const int row = 32 * mb + 16 * k + 8 * (i8 >> 2) + 4 * h + (i8 & 3);
                *reinterpret_cast<uint4 *>(W + legs_lt::frag_at((lane & 31) - i8, N, row)) =
                    make_uint4(w[0], w[1], w[2], w[3]);
                __builtin_amdgcn_sched_barrier(0);
            }
        half_wave_sums(c, col[0], lane);
        __builtin_amdgcn_sched_barrier(0);
        half_wave_sums(e, col[1], lane);
    }
    block_sums<KB * 16, 4>(col[0], s_col[0], lane, wave);
    block_sums<KB * 16, 4>(col[1], s_col[1], lane, wave);
    for (int j = threadIdx.x; j < 2 * N; j += 256)
        if ((&s_col[0][0])[j] != 0.0f) atomicAdd(A.col + j, (&s_col[0][0])[j]);
}

// sum_i W_ij F_ic over the features [x0, x1) of this workgroup, for the NC
// 128-dimension chunks from NC blockIdx.y; wave w computes code block w % KB
// and, of each chunk, 4 / (4 / KB) dimension blocks.
constexpr int WG_FEAT = 64;          // features per LDS step

template <int KB, int NC>
__global__ void __launch_bounds__(256, 2)
k_quant_wgrad(const _Float16 *__restrict__ F, int64_t K, int64_t Kp, int64_t Kall, int d, int dC, int64_t per_block,
              const void *__restrict__ weights, const float *__restrict__ invF, const float *__restrict__ invS,
              float lam_d, float *__restrict__ grad)
{
    constexpr int N = 32 * KB, WPB = 4 / KB, DB = 4 / WPB;   // waves per code block, dim blocks per wave
    __shared__ f16x8 tile[NC][WG_FEAT / 16][QCH / 32][64];   // B fragments of a step: [chunk][k-step][dim block][lane]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5;
    const int i8 = lane & 7;
    const bool b1 = (lane & 2) != 0;
    const uint32_t psel = (lane & 1) ? 0x03020706u : 0x05040100u;
    const int mb = wave % KB, db0 = (wave / KB) * DB;
    const int c0 = blockIdx.y * QCH * NC;
    const int nc = min(NC, d / QCH - (int)blockIdx.y * NC);
    const int64_t x0 = (int64_t)blockIdx.x * per_block;
    const int64_t x1 = min(x0 + per_block, Kp);
    f32x16 acc[NC][DB];
#pragma unroll
    for (int n = 0; n < NC; ++n)
#pragma unroll
        for (int q = 0; q < DB; ++q) acc[n][q] = (f32x16){};
    // the next step's feature rows, their norms and this wave's weight
    // fragments are loaded into registers while the current step computes
    f16x8 fv[NC][4], wa[WG_FEAT / 16];
    float fsc[NC][4];
    auto load_step = [&](int64_t s0) {
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            if (n >= nc) continue;
            const float *iF = invF + (c0 + n * QCH < dC ? 0 : Kp);
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int u = 4 * wave + it;
                const int64_t ii = s0 + 8 * (u >> 1) + i8;
                const int c8 = 64 * (u & 1) + 8 * (lane >> 3);
                fv[n][it] = ii < K ? *reinterpret_cast<const f16x8 *>(F + ii * d + c0 + n * QCH + c8) : (f16x8){};
                fsc[n][it] = ii < K ? iF[ii] : 0.0f;         // unit feature rows of this part
            }
        }
#pragma unroll
        for (int ks = 0; ks < WG_FEAT / 16; ++ks) {
            // operand order: the wave's fragments of (code block mb, features
            // s0 + 16 ks ..) are 1 KB contiguous
            const int64_t ia = s0 + 16 * ks;
            wa[ks] = ia < x1 ? *reinterpret_cast<const f16x8 *>(
                                   quant_weights(const_cast<void *>(weights), N, ia) +
                                   legs_lt::frag_at((ia & 31) + 8 * h, N, 32 * mb + (lane & 31)))
                             : (f16x8){};
        }
    };
    if (x0 < x1) load_step(x0);
    for (int64_t s0 = x0; s0 < x1; s0 += WG_FEAT) {
        ring_barrier();                                    // the previous step's readers are done
        // stage features [s0, s0 + 64) x dimensions [c0, c0 + 128 nc) as B
        // fragments: per chunk 16 units of 8 features x 64 dimensions, four per
        // wave; lane l holds dimensions 8 (l / 8) .. + 7 (of the unit's half) of
        // feature l % 8 (of the unit's block of 8), scales the row to unit
        // length, and the transpose across its group of 8 lanes leaves it
        // dimension 8 (l / 8) + l % 8 of the 8 features: one fragment
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            if (n >= nc) continue;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int u = 4 * wave + it, fb = u >> 1;
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    w[q] = pack_half2((float)fv[n][it][2 * q] * fsc[n][it], (float)fv[n][it][2 * q + 1] * fsc[n][it]);
                legs_lt::oct_transpose(w, b1, psel);
                const int c = 64 * (u & 1) + 8 * (lane >> 3) + i8;   // the dimension this lane now holds
                tile[n][fb >> 1][c >> 5][(c & 31) + 32 * (fb & 1)] =
                    __builtin_bit_cast(f16x8, make_uint4(w[0], w[1], w[2], w[3]));
            }
        }
        f16x8 a[WG_FEAT / 16];
#pragma unroll
        for (int ks = 0; ks < WG_FEAT / 16; ++ks) a[ks] = wa[ks];
        if (s0 + WG_FEAT < x1) load_step(s0 + WG_FEAT);
        ring_barrier();                                    // the staged fragments (LDS only: the
                                                           // loads just issued stay in flight)
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            if (n >= nc) continue;
#pragma unroll
            for (int ks = 0; ks < WG_FEAT / 16; ++ks)
#pragma unroll
                for (int q = 0; q < DB; ++q) {
                    const f16x8 b = tile[n][ks][db0 + q][lane];     // dimension 32 (db0 + q) + lane % 32
                    acc[n][q] = mfma16(a[ks], b, acc[n][q]);
                }
        }
    }
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        if (n >= nc) continue;
        const bool clip = c0 + n * QCH < dC;
        const float sc = (clip ? 1.0f : lam_d) / ((float)Kall * WSCALE);
        const float *is = invS + (clip ? 0 : N);
#pragma unroll
        for (int q = 0; q < DB; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = 32 * mb + legs_drow(r, h);
                const int c = c0 + n * QCH + 32 * (db0 + q) + (lane & 31);
                const float v = acc[n][q][r] * sc * is[j];
                if (v != 0.0f) atomicAdd(grad + (int64_t)j * d + c, v);
            }
    }
}

// grad[j][c] -= col^part_j S16_jc / |S16_j^part|^2; losses; r and p.
template <int KB>
__global__ void __launch_bounds__(256)
k_quant_finish(const float *__restrict__ S, int d, int dC, int64_t K, const float *__restrict__ invS,
               const float *__restrict__ col, float *__restrict__ grad, const uint32_t *__restrict__ counts,
               const float *__restrict__ psum, const double *__restrict__ lsum, float lam_cos, float lam_lb,
               float *__restrict__ prob_mean, float *__restrict__ losses)
{
    constexpr int N = 32 * KB;
    if (grad) {
        for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < (int64_t)N * d; q += (int64_t)gridDim.x * 256) {
            const int j = (int)(q / d), c = (int)(q % d);
            const int part = c >= dC;
            const float iv = invS[part * N + j];
            grad[q] -= col[part * N + j] * (float)(_Float16)S[q] * iv * iv;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < LEGS_WAVE) {
        const float invK = 1.0f / (float)K;
        float lb = 0.0f;
        for (int j = threadIdx.x; j < N; j += LEGS_WAVE) {
            const float p = psum[j] * invK;
            if (prob_mean) prob_mean[j] = p;
            lb += (float)counts[j] * invK * p;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) lb += __shfl_xor(lb, o, LEGS_WAVE);
        if (threadIdx.x == 0 && losses) {
            const float lc = (float)lsum[0] * invK;
            losses[0] = lc;
            losses[1] = lb;
            losses[2] = lam_cos * lc + lam_lb * lb;
        }
    }
}

// Features whose cosines a call keeps at once (a multiple of QGROUP; 4 GB at N =
// 128). A larger call with a gradient reads the features past the first so many
// once more, piece by piece, when the histogram is there, instead of asking for 8 N
// bytes for every one of them.
constexpr int64_t QKEEP = 1 << 22;
static_assert(QKEEP % QGROUP == 0, "pieces are whole rounds");

struct QuantLayout {
    int64_t img, invS, psum, col, lsum, spare, cos, invF, total, Kp;
};

QuantLayout quant_layout(int64_t K, int32_t N, int32_t d, bool grad)
{
    QuantLayout L;
    auto up = [](int64_t x) { return (x + 255) & ~(int64_t)255; };
    L.Kp = (std::min(K, QKEEP) + QGROUP - 1) / QGROUP * QGROUP;
    int64_t o = 0;
    L.img = o;  o = up(o + (int64_t)N * d * 2);
    L.invS = o; o = up(o + 2 * (int64_t)N * 4);
    L.psum = o; o = up(o + (int64_t)N * 4);
    L.col = o;  o = up(o + 2 * (int64_t)N * 4);
    L.lsum = o; o = up(o + 8);
    // the gradient's alone
    L.spare = o; o = up(o + (grad && K > QKEEP ? 8 + 2 * (int64_t)N * 4 : 0));
    L.cos = o;  o = up(o + (grad ? 2 * (int64_t)N * L.Kp * 4 : 0));
    L.invF = o; o = up(o + (grad ? 2 * L.Kp * 4 : 0));
    L.total = o;
    return L;
}

template <int KB>
void quantize_kernels(legs_ctx *ctx, const QuantArgs &all, const QuantLayout &Lw, char *ws, const float *S,
                      float *prob_mean, float *losses, float *grad, hipStream_t s)
{
    constexpr int N = 32 * KB;
    const int d = all.d, dC = all.dC;
    const int64_t cus = ctx->num_cus;
    // the features [i0, i0 + n) of the call
    const auto piece = [&](int64_t i0, int64_t n) {
        QuantArgs A = all;
        A.F += i0 * d;
        A.index += i0;
        A.K = n;
        A.Kp = (n + QGROUP - 1) / QGROUP * QGROUP;
        return A;
    };
    const auto pass = [&](const QuantArgs &A, bool keep) {
        const dim3 g((unsigned)std::min(A.Kp / QGROUP, cus));
        if (keep) hipLaunchKernelGGL((k_quant_pass<KB, true>), g, dim3(QTHREADS), 0, s, A);
        else hipLaunchKernelGGL((k_quant_pass<KB, false>), g, dim3(QTHREADS), 0, s, A);
    };
    // psum, col and lsum are contiguous (up to padding) in the workspace
    hipLaunchKernelGGL(k_quant_prep<KB>, dim3(64), dim3(256), 0, s, S, d, dC, reinterpret_cast<f16x8 *>(ws + Lw.img),
                       reinterpret_cast<float *>(ws + Lw.invS), all.counts,
                       reinterpret_cast<uint32_t *>(ws + Lw.psum), (int)((Lw.spare - Lw.psum) / 4), grad);
    if (!grad) pass(piece(0, all.K), false);
    else pass(piece(0, std::min(all.K, QKEEP)), true);
    if (grad && all.K > QKEEP) pass(piece(QKEEP, all.K - QKEEP), false);
    for (int64_t i0 = 0; grad && i0 < all.K; i0 += QKEEP) {
        const QuantArgs A = piece(i0, std::min(all.K - i0, QKEEP));
        if (i0 > 0) {                  // its cosines; the sums are in already
            QuantArgs again = A;
            again.lsum = reinterpret_cast<double *>(ws + Lw.spare);
            again.psum = reinterpret_cast<float *>(ws + Lw.spare + 8);
            again.counts = reinterpret_cast<uint32_t *>(again.psum + N);
            pass(again, true);
        }
        hipLaunchKernelGGL(k_quant_weights<KB>, dim3((unsigned)std::min((A.Kp / 32 + 3) / 4, cus * 8)), dim3(256), 0, s,
                           A);
        // feature ranges of the weight gradient, in steps of WG_FEAT: at most two
        // workgroups per CU over all of the dimension groups, so that all run at once
        // (rounded up instead, 515 of them at 1,280 dimensions left three for a
        // round of their own: 1M features x 128 codes 2,128 us, now 1,678)
        constexpr int NC = 2;
        const int64_t gy = (d / QCH + NC - 1) / NC, gx = std::max<int64_t>(2 * cus / gy, 1);
        const int64_t per_block =
            std::max<int64_t>(((A.Kp + gx - 1) / gx + WG_FEAT - 1) / WG_FEAT * WG_FEAT, 512);
        hipLaunchKernelGGL((k_quant_wgrad<KB, NC>), dim3((unsigned)((A.Kp + per_block - 1) / per_block), (unsigned)gy),
                           dim3(256), 0, s, A.F, A.K, A.Kp, A.Kall, d, dC, per_block, A.cos, A.invF, A.invS, A.lam_d,
                           grad);
    }
    const int64_t gz = ((int64_t)N * d + 255) / 256;
    hipLaunchKernelGGL(k_quant_finish<KB>, dim3((unsigned)(grad ? std::min<int64_t>(gz, 1024) : 1)), dim3(256), 0, s, S,
                       d, dC, all.K, all.invS, all.col, grad, all.counts, all.psum, all.lsum, all.lam_cos, all.lam_lb,
                       prob_mean, losses);
}

} // namespace

int64_t legs_quantize_workspace_bytes(int64_t K, int32_t N, int32_t d) { return quant_layout(K, N, d, true).total; }

int64_t legs_quantize_index_workspace_bytes(int64_t K, int32_t N, int32_t d)
{
    return quant_layout(K, N, d, false).total;
}

int32_t legs_launch_quantize(legs_ctx *ctx, const uint16_t *feat, int64_t K, int32_t d, int32_t dC,
                             const float *S, int32_t N, float lam_d, float lam_cos, float lam_lb,
                             void *workspace, int32_t *index, uint32_t *counts, float *prob_mean,
                             float *losses, float *grad, hipStream_t s)
{
    const QuantLayout Lw = quant_layout(K, N, d, grad != nullptr);
    char *ws = static_cast<char *>(workspace);
    QuantArgs A;
    A.F = reinterpret_cast<const _Float16 *>(feat);
    A.K = A.Kall = K;
    A.Kp = 0;                          // (set per launch)
    A.d = d;
    A.dC = dC;
    A.img = reinterpret_cast<const f16x8 *>(ws + Lw.img);
    A.invS = reinterpret_cast<const float *>(ws + Lw.invS);
    A.lam_d = lam_d;
    A.lam_cos = lam_cos;
    A.lam_lb = lam_lb;
    A.index = index;
    A.counts = counts;
    A.psum = reinterpret_cast<float *>(ws + Lw.psum);
    A.lsum = reinterpret_cast<double *>(ws + Lw.lsum);
    A.cos = reinterpret_cast<f32x4 *>(ws + Lw.cos);
    A.col = reinterpret_cast<float *>(ws + Lw.col);
    A.invF = reinterpret_cast<float *>(ws + Lw.invF);
    switch (N) {
    case 32: quantize_kernels<1>(ctx, A, Lw, ws, S, prob_mean, losses, grad, s); break;
    case 64: quantize_kernels<2>(ctx, A, Lw, ws, S, prob_mean, losses, grad, s); break;
    case 128: quantize_kernels<4>(ctx, A, Lw, ws, S, prob_mean, losses, grad, s); break;
    default: return legs_set_error(ctx, LEGS_ERR_ARG, "N must be 32, 64 or 128");
    }
    LEGS_CHECK_LAUNCH(ctx);
    return LEGS_OK;
}
