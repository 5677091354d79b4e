// Loss gradient of the full training step (gfx950): per view, the mean
// absolute error of the RGB and semantic channels against seeded targets plus
// lambda_u times the mean rendered uncertainty (Sec. 3.4.2 Eq. 11 regulariser
// L_u = sum R_u / (H W)). Writes dL/d(out) for every element and accumulates
// the loss value; one pass over out and target (HBM-bound).
#include "legs_internal.h"

namespace {

__device__ __forceinline__ float l1_grad(float d, float inv, float &lsum)
{
    lsum = fmaf(fabsf(d), inv, lsum);
    return d > 0.0f ? inv : (d < 0.0f ? -inv : 0.0f);
}

// Bound by HBM. Two workgroups of 1024 threads per CU, as many as run at once:
// each adds to the one loss, and 4,096 of 256 threads spent 45 us on that address
// in one view of 800 x 450 with 12 channels (66 us, 22 here) and rounded the loss
// eight times as often. They take pieces of the concatenated planes in turn, so a
// launch is as even with uneven views as with equal ones: with the workgroups
// divided among the planes instead, 16 views of 640 x 480 to 1920 x 1080 with 20
// channels took 979 us, here 632, and 15 of 160 x 120 beside one of 1920 x 1080
// 484, here 119. Pieces of 128 KB: of 16 KB, finding the plane shows (6 % on four
// 1920 x 1080 views), and one piece per workgroup leaves them reading in step, far
// apart (3 %). Four 1920 x 1080 views with 20 channels: 372 us, 5.3 TB/s.
constexpr int L1_THREADS = 1024;
constexpr int L1_STEP = 4 * L1_THREADS;          // elements of one float4 per thread
constexpr int L1_PIECE = 8 * L1_STEP;

// One part [e0, e1) of a (view, channel) plane, so that the weight and the kind
// of term are wave-uniform: four neighbouring elements per step between the first
// and the last multiple of four where the three buffers are 16-byte aligned (vec),
// one at a time otherwise and at the ends.
template <bool FIT>
__device__ __forceinline__ void l1_part(const float *__restrict__ out, const float *__restrict__ tgt,
                                        float *__restrict__ d_out, int64_t e0, int64_t e1, int vec, float inv,
                                        float &lsum)
{
    int64_t q0 = (e0 + 3) / 4, q1 = e1 / 4;
    if (!vec || q0 > q1) q0 = q1 = (e0 + 3) / 4;
    const auto one = [&](int64_t i) {
        if constexpr (FIT) {
            d_out[i] = l1_grad(out[i] - tgt[i], inv, lsum);
        } else {
            lsum = fmaf(out[i], inv, lsum);
            d_out[i] = inv;
        }
    };
    for (int64_t q = q0 + threadIdx.x; q < q1; q += L1_THREADS) {
        const float4 a = reinterpret_cast<const float4 *>(out)[q];
        float4 r;
        if constexpr (FIT) {
            const float4 b = reinterpret_cast<const float4 *>(tgt)[q];
            r.x = l1_grad(a.x - b.x, inv, lsum);
            r.y = l1_grad(a.y - b.y, inv, lsum);
            r.z = l1_grad(a.z - b.z, inv, lsum);
            r.w = l1_grad(a.w - b.w, inv, lsum);
        } else {
            lsum = fmaf(a.x, inv, lsum);
            lsum = fmaf(a.y, inv, lsum);
            lsum = fmaf(a.z, inv, lsum);
            lsum = fmaf(a.w, inv, lsum);
            r = make_float4(inv, inv, inv, inv);
        }
        reinterpret_cast<float4 *>(d_out)[q] = r;
    }
    const int64_t head = min(4 * q0, e1), tail = max(4 * q1, head);
    for (int64_t i = e0 + threadIdx.x; i < head; i += L1_THREADS) one(i);
    for (int64_t i = tail + threadIdx.x; i < e1; i += L1_THREADS) one(i);
}

// Pieces of `per` elements of the planes of all views, one after the other in
// memory, dealt to the workgroups in turn; a piece may span planes and views.
__global__ void __launch_bounds__(L1_THREADS)
k_l1(const float *__restrict__ out, const float *__restrict__ tgt, const legs_view *__restrict__ views,
     int n_views, int64_t per, int C, int n_fit, float lambda_u, int vec, float *__restrict__ d_out,
     float *__restrict__ loss)
{
    float lsum = 0.0f;
    const legs_view &z = views[n_views - 1];
    const int64_t all = C * (z.pixel_offset + (int64_t)z.cam.width * z.cam.height);
    for (int64_t e = C * views[0].pixel_offset + per * blockIdx.x; e < all; e += per * gridDim.x) {
        const int64_t end = min(e + per, all);
        int v = 0;                               // the last view that starts at or before e
        for (int lo = 1, hi = n_views - 1; lo <= hi;) {
            const int mid = (lo + hi) / 2;
            if ((int64_t)C * views[mid].pixel_offset <= e) {
                v = mid;
                lo = mid + 1;
            } else {
                hi = mid - 1;
            }
        }
        for (int64_t at = e; at < end && v < n_views; ++v) {
            const int64_t hw = (int64_t)views[v].cam.width * views[v].cam.height;
            const int64_t first = (int64_t)C * views[v].pixel_offset;
            for (int c = (int)((at - first) / hw); c < C && at < end; ++c) {
                const int64_t to = min(first + (c + 1) * hw, end);
                if (c < n_fit)     // mean absolute error of a fitted channel
                    l1_part<true>(out, tgt, d_out, at, to, vec, 1.0f / (float)((int64_t)n_fit * hw), lsum);
                else               // lambda_u times the mean rendered uncertainty
                    l1_part<false>(out, tgt, d_out, at, to, vec, lambda_u / (float)hw, lsum);
                at = to;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off, LEGS_WAVE);
    __shared__ float s_w[L1_THREADS / LEGS_WAVE];
    if (legs_lane() == 0) s_w[threadIdx.x / LEGS_WAVE] = lsum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < L1_THREADS / LEGS_WAVE; ++w) t += s_w[w];
        atomicAdd(loss, (float)t);
    }
}

__global__ void k_zero1(float *p) { *p = 0.0f; }

// Zero n 32-bit words (16-byte stores where aligned; a kernel, so it records
// as a kernel node under graph capture).
__global__ void __launch_bounds__(256)
k_clear(uint32_t *__restrict__ p, int64_t n)
{
    const int64_t n4 = (reinterpret_cast<uintptr_t>(p) & 15) == 0 ? n / 4 : 0;
    uint4 *q = reinterpret_cast<uint4 *>(p);
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) q[i] = make_uint4(0, 0, 0, 0);
    for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) p[i] = 0u;
}

} // namespace

int32_t legs_launch_clear(legs_ctx *ctx, void *dev, int64_t words, hipStream_t s)
{
    if (words <= 0) return LEGS_OK;
    int64_t g = (words / 4 + 255) / 256;
    const int64_t cap = (int64_t)ctx->num_cus * 8;
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)g), dim3(256), 0, s, static_cast<uint32_t *>(dev), words);
    LEGS_CHECK_LAUNCH(ctx);
    return LEGS_OK;
}

int32_t legs_launch_l1_loss_grad(legs_ctx *ctx, const float *out, const float *target,
                                 const legs_view *views, int32_t n_views, int64_t total_pixels,
                                 int32_t C, int32_t n_fit, float lambda_u, float *d_out,
                                 float *loss, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero1, dim3(1), dim3(1), 0, s, loss);
    const int64_t total = (int64_t)C * total_pixels;
    if (total > 0 && n_views > 0 && C > 0) {
        const int64_t most = (int64_t)ctx->num_cus * 2;
        int64_t per = ((total + most - 1) / most + L1_STEP - 1) / L1_STEP * L1_STEP;
        if (per > L1_PIECE) per = L1_PIECE;
        const int64_t pieces = (total + per - 1) / per;
        const int vec = ((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(target) |
                          reinterpret_cast<uintptr_t>(d_out)) & 15) == 0;
        hipLaunchKernelGGL(k_l1, dim3((unsigned)(pieces < most ? pieces : most)), dim3(L1_THREADS), 0, s, out, target, views,
                           n_views, per, C, n_fit, lambda_u, vec, d_out, loss);
    }
    LEGS_CHECK_LAUNCH(ctx);
    return LEGS_OK;
}
