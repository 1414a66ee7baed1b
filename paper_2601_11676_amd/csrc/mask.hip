// Group mask (paper Sec. III-B.3): importance rank -> priority index -> device -> survivors.
// One workgroup per token; the work itself is in mask_device.hpp.
//
// mask_scores_kernel optionally computes the scores itself (second predictor layer,
// paper Sec. III-B.2, same fixed-order dot product as predictor.hip) so that the fused
// pass saves a launch; the arithmetic is shared, so the bits are the same.
#include "kernels.hpp"
#include "mask_device.hpp"

namespace halo {

constexpr int kMaskThreads = 1024;
constexpr int kOneLaunchRank = 128, kOneLaunchGroups = 128;

template <typename WT, bool FUSED_SCORES, int NT = kMaskThreads>
__global__ __launch_bounds__(NT) void mask_scores_kernel(
    const float *__restrict__ h, const WT *__restrict__ Bt, int r,      // FUSED_SCORES only
    float *__restrict__ scores, int G, int K, const int8_t *__restrict__ prio_dev, int n_dev,
    const uint8_t *__restrict__ drop, int32_t *__restrict__ order, int8_t *__restrict__ group_dev,
    uint8_t *__restrict__ mask, int32_t *__restrict__ surv_idx, int32_t *__restrict__ n_surv)
{
    __shared__ MaskShared sh;
    const size_t t = blockIdx.x;
    mask_scores_block<NT, WT, FUSED_SCORES>(
        sh, threadIdx.x, FUSED_SCORES ? h + t * r : nullptr, Bt, r, scores + t * G, G, K, prio_dev, n_dev,
        drop ? drop + t * n_dev : nullptr, order ? order + t * G : nullptr,
        group_dev ? group_dev + t * G : nullptr, mask + t * G, surv_idx ? surv_idx + t * K : nullptr,
        n_surv ? n_surv + t : nullptr);
}

// The whole prediction of a token in its workgroup: the first predictor layer too (same order, same bits), its results in LDS.
// A wave takes eight rows of At at a time, all requested together.
template <typename WT>
__device__ __forceinline__ void hidden_rows(const WT *__restrict__ x, const WT *__restrict__ At, int d, int r, int wave, int waves,
                                            int lane, float *h)
{
    constexpr int RB = 8;
    for (int j0 = wave * RB; j0 < r; j0 += waves * RB) {         // (r is a multiple of 8)
        float p[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) p[b] = 0.0f;
        for (int c = lane; c * 8 < d; c += kWave) {
            float xv[8];
            Piece8<WT> w[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) w[b].load(At + (size_t)(j0 + b) * d + c * 8);
            load8(x + c * 8, xv);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                float wv[8];
                w[b].get(wv);
#pragma unroll
                for (int e = 0; e < 8; ++e) p[b] = __builtin_fmaf(xv[e], wv[e], p[b]);
            }
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) p[b] = wave_sum(p[b]);
        if (lane == 0) {
#pragma unroll
            for (int b = 0; b < RB; ++b) h[j0 + b] = p[b] > 0.0f ? p[b] : 0.0f;
        }
    }
}

template <typename WT, int NT>
__global__ __launch_bounds__(NT) void predict_mask_kernel(
    const WT *__restrict__ x, const WT *__restrict__ At, int d, const WT *__restrict__ Bt, int r, float *__restrict__ scores,
    int G, int K, const int8_t *__restrict__ prio_dev, int n_dev, const uint8_t *__restrict__ drop, int32_t *__restrict__ order,
    int8_t *__restrict__ group_dev, uint8_t *__restrict__ mask, int32_t *__restrict__ surv_idx, int32_t *__restrict__ n_surv)
{
    __shared__ MaskShared sh;
    __shared__ __attribute__((aligned(16))) float h[kOneLaunchRank];
    const size_t t = blockIdx.x;
    hidden_rows(x + t * d, At, d, r, (int)(threadIdx.x >> 6), NT / kWave, (int)(threadIdx.x & 63), h);
    __syncthreads();
    mask_scores_block<NT, WT, true>(sh, threadIdx.x, h, Bt, r, scores + t * G, G, K, prio_dev, n_dev, drop ? drop + t * n_dev : nullptr,
                                    order ? order + t * G : nullptr, group_dev ? group_dev + t * G : nullptr, mask + t * G,
                                    surv_idx ? surv_idx + t * K : nullptr, n_surv ? n_surv + t : nullptr);
}

hipError_t launch_group_mask(const float *scores, int T, int G, int K, const int8_t *prio_dev,
                             int n_dev, const uint8_t *drop, int32_t *order, int8_t *group_dev,
                             uint8_t *mask, int32_t *surv_idx, int32_t *n_surv, hipStream_t s)
{
    mask_scores_kernel<float, false><<<dim3(T), dim3(kMaskThreads), 0, s>>>(
        nullptr, nullptr, 0, const_cast<float *>(scores), G, K, prio_dev, n_dev, drop, order,
        group_dev, mask, surv_idx, n_surv);
    return hipGetLastError();
}

// Threads of a token's workgroup where it computes the scores itself: as many waves as take all rows of Bt in one batch of
// eight slots each (two rows to a slot up to rank 256), at least two.  More only add to the barriers: 8 groups, rank 64 6.1 us with 1024
// threads, 5.4 with 512, 4.7 with 128; 27 groups, rank 512 5.9, 5.5 and (256) 5.4; with fewer the waves take turns: 92 groups,
// rank 64 6.5, 6.3, (256) 7.8; 138 groups, rank 256 6.6, 7.5.  With 64 tokens and more at most 512 for bf16, so that more workgroups
// share a compute unit (512 tokens of the 7B shape 11.5 us against 13.6 with 1024); float32 rows are twice the work of a wave (64 tokens,
// 200 groups, rank 512 19.8 us against 17.9 with 1024, both layers).
template <typename WT>
static int mask_threads(int T, int G, int r)
{
    const int slots = r <= 256 ? (G + 1) / 2 : G;
    const int threads = slots <= 16 ? 128 : slots <= 32 ? 256 : slots <= 64 ? 512 : kMaskThreads;
    return sizeof(WT) == 2 && T >= 64 && threads > 512 ? 512 : threads;
}

template <typename WT>
static void launch_fused(const float *h, const WT *Bt, int r, float *scores, int T, int G, int K, const int8_t *prio_dev,
                         int n_dev, const uint8_t *drop, int32_t *order, int8_t *group_dev, uint8_t *mask,
                         int32_t *surv_idx, int32_t *n_surv, hipStream_t s)
{
#define HALO_MASK_CASE(NT)                                                                                            \
    case NT:                                                                                                          \
        mask_scores_kernel<WT, true, NT><<<dim3(T), dim3(NT), 0, s>>>(h, Bt, r, scores, G, K, prio_dev, n_dev, drop,  \
                                                                      order, group_dev, mask, surv_idx, n_surv);      \
        break;
    switch (mask_threads<WT>(T, G, r)) {
        HALO_MASK_CASE(128)
        HALO_MASK_CASE(256)
        HALO_MASK_CASE(512)
        HALO_MASK_CASE(kMaskThreads)
    }
#undef HALO_MASK_CASE
}

hipError_t launch_scores_and_mask(int dtype, const float *h, const void *Bt, int r, float *scores,
                                  int T, int G, int K, const int8_t *prio_dev, int n_dev,
                                  const uint8_t *drop, int32_t *order, int8_t *group_dev,
                                  uint8_t *mask, int32_t *surv_idx, int32_t *n_surv, hipStream_t s)
{
    if (dtype != 0 && scores_apart(T, r, G)) {
        // many scores: on the matrix cores in a launch of their own (here a token's workgroup reads all of Bt for itself)
        const hipError_t e = launch_scores_many(h, (const bf16_t *)Bt, T, r, G, scores, s);
        if (e != hipSuccess) return e;
        mask_scores_kernel<float, false, 512><<<dim3(T), dim3(512), 0, s>>>(
            nullptr, nullptr, 0, scores, G, K, prio_dev, n_dev, drop, order, group_dev, mask, surv_idx, n_surv);
    } else if (dtype != 0) {
        launch_fused(h, (const bf16_t *)Bt, r, scores, T, G, K, prio_dev, n_dev, drop, order, group_dev, mask, surv_idx, n_surv, s);
    } else {
        launch_fused(h, (const float *)Bt, r, scores, T, G, K, prio_dev, n_dev, drop, order, group_dev, mask, surv_idx, n_surv, s);
    }
    return hipGetLastError();
}

template <typename WT>
static void launch_predict_mask(const void *x, int T, int d, int r, int G, const void *At, const void *Bt, float *scores, int K,
                                const int8_t *prio_dev, int n_dev, const uint8_t *drop, int32_t *order, int8_t *group_dev,
                                uint8_t *mask, int32_t *surv_idx, int32_t *n_surv, hipStream_t s)
{
    constexpr int NT = 512;                                      // 64 rows of At at a time (256 and 1024 threads: 8.2 and 7.1 us against 6.9)
    predict_mask_kernel<WT, NT><<<dim3(T), dim3(NT), 0, s>>>((const WT *)x, (const WT *)At, d, (const WT *)Bt, r, scores, G, K, prio_dev,
                                                             n_dev, drop, order, group_dev, mask, surv_idx, n_surv);
}

// Both predictor layers and the mask.  One launch where the first layer's weights are at most 128 KiB: every token's workgroup
// reads them for itself (from L2), which costs no more than a launch on the device (tiny block 6.9 us against 2.2 + 4.7) and saves the
// host one, and a pass over a small block waits for the host: tiny block 18.4 -> 17.6 us, d 1024 bf16, rank 64, 2 tokens 17.7 -> 17.1.
// Up to rank 128, two rounds of rows, and 128 groups, one round of eight waves over Bt: a block of d 256 in bf16, one token, in a
// graph, rank 64 / 128 / 256, two launches against one: 8 groups 12.0 / 12.3 / 12.3 us against 11.1 / 12.2 / 14.3, 128 groups 25.0 / 25.0 / 24.7
// against 23.8 / 24.7 / 26.7, 200 groups 32.1 / 32.3 / 32.0 against 32.6 / 33.8 / 35.6; float32, 16 tokens, 200 groups 27.7 against 29.2.
// At twice 128 KiB (d 512 float32, rank 128: 8.5 us against 3.2 + 4.6) it is level, beyond it slower (d 1000, rank 128: 11.7 against 9.0).
// Up to 64 tokens, the passes that wait for the host; with more the kernels that follow cover the launch (on the device one stays
// ahead: d 256 float32, 128 tokens 6.8 us against 3.3 + 4.6, 512 tokens 9.2 against 6.9 + 5.1).  Rows of bf16 that are no multiple of
// 128, up to 4 tokens: their FFN runs on the plain kernels, which gain from x in every die's L2, where the first layer's own launch
// leaves it (d 1000, 8 groups, rank 64, 64 tokens: their gate/up 50 us after two launches, 61 after one; 8 tokens 51.3 / 52.2 the pass).
hipError_t launch_predict_and_mask(int dtype, const void *x, int T, int d, int r, int G, const void *At, const void *Bt, float *h,
                                   float *scores, int K, const int8_t *prio_dev, int n_dev, const uint8_t *drop, int32_t *order,
                                   int8_t *group_dev, uint8_t *mask, int32_t *surv_idx, int32_t *n_surv, hipStream_t s)
{
    const int most = dtype != 0 && d % 128 != 0 ? 4 : 64;
    if (T <= most && r <= kOneLaunchRank && G <= kOneLaunchGroups && (size_t)r * d * (dtype == 0 ? 4 : 2) <= (size_t)128 << 10) {
        if (dtype == 0)
            launch_predict_mask<float>(x, T, d, r, G, At, Bt, scores, K, prio_dev, n_dev, drop, order, group_dev, mask, surv_idx, n_surv, s);
        else
            launch_predict_mask<bf16_t>(x, T, d, r, G, At, Bt, scores, K, prio_dev, n_dev, drop, order, group_dev, mask, surv_idx, n_surv, s);
        return hipGetLastError();
    }
    const hipError_t e = launch_predictor(dtype, x, T, d, r, G, At, Bt, h, nullptr, s);
    if (e != hipSuccess) return e;
    return launch_scores_and_mask(dtype, h, Bt, r, scores, T, G, K, prio_dev, n_dev, drop, order, group_dev, mask, surv_idx, n_surv, s);
}

}  // namespace halo
