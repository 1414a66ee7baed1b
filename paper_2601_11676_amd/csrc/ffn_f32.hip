// Group-sparse SwiGLU FFN in float32 on the matrix cores (paper Sec. II-A neuron groups; merge = sum).
//
// v_mfma_f32_16x16x4_f32 multiplies 16 weight rows by 16 tokens with float32 operands, products and sums, so
// the arithmetic is what a chain of fused multiply-adds gives, in another order.  The blocks this serves
// are small (the tiny block: 16 tokens, 256 x 1024): what bounds them is the chain of memory round trips in
// front of each result, not bytes or flops, so both kernels cut the reduction dimension over the waves of a
// workgroup until a wave's share is a handful of loads that are all requested together, and meet in LDS once.
//   gate/up : workgroup = 16 neurons of one group x up to 64 tokens; leaves at once when none of its tokens
//             keeps the group, so no list of groups is needed.  act[t][ffn] = mask ? SiLU(gate) * up : 0.
//   down    : workgroup = 16 outputs x up to 32 tokens, its waves share the pieces of the union's groups.
// WHICH 4 of a 16-element piece an instruction's lane group multiplies is free as long as both operands agree:
// lane (i, q) = (l % 16, l / 16) holds elements 4 q .. 4 q + 3 of row i in one 16-byte load, and instruction e
// multiplies element 4 q + e of every lane group.  D: lane l holds column (token) l % 16, rows 4 (l / 16) .. + 3.
// Tiny block: gate/up 4.6 us and down 6.9 us per launch, against 10.0 and 68 us for a wave per neuron / per output
// row that walked its groups one 4-byte load at a time; the pass called from Python 21 us (89).  1000 x 24 groups, one
// token: 28 us (265).  Error against 64 bits over d 128..1024, 4..24 groups, 1..64 tokens: 0.89..1.01 times theirs.
#include "kernels.hpp"

namespace halo {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4_t mfma4(float a, float b, const f32x4_t &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int N>
__device__ __forceinline__ f32x4_t pairwise_sum(f32x4_t (&p)[N])
{
#pragma unroll
    for (int off = N / 2; off >= 1; off >>= 1)
#pragma unroll
        for (int w = 0; w < N / 2; ++w)
            if (w < off) p[w] += p[w + off];
    return p[0];
}

constexpr int kGateUpF32Waves = 8, kDownF32Waves = 16;

// Where the lanes of group q load the four elements of piece p that they hold, in elements from the row's start.  The last
// piece may hold 8 elements, and the only one of a row of 8 as well: lanes past the end take the row's first four, unused.
__host__ __device__ constexpr bool in_row(int p, int q, int d) { return p * 16 + 4 * q < d; }
__host__ __device__ constexpr int piece_at(int p, int q, int d) { return in_row(p, q, d) ? p * 16 + 4 * q : 0; }
constexpr bool loads_stay_in_row(int d)
{
    for (int p = 0; p < (d + 15) / 16; ++p)
        for (int q = 0; q < 4; ++q)
            if (piece_at(p, q, d) < 0 || piece_at(p, q, d) + 4 > d) return false;
    return true;
}
static_assert(loads_stay_in_row(8) && loads_stay_in_row(16) && loads_stay_in_row(24) && loads_stay_in_row(520), "d is a multiple of 8");

// NT: token tiles of 16 per workgroup.  grid (ffn / 16, ceil(T / (16 NT)))
template <int NT>
__global__ __launch_bounds__(kGateUpF32Waves * 64) void gate_up_f32(
    const float *__restrict__ x, int T, int d, int G, int gs, const float *__restrict__ Wg, const float *__restrict__ Wu,
    const uint8_t *__restrict__ mask, float *__restrict__ act, int ffn)
{
    constexpr int W = kGateUpF32Waves, U = NT == 4 ? 1 : 2;      // pieces per batch and wave
    __shared__ f32x4_t part[W][2][NT][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.x * 16, g = n0 / gs, t0 = blockIdx.y * 16 * NT;
    const uint8_t mine = mask[(size_t)min(t0 + min(lane, 16 * NT - 1), T - 1) * G + g];
    if (__ballot(mine != 0) == 0ull) return;                     // uniform: the same bytes in every wave
    const float *wg = Wg + (size_t)(n0 + i) * d, *wu = Wu + (size_t)(n0 + i) * d;
    const float *xr[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) xr[n] = x + (size_t)min(t0 + 16 * n + i, T - 1) * d;
    const int np = (d + 15) / 16;                                // pieces of 16; the last one may hold 8
    struct Batch {
        f32x4_t g[U], u[U], x[NT][U];
    };
    auto fetch = [&](Batch &b, int p0) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int p = p0 + W * k;
            if (p < np) {                                        // uniform
                const bool ok = in_row(p, q, d);
                const int at = piece_at(p, q, d);
                b.g[k] = *reinterpret_cast<const f32x4_t *>(wg + at);
                b.u[k] = *reinterpret_cast<const f32x4_t *>(wu + at);
#pragma unroll
                for (int n = 0; n < NT; ++n) b.x[n][k] = *reinterpret_cast<const f32x4_t *>(xr[n] + at);
                if (!ok) {
                    b.g[k] = b.u[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int n = 0; n < NT; ++n) b.x[n][k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
    };
    f32x4_t cg[NT], cu[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) cg[n] = cu[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // A batch has a sum per instruction of a piece, folded pairwise at its end: no chain is longer than 8 products, as in
    // a wave per row (one running sum per wave was up to twice as far from 64 bits, chains of 16 up to 1.1 times).
    f32x4_t bg[NT][4], bu[NT][4];
    auto multiply = [&](const Batch &b, int p0) {
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (p0 + W * k < np) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        bg[n][e] = mfma4(b.g[k][e], b.x[n][k][e], bg[n][e]);
                        bu[n][e] = mfma4(b.u[k][e], b.x[n][k][e], bu[n][e]);
                    }
            }
    };
    Batch A, B;
    fetch(A, wave);
    auto clear = [&]() {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) bg[n][e] = bu[n][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto fold = [&]() {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            cg[n] += (bg[n][0] + bg[n][1]) + (bg[n][2] + bg[n][3]);
            cu[n] += (bu[n][0] + bu[n][1]) + (bu[n][2] + bu[n][3]);
        }
    };
    for (int p0 = wave; p0 < np; p0 += 2 * W * U) {
        clear();
        fetch(B, p0 + W * U);
        multiply(A, p0);
        if (U > 1) {
            fold();
            clear();
        }
        fetch(A, p0 + 2 * W * U);
        multiply(B, p0 + W * U);
        fold();
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        part[wave][0][n][lane] = cg[n];
        part[wave][1][n][lane] = cu[n];
    }
    __syncthreads();
    if (wave < NT) {
        f32x4_t pg[W], pu[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            pg[w] = part[w][0][wave][lane];
            pu[w] = part[w][1][wave][lane];
        }
        const f32x4_t sg = pairwise_sum(pg), su = pairwise_sum(pu);
        const int t = t0 + 16 * wave + i;
        if (t < T) {
            const bool keep = mask[(size_t)t * G + g] != 0;
            f32x4_t v;
#pragma unroll
            for (int m = 0; m < 4; ++m) v[m] = keep ? silu_mul(sg[m], su[m]) : 0.0f;
            *reinterpret_cast<f32x4_t *>(act + (size_t)t * ffn + n0 + 4 * q) = v;
        }
    }
}

// grid (ceil(d / 16), ceil(T / (16 NT))); reads act of the groups that a token of its own range keeps
template <int NT>
__global__ __launch_bounds__(kDownF32Waves * 64) void down_f32(
    const float *__restrict__ act, int ffn, int T, int d, int G, int gs, const float *__restrict__ Wd,
    const uint8_t *__restrict__ mask, float *__restrict__ y)
{
    constexpr int W = kDownF32Waves, U = 2;
    __shared__ f32x4_t part[W][NT][64];
    __shared__ int s_list[1024], s_cnt[W];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i = lane & 15, q = lane >> 4;
    const int j0 = blockIdx.x * 16, t0 = blockIdx.y * 16 * NT, t1 = min(T, t0 + 16 * NT);
    // the union of the range's groups, ascending: a thread per group (G <= 1024)
    const int g = threadIdx.x;
    unsigned any = 0;
    for (int t = t0; t < t1; t += 8) {
        uint8_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = mask[(size_t)min(t + k, t1 - 1) * G + min(g, G - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) any |= v[k];
    }
    const unsigned long long kept = __ballot(g < G && any != 0u);
    if (lane == 0) s_cnt[wave] = __popcll(kept);
    __syncthreads();
    int before = 0, n_u = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        before += w < wave ? s_cnt[w] : 0;
        n_u += s_cnt[w];
    }
    if ((kept >> lane) & 1ull) s_list[before + __popcll(kept & ((1ull << lane) - 1ull))] = g;
    __syncthreads();
    const int per = gs / 16, items = n_u * per;                  // pieces of 16 neurons
    const float *wrow = Wd + (size_t)min(j0 + i, d - 1) * gs + 4 * q;
    const float *ar[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) ar[n] = act + (size_t)min(t0 + 16 * n + i, T - 1) * ffn + 4 * q;
    struct Batch {
        f32x4_t w[U], a[NT][U];
    };
    auto fetch = [&](Batch &b, int p0) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int p = p0 + W * k;
            if (p < items) {                                     // uniform
                const int u = p / per, m = (p - u * per) * 16, gu = s_list[u];
                b.w[k] = *reinterpret_cast<const f32x4_t *>(wrow + (size_t)gu * d * gs + m);
#pragma unroll
                for (int n = 0; n < NT; ++n) b.a[n][k] = *reinterpret_cast<const f32x4_t *>(ar[n] + (size_t)gu * gs + m);
            }
        }
    };
    f32x4_t c[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) c[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    f32x4_t bs[NT][4];                                           // as in gate_up_f32
    auto multiply = [&](const Batch &b, int p0) {
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (p0 + W * k < items) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int n = 0; n < NT; ++n) bs[n][e] = mfma4(b.w[k][e], b.a[n][k][e], bs[n][e]);
            }
    };
    Batch A, B;
    fetch(A, wave);
    auto clear = [&]() {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) bs[n][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto fold = [&]() {
#pragma unroll
        for (int n = 0; n < NT; ++n) c[n] += (bs[n][0] + bs[n][1]) + (bs[n][2] + bs[n][3]);
    };
    for (int p0 = wave; p0 < items; p0 += 2 * W * U) {
        clear();
        fetch(B, p0 + W * U);
        multiply(A, p0);
        if (NT == 1) {                                           // (two tiles: the registers of a second fold spill)
            fold();
            clear();
        }
        fetch(A, p0 + 2 * W * U);
        multiply(B, p0 + W * U);
        fold();
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) part[wave][n][lane] = c[n];
    __syncthreads();
    if (wave < NT) {
        f32x4_t p[W];
#pragma unroll
        for (int w = 0; w < W; ++w) p[w] = part[w][wave][lane];
        const f32x4_t s = pairwise_sum(p);
        const int t = t0 + 16 * wave + i, j = j0 + 4 * q;
        if (t < T && j < d) *reinterpret_cast<f32x4_t *>(y + (size_t)t * d + j) = s;     // (d is a multiple of 8)
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
bool f32_path_supported(int gs) { return gs % 16 == 0; }

template <int NT>
static void launch_gate_up(const float *x, int T, int d, int G, int gs, const float *Wg, const float *Wu,
                           const uint8_t *mask, float *act, hipStream_t s)
{
    const int ffn = G * gs;
    launch_timed("gate_up_f32", gate_up_f32<NT>, dim3(ffn / 16, (T + 16 * NT - 1) / (16 * NT)), dim3(kGateUpF32Waves * 64), s,
                 x, T, d, G, gs, Wg, Wu, mask, act, ffn);
}

template <int NT>
static void launch_down(const float *act, int T, int d, int G, int gs, const float *Wd, const uint8_t *mask, float *y,
                        hipStream_t s)
{
    down_f32<NT><<<dim3((d + 15) / 16, (T + 16 * NT - 1) / (16 * NT)), dim3(kDownF32Waves * 64), 0, s>>>(act, G * gs, T, d, G,
                                                                                                   gs, Wd, mask, y);
}

// The weights are read once per range of tokens (from L2 after the first), so a range takes as many tokens as the
// registers of its waves allow: 64 in gate/up, 32 in down (sixteen waves).  A range of down lies within one of gate/up,
// so the groups it walks have been written.
static void launch_blocks(const float *x, int T, int d, int G, int gs, const float *Wg, const float *Wu, const float *Wd,
                          const uint8_t *mask, float *y, float *act, hipStream_t s)
{
    if (T <= 16)
        launch_gate_up<1>(x, T, d, G, gs, Wg, Wu, mask, act, s);
    else if (T <= 32)
        launch_gate_up<2>(x, T, d, G, gs, Wg, Wu, mask, act, s);
    else
        launch_gate_up<4>(x, T, d, G, gs, Wg, Wu, mask, act, s);
    if (T <= 16)
        launch_down<1>(act, T, d, G, gs, Wd, mask, y, s);
    else
        launch_down<2>(act, T, d, G, gs, Wd, mask, y, s);
}

hipError_t launch_ffn_f32(const float *x, int T, int d, int G, int gs, const float *Wg, const float *Wu, const float *Wd,
                          const uint8_t *mask, float *y, float *act, hipStream_t s)
{
    constexpr int kRun = 1 << 20;                                // ranges of tokens are a grid's y, which ends at 65535
    for (int t0 = 0;; t0 += kRun) {
        const size_t t = (size_t)t0;
        launch_blocks(x + t * d, T - t0 < kRun ? T - t0 : kRun, d, G, gs, Wg, Wu, Wd, mask + t * G, y + t * d,
                      act + t * G * gs, s);
        if (T - t0 <= kRun) return hipGetLastError();
    }
}

}  // namespace halo
