// Semantic-aware predictor (paper Sec. III-B.2): h = ReLU(x A), scores = h B.
//
// Both layers are the same operation, out[t][j] = f(dot(X[t], W[j])), with the
// float32 summation order fixed so that the ranking derived from the scores is
// reproducible bit for bit: element i goes to partial sum (i/8) mod 64 (one
// partial per lane of a wave64, eight consecutive elements = one 16-byte bf16
// load), each partial is a fused-multiply-add chain in increasing i starting at
// +0, and the 64 partials are combined by a butterfly at distances 32..1.
// A matrix instruction that reduces several elements at once would not expose its
// internal summation order; one that takes a single element per instruction has none
// (hidden_mfma_kernel below), and a few tokens stay on the plain float ALUs.
#include "kernels.hpp"
#include "lds_loads.hpp"

namespace halo {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <typename XT, typename WT, bool RELU>
__global__ __launch_bounds__(256) void dot_rows_kernel(const XT *__restrict__ X,
                                                       const WT *__restrict__ W,
                                                       float *__restrict__ out, int T, int R, int n)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long idx = (long long)blockIdx.x * 4 + wave;
    if (idx >= (long long)T * R) return;                 // uniform per wave
    const int t = (int)(idx / R), j = (int)(idx % R);
    const float p = dot_order64(X + (size_t)t * n, W + (size_t)j * n, n, lane);
    if (lane == 0) out[idx] = RELU ? (p > 0.0f ? p : 0.0f) : p;
}

// The first layer for a tile's worth of tokens and more, bf16, where there are too few results for the matrix cores (hidden_mfma_kernel).
// A wave: four tokens against one row of At, so a row is loaded and unpacked once for four of them, and four butterflies are one from distance
// 16 down.  The loads of four steps of 512 elements are under way, without which the walk waits on each.  17 tokens, d 8192, rank 512: 17 us
// with a wave per result, now 12; its multiply-adds and conversions alone are 5, and 2.5 waves a SIMD don't hide the rest.
constexpr int kRowTokens = 4, kRowAhead = 4;

__global__ __launch_bounds__(256) void dot_rows_tokens_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W,
                                                              float *__restrict__ out, int T, int R, int n)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row_blocks = (R + 3) / 4;                          // a die keeps its rows for every token where this is a multiple of eight
    const int t0 = blockIdx.x / row_blocks * kRowTokens, j = blockIdx.x % row_blocks * 4 + wave;
    if (j >= R) return;
    const __amdgpu_buffer_rsrc_t bw = buffer_of(W + (size_t)j * n, 2 * n);
    __amdgpu_buffer_rsrc_t bx[kRowTokens];
#pragma unroll
    for (int t = 0; t < kRowTokens; ++t) {
        const bool any = t0 + t < T;
        bx[t] = buffer_of(X + (size_t)(any ? t0 + t : 0) * n, any ? 2 * n : 0);
    }
    // a piece past the end is zeros on both sides and leaves the chains as they are
    u32x4 wv[kRowAhead], xv[kRowAhead][kRowTokens];
    auto request = [&](int s, int k) __attribute__((always_inline)) {
        const uint32_t at = (uint32_t)k * 1024u + lane * 16;
        wv[s] = buffer_load16<0>(bw, at, 0);
#pragma unroll
        for (int t = 0; t < kRowTokens; ++t) xv[s][t] = buffer_load16<0>(bx[t], at, 0);
    };
    float p[kRowTokens] = {0.0f, 0.0f, 0.0f, 0.0f};
    const int nk = (n + 511) / 512;
#pragma unroll
    for (int s = 0; s < kRowAhead; ++s) request(s, s);
    for (int k = 0; k < nk; k += kRowAhead) {
#pragma unroll
        for (int s = 0; s < kRowAhead; ++s) {
            if (k + s < nk) {                                    // uniform
                float w[8];
                unpack8(wv[s], w);
#pragma unroll
                for (int t = 0; t < kRowTokens; ++t) {
                    float x[8];
                    unpack8(xv[s][t], x);
#pragma unroll
                    for (int e = 0; e < 8; ++e) p[t] = __builtin_fmaf(x[e], w[e], p[t]);
                }
            }
            request(s, k + kRowAhead + s);
        }
    }
    // the four butterflies as one from distance 16 down: half a wave, then a quarter, holds a token's
    auto meet = [](float a, float b, auto swap) {
        const auto v = swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b));
        return __builtin_bit_cast(float, (unsigned)v[0]) + __builtin_bit_cast(float, (unsigned)v[1]);
    };
    auto swap32 = [](unsigned a, unsigned b) { return __builtin_amdgcn_permlane32_swap(a, b, false, false); };
    auto swap16 = [](unsigned a, unsigned b) { return __builtin_amdgcn_permlane16_swap(a, b, false, false); };
    float v = meet(meet(p[0], p[1], swap32), meet(p[2], p[3], swap32), swap16);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    // quarters of the wave: tokens 0, 2, 1, 3
    const int quarter = lane >> 4, t = t0 + ((quarter & 1) << 1 | quarter >> 1);
    if ((lane & 15) == 0 && t < T) out[(size_t)t * R + j] = v > 0.0f ? v : 0.0f;
}

// The first layer for many tokens, bf16, on the matrix cores in the fixed order.
//
// v_mfma_f32_16x16x1_4b_f32 multiplies four independent blocks of 16 x 16 results by ONE element of the
// reduction dimension: every result is c = fma(a, b, c), rounded once (checked bit by bit against fmaf over
// ordinary values, denormals, overflow and infinities), so the order of a chain is the order in which the
// instructions are issued, which is exactly what the fixed order asks for.  Block b of a wave's instruction
// holds partial sums l + 16 b: lane (b, i) supplies element e of piece 64 k + l + 16 b of row i, e = 0..7 are
// eight instructions, and k walks the row.  Wave l of sixteen owns partial sums l + 16 b, so a
// workgroup holds all 64 partial sums of its (16 JT rows of At) x (16 TT tokens); distances 32 and 16 are
// then additions between a lane's own blocks, 8 .. 1 go through LDS once at the end.
// Nothing is spent on lane-crossing sums per result (half of the instructions of a wave-per-row form).
// Rows go to LDS a step of 512 elements at a time (a load: one row's 1 KiB; a row is padded by 16 bytes so that 16 rows'
// pieces fall into different banks).  BUFS >= 2: straight there, into that many buffers, and a step's fragments are read while the matrix
// instructions of the step before run, so that the barrier between two steps has work on both sides.  BUFS = 1: through registers
// into two buffers, a step's fragments read behind its barrier.  BUFS = 0, rows of up to two steps: fragments straight from memory.
// launch_hidden_mfma's caller says which is the faster where.  The longest walk, 1000 tokens, d = 8192, rank 512, takes 87 us with
// the second layer (107 through registers, eight waves of two partial sums): the matrix instruction needs 66 of them at the 130
// TFLOP/s that it reaches alone; with loads that move nothing a few less, so the rest is the conversions and LDS reads beside it.
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr int kHidRow = 1024 + 16;          // padded LDS row, bytes
constexpr int kHidWaves = 16;

template <int TT, int JT, int BUFS>
__global__ __launch_bounds__(kHidWaves * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void hidden_mfma_kernel(
    const bf16_t *__restrict__ X, const bf16_t *__restrict__ At, float *__restrict__ h, int T, int d, int r,
    int n_tt, int n_jt)
{
    constexpr int kTiles = TT * JT, kSets = TT + JT, kRows = 16 * kSets, kStage = kRows * kHidRow;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];   // BUFS of: TT * 16 token rows, then JT * 16 rows of At; at the end the sums
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // a die (workgroups are dealt round-robin to eight) takes consecutive items, the rows of At fastest: its
    // token rows stay in its L2
    const int n_items = n_tt * n_jt, per_die = (n_items + 7) >> 3;
    const int slot = blockIdx.x >> 3, item = (blockIdx.x & 7) * per_die + slot;
    if (slot >= per_die || item >= n_items) return;
    const int t0 = (item / n_jt) * 16 * TT, j0 = (item % n_jt) * 16 * JT;
    const int nk = (d + 511) / 512;
    const int i = lane & 15, b = lane >> 4;
    u32x4 raw[2][kSets];
    f32x16_t acc[kTiles];
#pragma unroll
    for (int n = 0; n < kTiles; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[n][e] = 0.0f;
    auto multiply = [&](const u32x4 (&cur)[kSets], int e) {      // element e of the fragments
        float f[kSets];
#pragma unroll
        for (int n = 0; n < kSets; ++n) f[n] = e % 2 == 0 ? bf16_lo(cur[n][e / 2]) : bf16_hi(cur[n][e / 2]);
#pragma unroll
        for (int n = 0; n < kTiles; ++n)
            acc[n] = __builtin_amdgcn_mfma_f32_16x16x1f32(f[TT + n % JT], f[n / JT], acc[n], 0, 0, 0);
    };
    if constexpr (BUFS == 0) {
        // rows of up to two steps: all of the wave's fragments straight from memory, requested together
        const __amdgpu_buffer_rsrc_t rx = buffer_of(X + (size_t)t0 * d), ra = buffer_of(At + (size_t)j0 * d);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int n = 0; n < kSets; ++n) {
                const uint32_t row = n < TT ? min(i + 16 * n, T - 1 - t0) : min(i + 16 * (n - TT), r - 1 - j0), at = k * 512 + (wave + 16 * b) * 8;
                raw[k][n] = buffer_load16<0>(n < TT ? rx : ra, at < (uint32_t)d ? (row * d + at) * 2 : kOutOfRange, 0);
            }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (k < nk) {
#pragma unroll
                for (int e = 0; e < 8; ++e) multiply(raw[k], e);
            }
    } else {
        // this wave loads row `wave` of every set of 16; rows past the end repeat the last one (never stored)
        uint32_t row_at[kSets];
#pragma unroll
        for (int n = 0; n < kSets; ++n)
            row_at[n] = (uint32_t)(n < TT ? min(wave + 16 * n, T - 1 - t0) : min(wave + 16 * (n - TT), r - 1 - j0)) * (uint32_t)d * 2;
        auto read = [&](u32x4 (&f)[kSets], int buf) {
            const unsigned char *piece = lds + buf * kStage + i * kHidRow + (wave + 16 * b) * 16;
#pragma unroll
            for (int n = 0; n < kSets; ++n) f[n] = *reinterpret_cast<const u32x4 *>(piece + n * 16 * kHidRow);
        };
        if constexpr (BUFS == 1) {
            // through registers, into two buffers: step k is multiplied, step k + 1 goes to LDS beside it, step k + 2 is asked for behind it
            const __amdgpu_buffer_rsrc_t rx = buffer_of(X + (size_t)t0 * d), ra = buffer_of(At + (size_t)j0 * d);
            u32x4 v[kSets];
            auto fetch = [&](int k) {
                const uint32_t at = k * 512 + lane * 8;          // (d is a multiple of 8; 0 * 0 leaves a chain as it is)
#pragma unroll
                for (int n = 0; n < kSets; ++n) v[n] = buffer_load16<0>(n < TT ? rx : ra, at < (uint32_t)d ? row_at[n] + at * 2 : kOutOfRange, 0);
            };
            auto park = [&](int k, int n) {
                *reinterpret_cast<u32x4 *>(lds + (k & 1) * kStage + (n * 16 + wave) * kHidRow + lane * 16) = v[n];
            };
            fetch(0);
#pragma unroll
            for (int n = 0; n < kSets; ++n) park(0, n);
            fetch(1);
            for (int k = 0; k < nk; ++k) {
                __syncthreads();                                 // step k is in LDS, step k - 1 is used up
                read(raw[0], k & 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    multiply(raw[0], e);
                    if (e < kSets) park(k + 1, e);
                    __builtin_amdgcn_sched_barrier(0);
                }
                fetch(k + 2);
            }
            __syncthreads();
        } else {
            const srd_t srd_x = make_srd(X + (size_t)t0 * d, true), srd_a = make_srd(At + (size_t)j0 * d, true);
            const uint32_t lds0 = (uint32_t)(size_t)lds + wave * kHidRow;
            auto load = [&](int n, int k, int buf) {                     // its row of set n, step k; zeros past the row's or the walk's end
                const uint32_t at = k * 512 + lane * 8 < d ? lane * 16u : kNoRow;
                load_to_lds16(n < TT ? srd_x : srd_a, at, k < nk ? row_at[n] + k * 1024u : 0u, lds0 + buf * kStage + n * 16 * kHidRow);
            };
#pragma unroll
            for (int k = 0; k < BUFS; ++k)
#pragma unroll
                for (int n = 0; n < kSets; ++n)
                    if (BUFS > 2 || k < nk) load(n, k, k);
            if (BUFS > 2 || nk > 1)
                wait_loads<(BUFS - 1) * kSets>();
            else
                wait_loads<0>();
            __syncthreads();
            read(raw[0], 0);
            int buf = 0;                                                 // buffer of step k
            // At the top of step k its fragments are in registers.  The barrier says that step k + 1 has landed and that everybody has
            // read step k, whose buffer is then handed to step k + BUFS.
            auto step = [&](const u32x4 (&cur)[kSets], u32x4 (&next)[kSets], int k) __attribute__((always_inline)) {
                const int nbuf = buf == BUFS - 1 ? 0 : buf + 1;
                if (BUFS > 2 || k + 1 < nk) {
                    wait_loads<(BUFS - 2) * kSets>();
                    __syncthreads();
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    multiply(cur, e);
                    if (e == 0 && (BUFS > 2 || k + 1 < nk)) read(next, nbuf);
                    if (e >= 1 && e - 1 < kSets && (BUFS > 2 || k + 2 < nk)) load(e - 1, k + BUFS, buf);
                    __builtin_amdgcn_sched_barrier(0);
                }
                buf = nbuf;
            };
            for (int k = 0; k < nk; k += 2) {
                step(raw[0], raw[1], k);
                if (k + 1 < nk) step(raw[1], raw[0], k + 1);
            }
            wait_loads<0>();                                             // (of loads that move zeros)
            __syncthreads();
        }
    }
    // distances 32 and 16: blocks (0, 2) and (1, 3); result element 4 b + m of a lane is block b, row 4 (lane / 16) + m,
    // token lane % 16
    f32x4_t *sums = reinterpret_cast<f32x4_t *>(lds);            // [l][tile][lane]
#pragma unroll
    for (int n = 0; n < kTiles; ++n) {
        f32x4_t s;
#pragma unroll
        for (int m = 0; m < 4; ++m) s[m] = (acc[n][m] + acc[n][8 + m]) + (acc[n][4 + m] + acc[n][12 + m]);
        sums[(wave * kTiles + n) * 64 + lane] = s;
    }
    __syncthreads();
    // distances 8, 4, 2, 1
    if (wave < kTiles) {
        const int n = wave;
        f32x4_t p[16];
#pragma unroll
        for (int l = 0; l < 16; ++l) p[l] = sums[(l * kTiles + n) * 64 + lane];
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
            for (int l = 0; l < 8; ++l)
                if (l < off)
#pragma unroll
                    for (int m = 0; m < 4; ++m) p[l][m] = p[l][m] + p[l + off][m];
        const int t = t0 + (n / JT) * 16 + i, j = j0 + (n % JT) * 16 + 4 * b;
        if (t < T) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (j + m < r) h[(size_t)t * r + j + m] = p[0][m] > 0.0f ? p[0][m] : 0.0f;
        }
    }
}

template <int TT, int JT, int BUFS>
static hipError_t launch_hidden_mfma(const bf16_t *x, int T, int d, int r, const bf16_t *At, float *h, hipStream_t s)
{
    constexpr int kStages = (BUFS == 1 ? 2 : BUFS) * 16 * (TT + JT) * kHidRow, kSums = TT * JT * 16 * 1024, lds = kStages > kSums ? kStages : kSums;
    const hipError_t lds_ok = allow_lds<hidden_mfma_kernel<TT, JT, BUFS>>(lds);
    if (lds_ok != hipSuccess) return lds_ok;
    const int n_tt = (T + 16 * TT - 1) / (16 * TT), n_jt = (r + 16 * JT - 1) / (16 * JT);
    hidden_mfma_kernel<TT, JT, BUFS><<<dim3((n_tt * n_jt + 7) / 8 * 8), dim3(kHidWaves * 64), lds, s>>>(x, At, h, T, d, r, n_tt, n_jt);
    return hipSuccess;
}

// The second layer for many tokens: scores[t][g] = h[t] . Bt[g], the same instruction and order.  The rows are short (one
// or two pieces per lane), so a 16 x 16 tile is all a workgroup does and its lanes take their pieces straight from memory,
// nothing is staged.  Eight waves: two values of l each.  Bound by the launch and one memory round trip
// (1000 x 512 x 224: 9.7 us).
constexpr int kScoreWaves = 8;

__global__ __launch_bounds__(kScoreWaves * 64) void scores_mfma_kernel(
    const float *__restrict__ H, const bf16_t *__restrict__ Bt, float *__restrict__ scores, int T, int r, int G)
{
    constexpr int kL = 16 / kScoreWaves;
    __shared__ __attribute__((aligned(16))) f32x4_t sums[16 * 64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, i = lane & 15, b = lane >> 4;
    const int t0 = blockIdx.y * 16, g0 = blockIdx.x * 16;
    const float *hrow = H + (size_t)min(t0 + i, T - 1) * r;      // rows past the end repeat the last one (never stored)
    const bf16_t *brow = Bt + (size_t)min(g0 + i, G - 1) * r;
    const int nk = (r + 511) / 512;
    f32x16_t acc[kL];
#pragma unroll
    for (int l = 0; l < kL; ++l)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[l][e] = 0.0f;
    float hv[kL][8], bv[kL][8];
    auto fetch = [&](int k) {
#pragma unroll
        for (int l = 0; l < kL; ++l) {
            const int e0 = (64 * k + kL * wave + l + 16 * b) * 8;
            const bool ok = e0 < r;                              // (r is a multiple of 8)
            load8(hrow + (ok ? e0 : 0), hv[l]);
            load8(brow + (ok ? e0 : 0), bv[l]);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                hv[l][e] = ok ? hv[l][e] : 0.0f;                 // 0 * 0 leaves a chain as it is
                bv[l][e] = ok ? bv[l][e] : 0.0f;
            }
        }
    };
    for (int k = 0; k < nk; ++k) {
        fetch(k);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int l = 0; l < kL; ++l) acc[l] = __builtin_amdgcn_mfma_f32_16x16x1f32(bv[l][e], hv[l][e], acc[l], 0, 0, 0);
    }
    // as in hidden_mfma_kernel: distances 32 and 16 are a lane's own blocks
#pragma unroll
    for (int l = 0; l < kL; ++l) {
        f32x4_t s;
#pragma unroll
        for (int m = 0; m < 4; ++m) s[m] = (acc[l][m] + acc[l][8 + m]) + (acc[l][4 + m] + acc[l][12 + m]);
        sums[(kL * wave + l) * 64 + lane] = s;
    }
    __syncthreads();
    // distances 8, 4, 2, 1: a thread per score, token c of the tile, group row
    if (tid < 256) {
        const int c = tid >> 4, row = tid & 15;
        const float *one = reinterpret_cast<const float *>(sums) + ((row >> 2) * 16 + c) * 4 + (row & 3);
        float p[16];
#pragma unroll
        for (int l = 0; l < 16; ++l) p[l] = one[l * 256];
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
            for (int l = 0; l < 8; ++l)
                if (l < off) p[l] = p[l] + p[l + off];
        if (t0 + c < T && g0 + row < G) scores[(size_t)(t0 + c) * G + g0 + row] = p[0];
    }
}

// whether a launch of their own pays: inside the mask kernel a token's workgroup reads all of Bt for itself and spends most
// instructions on lane-crossing sums, but the second launch costs a few microseconds.  us, both kernels against the one
// (T x r x G): 1000 x 512 x 224 22.0 against 36.8, 700 x 512 x 120 12.0 against 16.2, 2000 x 256 x 86 16.5 against 20.6;
// 512 x 256 x 86 11.4 against 9.3.  Every shape measured from 40 Mi on gains (2 to 90 us of a pass).  Below, the two cross
// at 10 to 20 Mi where there are 86 to 160 groups (900 x 256 x 86, 19 Mi: level; 512 x 256 x 86, 11 Mi: 1.3 lost), lower with
// more groups or ranks of 64 and less (200 x 512 x 224, 22 Mi: 3.5 to be had; 1500 x 64 x 224, 21 Mi: 9), and at 28 Mi with
// 64 groups.
bool scores_apart(int T, int r, int G) { return T >= 64 && (long long)T * r * G >= 40ll << 20; }

hipError_t launch_scores_many(const float *h, const bf16_t *Bt, int T, int r, int G, float *scores, hipStream_t s)
{
    constexpr int kRun = 65535 * 16;                             // tokens of a launch: a grid's y ends at 65535
    for (int t0 = 0;; t0 += kRun) {
        const int n = T - t0 < kRun ? T - t0 : kRun;
        scores_mfma_kernel<<<dim3((G + 15) / 16, (n + 15) / 16), dim3(kScoreWaves * 64), 0, s>>>(
            h + (size_t)t0 * r, Bt, scores + (size_t)t0 * G, n, r, G);
        if (T - t0 <= kRun) return hipGetLastError();
    }
}

// The largest tile that still gives every compute unit a workgroup: the bytes staged per result fall with the
// tile (2 x 2: 64 rows per 1024 results, 1 x 1: 32 per 256), but a unit without a workgroup does nothing.  Fewer
// than 16 tokens do not fill a tile and stay with a wave per result (2..8 tokens: 7-13 us), and so do few results: a
// tile's workgroup walks its row in steps of 512 with a barrier each, while a wave per result has all of it under
// way.  Both layers in us, wave against tile: 16 x 64 results d 1024 4.7 against 6.6, d 8192 6.9 against 17.6; 48 x 256
// d 4096 10.4 against 11.5; 64 x 256 d 4096 12.3 against 11.5; 32 x 512 d 8192 19.9 against 17.7.  The two meet between
// 12800 and 16384 results at every d from 128 to 8192.
static bool hidden_rows_tiled(const bf16_t *x, int T, int d, int r, const bf16_t *At, float *h, hipStream_t s, hipError_t &e)
{
    if (T < 16 || (long long)T * r < 14 * 1024 || d > 1 << 24) return false;   // (rows are addressed with 32-bit offsets)
    const int n_tt = (T + 31) / 32;
    // How the rows come (both layers, us): up to 768 elements straight to registers, 32 tokens, rank 512, d 512 5.5 against 5.6 and 5.7, d 768
    // 6.1 against 6.4 and 6.7, but d 1024 6.5 against 6.4; tiles of one by one through registers up to 3072, 128 tokens, rank 256, d 1024
    // 6.8 against 7.1 (loads to two buffers) to 7.5 (four), d 2048 8.4 against 8.7 and 8.9, d 3072 10.0 against 10.3, d 4096 11.6
    // against 11.7, but 32 tokens, rank 512, d 8192 17.5 against 16.4; loads to LDS in the larger tiles, 1000 tokens, rank 512, d 1024 25.2
    // against 23.9, d 8192 94 against 87.
    if (n_tt * ((r + 31) / 32) >= 256)
        e = d <= 768 ? launch_hidden_mfma<2, 2, 0>(x, T, d, r, At, h, s) : launch_hidden_mfma<2, 2, 2>(x, T, d, r, At, h, s);
    else if (n_tt * ((r + 15) / 16) >= 256)
        e = d <= 768    ? launch_hidden_mfma<2, 1, 0>(x, T, d, r, At, h, s)
            : d <= 2048 ? launch_hidden_mfma<2, 1, 2>(x, T, d, r, At, h, s)
                        : launch_hidden_mfma<2, 1, 3>(x, T, d, r, At, h, s);
    else
        e = d <= 768    ? launch_hidden_mfma<1, 1, 0>(x, T, d, r, At, h, s)
            : d <= 3072 ? launch_hidden_mfma<1, 1, 1>(x, T, d, r, At, h, s)
                        : launch_hidden_mfma<1, 1, 4>(x, T, d, r, At, h, s);
    return true;
}
static bool hidden_rows_tiled(const float *, int, int, int, const float *, float *, hipStream_t, hipError_t &) { return false; }

// A wave per four results instead of one where that leaves each SIMD more than two waves and a wave a walk of eight steps and more.
// A pass, us, one / four: 17 tokens, d 8192, rank 512, 4-bit weights 147.9 / 143.1, 26 155.0 / 152.7; 34 x 256 of d 4096 56.7 / 55.7, 40 x 256
// in bf16 80.7 / 79.7; 48 x 256 of d 5120 71.6 / 70.6.  With 8192 results and fewer the waves are too few to hide their loads (17 x 256 of
// d 4096 level, 32 x 256 of d 5120 64.4 / 64.8, 100 x 64 of d 2048 47.4 / 48.1), and short walks do better in many waves (40 x 256 of
// d 2048 level, 25 x 512 of d 1024 34.7 / 36.9).
template <typename WT>
static bool hidden_rows_shared(int T, int d, long long results)
{
    return sizeof(WT) == 2 && T >= 16 && results > 8192 && d >= 4096 && d <= 1 << 24;
}

template <typename WT>
static hipError_t predict_t(const WT *x, int T, int d, int r, int G, const WT *At, const WT *Bt,
                            float *h, float *scores, hipStream_t s)
{
    long long n1 = (long long)T * r, n2 = (long long)T * G;
    hipError_t e = hipSuccess;
    if (hidden_rows_tiled(x, T, d, r, At, h, s, e)) {
    } else if (hidden_rows_shared<WT>(T, d, n1)) {
        dot_rows_tokens_kernel<<<dim3((unsigned)((r + 3) / 4 * ((T + kRowTokens - 1) / kRowTokens))), dim3(256), 0, s>>>(
            (const bf16_t *)x, (const bf16_t *)At, h, T, r, d);
    } else {
        dot_rows_kernel<WT, WT, true><<<dim3((unsigned)((n1 + 3) / 4)), dim3(256), 0, s>>>(x, At, h, T, r, d);
    }
    if (e != hipSuccess) return e;
    if (scores && sizeof(WT) == 2 && scores_apart(T, r, G)) return launch_scores_many(h, (const bf16_t *)Bt, T, r, G, scores, s);
    if (scores)
        dot_rows_kernel<float, WT, false><<<dim3((unsigned)((n2 + 3) / 4)), dim3(256), 0, s>>>(h, Bt, scores, T, G, r);
    return hipGetLastError();
}

// scores == nullptr: first layer only (h), the second layer is then fused into the mask kernel
hipError_t launch_predictor(int dtype, const void *x, int T, int d, int r, int G, const void *At,
                            const void *Bt, float *h, float *scores, hipStream_t s)
{
    if (dtype == 0)
        return predict_t<float>((const float *)x, T, d, r, G, (const float *)At, (const float *)Bt, h, scores, s);
    return predict_t<bf16_t>((const bf16_t *)x, T, d, r, G, (const bf16_t *)At, (const bf16_t *)Bt, h, scores, s);
}

}  // namespace halo
