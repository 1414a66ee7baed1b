// Group-sparse SwiGLU FFN in float32 on the matrix cores (paper Sec. II-A neuron groups; merge = sum).
//
// v_mfma_f32_16x16x4_f32 multiplies 16 weight rows by 16 tokens with float32 operands, products and sums, so
// the arithmetic is what a chain of fused multiply-adds gives, in another order.  The blocks this serves
// are small (the tiny block: 16 tokens, 256 x 1024): what bounds them is the chain of memory round trips in
// front of each result, not bytes or flops, so both kernels cut the reduction dimension over the waves of a
// workgroup until a wave's share is a handful of loads that are all requested together, and meet in LDS once.
//   gate/up : workgroup = 16 neurons of one group x up to 64 tokens; leaves at once when none of its tokens
//             keeps the group, so no list of groups is needed.  act = mask ? SiLU(gate) * up : 0.
//   down    : workgroup = 16 outputs x up to 16 or 32 tokens, its waves share the pieces of the union's groups.
// WHICH 4 of a 16-element piece an instruction's lane group multiplies is free as long as both operands agree:
// lane (i, q) = (l % 16, l / 16) holds elements 4 q .. 4 q + 3 of row i in one 16-byte load, and instruction e
// multiplies element 4 q + e of every lane group.  D: lane l holds column (token) l % 16, rows 4 (l / 16) .. + 3.
// Tiny block: gate/up 4.6 us and down 5.8 us per launch; a wave per neuron / per output
// row that walked its groups one 4-byte load at a time took 10, 68 and 89.  Error against 64 bits over d 128..1024, 4..24 groups,
// 1..64 tokens: 0.89..1.01 times theirs.
#include "kernels.hpp"
#include "mask_device.hpp"

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
constexpr int kRowF32 = 128 + 4;                                 // padded LDS row of a chunk of 128 elements

__device__ __forceinline__ f32x4_t load4(__amdgpu_buffer_rsrc_t b, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(f32x4_t, buffer_load16<0>(b, voff, soff));
}

// Sums of products over pieces of 16 elements, taken in pairs: a sum per instruction of a piece, folded pairwise after every
// second piece, so that no chain is longer than 8 products, as in a wave per row (one running sum per wave was up to twice as
// far from 64 bits, chains of 16 up to 1.1 times).
template <int NT>
struct PairSum {
    f32x4_t s[NT][4];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[n][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add(const f32x4_t &w, const f32x4_t (&x)[NT])
    {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int n = 0; n < NT; ++n) s[n][e] = mfma4(w[e], x[n][e], s[n][e]);
    }
    __device__ __forceinline__ void fold(f32x4_t (&c)[NT])
    {
#pragma unroll
        for (int n = 0; n < NT; ++n) c[n] += (s[n][0] + s[n][1]) + (s[n][2] + s[n][3]);
    }
};

// NT: token tiles of 16 per workgroup.  grid (ffn / 16, ceil(T / (16 NT)))
// A wave takes every eighth pair of pieces, 128 bytes of a row: with single pieces dealt out, two waves asked for the halves
// of every cache line.  A pair is in flight (two: d 4096, 16 groups, 5 tokens 33.0 -> 38.0 us for both projections, 128 wide and 8
// groups, 16 tokens 9.6 -> 10.0), and no load stands behind a condition.  (d 616, 13 groups, 36 tokens 13.2 -> 7.4 us, half of it because
// two token tiles to a workgroup, not four, leave no compute unit idle; d 1000, 24 groups, 60 tokens 16.6 -> 16.2, either number of tiles.
// Chunks of 128 elements through LDS, as in the down projection: 4.5 us at the tiny block, but 10 and 21 at these two.)
// ASK, for the few tokens that leave groups unwanted: the first loads wait for the mask bytes, and a compute unit takes one workgroup, so
// that those that leave at once do not pair the others up.  Else the first pair is requested beside the mask bytes.
enum class F32Asks { kAfterMask, kBeside, kAll };                // kAll: no mask, act of every group and token

template <int NT, F32Asks ASKS>
__device__ __forceinline__ void gate_up_f32_block(int tile_x, int tile_y, const float *__restrict__ x, int T, int d, int G, int gs,
                                                  const float *__restrict__ Wg, const float *__restrict__ Wu,
                                                  const uint8_t *__restrict__ mask, float *__restrict__ act, size_t group_stride, int token_stride)
{
    constexpr int W = kGateUpF32Waves;
    __shared__ f32x4_t part[W][2][NT][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = lane & 15, q = lane >> 4;
    constexpr bool kAll = ASKS == F32Asks::kAll;
    const int n0 = tile_x * 16, g = n0 / gs, t0 = tile_y * 16 * NT;
    const uint8_t mine = kAll ? 1 : mask[(size_t)min(t0 + min(lane, 16 * NT - 1), T - 1) * G + g];
    // (descriptors of the workgroup's own rows: the offsets stay small whatever the matrices' sizes)
    const __amdgpu_buffer_rsrc_t bg = buffer_of(Wg + (size_t)n0 * d), bu = buffer_of(Wu + (size_t)n0 * d),
                                 bx = buffer_of(x + (size_t)t0 * d);
    const uint32_t at_w = (uint32_t)(i * d + 4 * q) * 4;
    uint32_t at_x[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) at_x[n] = (uint32_t)(min(16 * n + i, T - 1 - t0) * d + 4 * q) * 4;
    const int np = (d + 15) / 16;                                // pieces of 16; the last one may hold 8
    struct Piece {
        f32x4_t g, u, x[NT];
    };
    auto fetch = [&](Piece &b, int p) {                          // zeros past the end of the row
        const bool ok = p * 16 + 4 * q < d;
        b.g = load4(bg, ok ? at_w : kOutOfRange, p * 64);
        b.u = load4(bu, ok ? at_w : kOutOfRange, p * 64);
#pragma unroll
        for (int n = 0; n < NT; ++n) b.x[n] = load4(bx, ok ? at_x[n] : kOutOfRange, p * 64);
    };
    const bool wanted_by_any = __ballot(mine != 0) != 0ull;      // uniform: the same bytes in every wave
    if (ASKS == F32Asks::kAfterMask && !wanted_by_any) return;
    Piece b[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) fetch(b[k], 2 * wave + k);
    if (ASKS == F32Asks::kBeside && !wanted_by_any) return;
    f32x4_t cg[NT], cu[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) cg[n] = cu[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    PairSum<NT> sg, su;
    for (int p = 2 * wave; p < np; p += 2 * W) {
        sg.clear();
        su.clear();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            sg.add(b[k].g, b[k].x);
            su.add(b[k].u, b[k].x);
            fetch(b[k], p + 2 * W + k);
        }
        sg.fold(cg);
        su.fold(cu);
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
        const f32x4_t g_ = pairwise_sum(pg), u_ = pairwise_sum(pu);
        const int t = t0 + 16 * wave + i;
        const bool wanted = kAll || __shfl(mine, 16 * wave + i) != 0;
        if (t < T) {
            f32x4_t v;
#pragma unroll
            for (int m = 0; m < 4; ++m) v[m] = wanted ? silu_mul(g_[m], u_[m]) : 0.0f;
            *reinterpret_cast<f32x4_t *>(act + g * group_stride + (size_t)t * token_stride + (n0 - g * gs) + 4 * q) = v;
        }
    }
}

template <int NT, bool ASK>
__global__ __launch_bounds__(kGateUpF32Waves * 64) __attribute__((amdgpu_waves_per_eu(2, ASK ? 2 : 8))) void gate_up_f32(
    const float *__restrict__ x, int T, int d, int G, int gs, const float *__restrict__ Wg, const float *__restrict__ Wu,
    const uint8_t *__restrict__ mask, float *__restrict__ act, size_t group_stride, int token_stride)
{
    gate_up_f32_block<NT, ASK ? F32Asks::kAfterMask : F32Asks::kBeside>(blockIdx.x, blockIdx.y, x, T, d, G, gs, Wg, Wu, mask, act,
                                                                        group_stride, token_stride);
}

// The whole pass of a small block in two launches: gate/up of EVERY group beside the first predictor layer, then the down projection,
// whose workgroups work out the masks of their tokens.  Such a pass is a chain of launches that each wait for the one before: prediction,
// gate/up and down of the tiny block take 6.6 + 4.5 + 5.7 us, these two 4.5 + 7.6, a pass 16.1 -> 11.6 us.  Reading the groups that nobody
// keeps costs less than the launches while the weights are few (forward_f32_supported has the line).
// This one: n_gu workgroups of gate/up, 8 G to a range of tokens, then a wave per result of the first layer.  Groups of 128, act [g][t][128].
template <int NT>
__global__ __launch_bounds__(kGateUpF32Waves * 64) void hidden_gate_up_f32(
    const float *__restrict__ x, int T, int d, int G, const float *__restrict__ Wg, const float *__restrict__ Wu, float *__restrict__ act,
    const float *__restrict__ x_pred, const float *__restrict__ At, int r, float *__restrict__ h, int n_gu)
{
    if ((int)blockIdx.x < n_gu) {
        const int n_x = G * 8;                                   // tiles of 16 neurons
        gate_up_f32_block<NT, F32Asks::kAll>(blockIdx.x % n_x, blockIdx.x / n_x, x, T, d, G, 128, Wg, Wu, nullptr, act, (size_t)T * 128, 128);
        return;
    }
    const int lane = threadIdx.x & 63, idx = (blockIdx.x - n_gu) * kGateUpF32Waves + (threadIdx.x >> 6);
    if (idx >= T * r) return;                                    // uniform per wave
    const int t = idx / r, j = idx - t * r;
    const float p = dot_order64(x_pred + (size_t)t * d, At + (size_t)j * d, d, lane);
    if (lane == 0) h[idx] = p > 0.0f ? p : 0.0f;
}

// Groups of 128 neurons, act[g][t][128].  grid (ceil(d / 16), ceil(T / 16)); uses act and Wd of the groups that a token of its own
// range keeps.  A group's 16 rows of Wd are 8 KiB of consecutive bytes and so are its 16 tokens of act: a thread moves one
// 16-byte slot of one of the two per group, four groups go through LDS at a time and four more are on their way; wave w multiplies
// pieces 2 w and 2 w + 1 of the 32.  (In operand order a load was 64 bytes of sixteen rows, and a compute unit's loads took
// several times as long as their bytes: tiny block 7.2 -> 5.8 us, d 504, 20 groups, 25 tokens 18.8 -> 9.9, d 1000, 24 groups, 60
// tokens 22.5 -> 13.2.)  The first eight groups are requested beside the mask bytes and used if the mask says so;
// the rest comes from the list of the other groups that are kept.
constexpr int kTurn = 4, kFirst = 2 * kTurn;

__global__ __launch_bounds__(kDownF32Waves * 64) void down_f32_128(
    const float *__restrict__ act, int T, int d, int G, const float *__restrict__ Wd, const uint8_t *__restrict__ mask,
    float *__restrict__ y)
{
    constexpr int W = kDownF32Waves, gs = 128;
    __shared__ __attribute__((aligned(16))) float stage[kTurn * 2 * 16 * kRowF32];      // [group of the turn][Wd, act][row][kRowF32]
    __shared__ int s_list[1024], s_cnt[W];
    __shared__ unsigned long long s_first;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, q = lane >> 4, half = wave >> 3, row = (tid >> 5) & 15, col = (tid & 31) * 4;
    const int j0 = blockIdx.x * 16, t0 = blockIdx.y * 16, n_tok = min(T - t0, 16);
    // the union of the range's groups: a thread per group (G <= 1024)
    unsigned any = 0;
    if (wave * 64 < G) {                                         // uniform
        uint8_t v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = mask[(size_t)(t0 + min(k, n_tok - 1)) * G + min(tid, G - 1)];
#pragma unroll
        for (int k = 0; k < 16; ++k) any |= v[k];
    }
    const uint32_t voff = half ? (row < n_tok ? (uint32_t)(row * gs + col) * 4 : kOutOfRange) : (uint32_t)(min(row, d - 1 - j0) * gs + col) * 4;
    auto fetch = [&](int g, bool yes) -> f32x4_t {
        const float *p = half ? act + ((size_t)g * T + t0) * gs : Wd + ((size_t)g * d + j0) * gs;
        return load4(buffer_of(p, yes ? 0x7fffffff : 0), voff, 0);
    };
    f32x4_t A[kTurn], B[kTurn];
#pragma unroll
    for (int k = 0; k < kTurn; ++k) A[k] = fetch(min(k, G - 1), k < G);
#pragma unroll
    for (int k = 0; k < kTurn; ++k) B[k] = fetch(min(k + kTurn, G - 1), k + kTurn < G);
    const unsigned long long kept = __ballot(tid < G && any != 0u), rest = wave == 0 ? kept & ~((1ull << kFirst) - 1ull) : kept;
    if (lane == 0) s_cnt[wave] = __popcll(rest);
    if (tid == 0) s_first = kept;
    __syncthreads();
    int before = 0, n_u = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        before += w < wave ? s_cnt[w] : 0;
        n_u += s_cnt[w];
    }
    if ((rest >> lane) & 1ull) s_list[before + __popcll(rest & ((1ull << lane) - 1ull))] = tid;
    const unsigned first = (unsigned)__builtin_amdgcn_readfirstlane((uint32_t)s_first);
    // act of a group that nobody keeps was never written, and its weights are not to be used
#pragma unroll
    for (int k = 0; k < kTurn; ++k) {
        const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
        A[k] = (first >> k) & 1u ? A[k] : zero;
        B[k] = (first >> (k + kTurn)) & 1u ? B[k] : zero;
    }
    f32x4_t c[1] = {f32x4_t{0.f, 0.f, 0.f, 0.f}};
    // turn k takes what b holds, and asks for the groups at positions 4 k .. of the list
    auto turn = [&](f32x4_t (&b)[kTurn], int at) {
#pragma unroll
        for (int k = 0; k < kTurn; ++k) *reinterpret_cast<f32x4_t *>(stage + ((k * 2 + half) * 16 + row) * kRowF32 + col) = b[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kTurn; ++k) {
            const bool yes = at + k < n_u;                       // uniform
            b[k] = fetch(yes ? __builtin_amdgcn_readfirstlane(s_list[at + k]) : 0, yes);
        }
        PairSum<1> sum;
        sum.clear();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int p = 2 * wave + k;
            auto operand = [&](int m) { return *reinterpret_cast<const f32x4_t *>(stage + (((p >> 3) * 2 + m) * 16 + i) * kRowF32 + (p & 7) * 16 + 4 * q); };
            const f32x4_t a[1] = {operand(1)};
            sum.add(operand(0), a);
        }
        sum.fold(c);
        __syncthreads();
    };
    turn(A, 0);
    if (G > kTurn) turn(B, kTurn);
    for (int at = 0; at < n_u; at += kFirst) {
        turn(A, at + kFirst);
        if (at + kTurn < n_u) turn(B, at + kFirst + kTurn);
    }
    f32x4_t *part = reinterpret_cast<f32x4_t *>(stage);
    part[tid] = c[0];
    __syncthreads();
    if (wave == 0) {
        f32x4_t p[W];
#pragma unroll
        for (int w = 0; w < W; ++w) p[w] = part[w * 64 + lane];
        const f32x4_t s = pairwise_sum(p);
        const int t = t0 + i, j = j0 + 4 * q;
        if (t < T && j < d) *reinterpret_cast<f32x4_t *>(y + (size_t)t * d + j) = s;     // (d is a multiple of 8)
    }
}

// ... and this one: the down projection with the mask of its 16 tokens worked out by its 16 waves, up to 32 groups: the second predictor
// layer in the fixed order (same bits as mask_scores_block), a group's rank by comparing its key with all others, a lane per group.  act holds every token's activations
// of every group here, so what a token does not keep is dropped as it is loaded.  The workgroups of the first 16 outputs write the
// prediction's results.
// It adds up as the kernel does that launch_ffn_f32 takes for the shape, so that the pass has the bits of its parts: BY_GROUP as down_f32_128
// (the first eight groups asked for beside the prediction and taken by position), else as down_f32<1> (the groups that are kept, four to a turn,
// a wave's two pieces 16 apart).
struct PredictF32 {
    const float *h, *Bt;
    int r, K, n_dev, share;                                      // share: waves to a row (pair of rows) of Bt
    unsigned long long parts;                                    // four bits a wave: which of them it is
    const int8_t *prio_dev;
    const uint8_t *drop;
    float *scores;
    int32_t *order;
    int8_t *group_dev;
    uint8_t *mask;
    int32_t *surv_idx, *n_surv;
};
// rows, or pairs of them, that a wave of the 16 can take
static int f32_score_slots(int G, int r) { return r <= 256 ? (G + 1) / 2 : G; }

// What the prediction of 16 tokens holds in LDS, in the place of the projection's stages: h padded with zeros to 256 or 512 elements,
// scores and rank keys of up to 32 groups.
struct PredictF32Lds {
    __attribute__((aligned(16))) float h[16 * 512];
    __attribute__((aligned(16))) unsigned long long key[16][32];
    float score[16][32];
};

// Scores and keys of tokens t0 .. + n_tok - 1 (at most 16); called by the whole workgroup of 16 waves.  A row of Bt (up to rank 256: a pair
// of rows, one to each half of the wave, as in mask_scores_block) and four tokens at a time are a wave's share (with a token to every wave,
// from memory, the rows went through the unit's cache 16 times: 3.3 to 6 us more than without a mask to make).  The four tokens' butterflies
// share their first two steps: what two tokens send across a distance is swapped in one exchange, and the partial sums meet as they
// do in xor_add, so the bits are the same (four butterflies of their own: d 816, 20 groups, rank 128, 20 tokens 14.1 us).
// beside(): what else is to be asked for behind the requests here.
template <typename Beside>
__device__ __forceinline__ void scores_f32_block(const PredictF32 &p, int t0, int n_tok, int G, int tid, PredictF32Lds &sh, Beside beside)
{
    constexpr int W = kDownF32Waves, TB = 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r = p.r;
    const bool paired = r <= 256;
    const int pl = paired ? (lane & 31) : lane, half = paired ? (lane >> 5) : 0, n_slots = paired ? (G + 1) / 2 : G;
    // as many waves to a slot as there are, each some of the tokens
    const int part = (int)(p.parts >> (4 * wave)) & 15, slot = wave - part * n_slots, row = paired ? 2 * slot + half : slot;
    const int shift = paired ? 6 : 7, pitch = paired ? 256 : 512;                    // 16-byte pieces of a token's h: 64 or 128
    const __amdgpu_buffer_rsrc_t bh = buffer_of(p.h + (size_t)t0 * r), bb = buffer_of(p.Bt);
    f32x4_t hv[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int idx = tid + k * W * 64, t = idx >> shift, c = (idx - (t << shift)) * 4;
        hv[k] = load4(bh, t < n_tok && c < r ? (uint32_t)(t * r + c) * 4 : kOutOfRange, 0);
    }
    const uint32_t at_row = pl * 8 < r && row < G ? (uint32_t)(row * r + pl * 8) * 4 : kOutOfRange;
    const f32x4_t w0 = load4(bb, at_row, 0), w1 = load4(bb, at_row, 16);
    beside();
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 512) (&sh.key[0][0])[tid] = 0ull;                  // (the pad of an odd number of groups)
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (k == 0 || !paired) reinterpret_cast<f32x4_t *>(sh.h)[tid + k * W * 64] = hv[k];
    __syncthreads();
    for (int t = part * TB; part < p.share && t < n_tok; t += p.share * TB) {        // uniform
        float q[TB];
#pragma unroll
        for (int k = 0; k < TB; ++k) {
            const f32x4_t *hp = reinterpret_cast<const f32x4_t *>(sh.h + (t + k) * pitch + pl * 8);
            const f32x4_t h0 = hp[0], h1 = hp[1];
            q[k] = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[k] = __builtin_fmaf(h0[e], w0[e], q[k]);
#pragma unroll
            for (int e = 0; e < 4; ++e) q[k] = __builtin_fmaf(h1[e], w1[e], q[k]);
        }
        auto as_u = [](float v) { return __builtin_bit_cast(unsigned, v); };
        auto as_f = [](unsigned v) { return __builtin_bit_cast(float, v); };
        float v;
        int k;                                                   // whose sum this lane ends with
        bool writes;
        if (paired) {
            // distance 32: the upper half's partial sums are +0
#pragma unroll
            for (int n = 0; n < TB; ++n) q[n] = q[n] + 0.0f;
            const auto ab = __builtin_amdgcn_permlane16_swap(as_u(q[0]), as_u(q[1]), false, false), cd = __builtin_amdgcn_permlane16_swap(as_u(q[2]), as_u(q[3]), false, false);
            const float s01 = xor_add<8>(as_f(ab[0]) + as_f(ab[1])), s23 = xor_add<8>(as_f(cd[0]) + as_f(cd[1]));
            v = lane & 8 ? s23 : s01;
            k = (lane >> 4 & 1) + (lane & 8 ? 2 : 0);
            writes = (lane & 7) == 0;
        } else {
            const auto ab = __builtin_amdgcn_permlane32_swap(as_u(q[0]), as_u(q[1]), false, false), cd = __builtin_amdgcn_permlane32_swap(as_u(q[2]), as_u(q[3]), false, false);
            const auto m = __builtin_amdgcn_permlane16_swap(as_u(as_f(ab[0]) + as_f(ab[1])), as_u(as_f(cd[0]) + as_f(cd[1])), false, false);
            v = xor_add<8>(as_f(m[0]) + as_f(m[1]));
            k = (lane >> 5) + (lane & 16 ? 2 : 0);
            writes = (lane & 15) == 0;
        }
        v = xor_add<4>(v);
        v = xor_add<2>(v);
        v = xor_add<1>(v);
        if (writes && row < G && t + k < n_tok) {
            sh.score[t + k][row] = v;
            sh.key[t + k][row] = rank_key(v, row);
        }
    }
    __syncthreads();
}

// The groups that token t keeps, from the keys in LDS; called by a whole wave, whose halves share the comparisons: lane g and lane g + 32 are
// group g's.
__device__ __forceinline__ uint32_t token_mask_32(const PredictF32 &p, int t, int G, int lane, const unsigned long long *keys, float score, int8_t prio,
                                                  uint8_t lost, bool write)
{
    const int g = lane & 31, n2 = (G + 1) / 2;
    const unsigned long long key = keys[g];
    const ulonglong2 *k2 = reinterpret_cast<const ulonglong2 *>(keys);
    int pos = 0;                                                 // groups that come before this lane's
    for (int o = 0; o < n2; o += 4) {                            // (keys past the groups are 0 and come before none)
        const ulonglong2 a = k2[o + (lane >> 5)], b = k2[o + 2 + (lane >> 5)];
        pos += (a.x > key ? 1 : 0) + (a.y > key ? 1 : 0) + (b.x > key ? 1 : 0) + (b.y > key ? 1 : 0);
    }
    pos += __shfl_xor(pos, 32);
    const int planned = __shfl((int)prio, min(pos, 63));         // (all lanes take part: the bytes lie in each of them)
    const int dev = lane < G && pos < p.K && planned >= 0 && planned < p.n_dev ? planned : -1;      // malformed entry: not executed
    const int gone = __shfl((int)lost, max(dev, 0));
    const bool keep = dev >= 0 && gone == 0;
    const uint32_t kept = (uint32_t)__ballot(keep);              // (G <= 32)
    if (write && lane < G) {
        const size_t at = (size_t)t * G + lane;
        p.scores[at] = score;
        if (p.order) p.order[(size_t)t * G + pos] = lane;
        if (p.group_dev) p.group_dev[at] = (int8_t)dev;
        p.mask[at] = keep ? 1 : 0;
        const int total = __popc(kept);
        if (p.surv_idx) {
            if (keep) p.surv_idx[(size_t)t * p.K + __popc(kept & ((1u << lane) - 1u))] = lane;
            if (lane >= total && lane < p.K) p.surv_idx[(size_t)t * p.K + lane] = -1;
        }
        if (p.n_surv && lane == 0) p.n_surv[t] = total;
    }
    return kept;
}

template <bool BY_GROUP>
__global__ __launch_bounds__(kDownF32Waves * 64) void predict_down_f32(const float *__restrict__ act, int T, int d, int G,
                                                                       const float *__restrict__ Wd, float *__restrict__ y, PredictF32 pr)
{
    constexpr int W = kDownF32Waves, gs = 128;
    __shared__ __attribute__((aligned(16))) float stage[kTurn * 2 * 16 * kRowF32];
    static_assert(sizeof(PredictF32Lds) <= sizeof(stage), "the prediction comes before the stages");
    __shared__ uint32_t s_kept[W];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, q = lane >> 4, half = wave >> 3, row = (tid >> 5) & 15, col = (tid & 31) * 4;
    const int j0 = blockIdx.x * 16, t0 = blockIdx.y * 16, n_tok = min(T - t0, 16);
    const uint32_t voff = half ? (row < n_tok ? (uint32_t)(row * gs + col) * 4 : kOutOfRange) : (uint32_t)(min(row, d - 1 - j0) * gs + col) * 4;
    auto fetch = [&](int g, bool yes) -> f32x4_t {
        const float *p = half ? act + ((size_t)g * T + t0) * gs : Wd + ((size_t)g * d + j0) * gs;
        return load4(buffer_of(p, yes ? 0x7fffffff : 0), voff, 0);
    };
    // schedule and loss outcomes, a byte per lane
    const int t = t0 + min(wave, n_tok - 1);
    const int8_t prio = pr.K > 0 ? pr.prio_dev[min(lane, pr.K - 1)] : (int8_t)-1;
    const uint8_t lost = pr.drop ? pr.drop[(size_t)t * pr.n_dev + min(lane, pr.n_dev - 1)] : (uint8_t)0;
    PredictF32Lds &sh = *reinterpret_cast<PredictF32Lds *>(stage);
    f32x4_t A[kTurn], B[kTurn];
    scores_f32_block(pr, t0, n_tok, G, tid, sh, [&]() __attribute__((always_inline)) {
        if (!BY_GROUP) return;
#pragma unroll
        for (int k = 0; k < kTurn; ++k) A[k] = fetch(min(k, G - 1), k < G);
#pragma unroll
        for (int k = 0; k < kTurn; ++k) B[k] = fetch(min(k + kTurn, G - 1), k + kTurn < G);
    });
    const uint32_t own = wave < n_tok ? token_mask_32(pr, t, G, lane, sh.key[wave], sh.score[wave][lane & 31], prio, lost, blockIdx.x == 0) : 0u;
    if (lane == 0) s_kept[wave] = own;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) any |= s_kept[w];
    any = (uint32_t)__builtin_amdgcn_readfirstlane((int)any);
    const uint32_t mine = half ? s_kept[row] : any;              // the groups whose values this thread may use
    uint32_t rest = BY_GROUP ? any & ~((1u << kFirst) - 1u) : any;                   // not asked for yet
    f32x4_t c[1] = {f32x4_t{0.f, 0.f, 0.f, 0.f}};
    int ga[kTurn], gb[kTurn];                                    // the groups that A and B hold, -1: none
    auto ask = [&](f32x4_t (&b)[kTurn], int (&gk)[kTurn]) {
#pragma unroll
        for (int k = 0; k < kTurn; ++k) {
            const bool yes = rest != 0u;                         // uniform
            gk[k] = yes ? __builtin_ctz(rest) : -1;
            rest &= rest - 1u;                                   // (0 stays 0)
            b[k] = fetch(yes ? gk[k] : 0, yes);
        }
    };
    if (BY_GROUP) {
#pragma unroll
        for (int k = 0; k < kTurn; ++k) {
            ga[k] = k < G ? k : -1;
            gb[k] = k + kTurn < G ? k + kTurn : -1;
        }
    } else {
        ask(A, ga);
        ask(B, gb);
    }
    auto turn = [&](f32x4_t (&b)[kTurn], int (&gk)[kTurn]) {
#pragma unroll
        for (int k = 0; k < kTurn; ++k)
            *reinterpret_cast<f32x4_t *>(stage + ((k * 2 + half) * 16 + row) * kRowF32 + col) =
                gk[k] >= 0 && ((mine >> gk[k]) & 1u) ? b[k] : f32x4_t{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
        ask(b, gk);
        PairSum<1> sum;
        sum.clear();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int p = BY_GROUP ? 2 * wave + k : wave + W * k;
            auto operand = [&](int m) { return *reinterpret_cast<const f32x4_t *>(stage + (((p >> 3) * 2 + m) * 16 + i) * kRowF32 + (p & 7) * 16 + 4 * q); };
            const f32x4_t a[1] = {operand(1)};
            sum.add(operand(0), a);
        }
        sum.fold(c);
        __syncthreads();
    };
    if (BY_GROUP) {
        turn(A, ga);
        if (G > kTurn) turn(B, gb);
    }
    while (ga[0] >= 0) {
        turn(A, ga);
        if (gb[0] >= 0) turn(B, gb);
    }
    f32x4_t *part = reinterpret_cast<f32x4_t *>(stage);
    part[tid] = c[0];
    __syncthreads();
    if (wave == 0) {
        f32x4_t p[W];
#pragma unroll
        for (int w = 0; w < W; ++w) p[w] = part[w * 64 + lane];
        const f32x4_t s = pairwise_sum(p);
        const int ty = t0 + i, j = j0 + 4 * q;
        if (ty < T && j < d) *reinterpret_cast<f32x4_t *>(y + (size_t)ty * d + j) = s;     // (d is a multiple of 8)
    }
}

// Groups of any multiple of 16 neurons, and of 128 where that is the better one (see launch_ffn_f32), act[t][ffn].  grid (ceil(d / 16), ceil(T / (16 NT))); reads act of the groups that a token of its own range keeps
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
    f32x4_t bs[NT][4];                                           // as in PairSum
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
// (offsets within a workgroup's rows have 32 bits)
bool f32_path_supported(int d, int gs) { return gs % 16 == 0 && d <= 1 << 22; }

template <int NT, bool ASK = false>
static void launch_gate_up(const float *x, int T, int d, int G, int gs, const float *Wg, const float *Wu,
                           const uint8_t *mask, float *act, bool by_group, hipStream_t s)
{
    const int ffn = G * gs;
    launch_timed("gate_up_f32", gate_up_f32<NT, ASK>, dim3(ffn / 16, (T + 16 * NT - 1) / (16 * NT)), dim3(kGateUpF32Waves * 64), s,
                 x, T, d, G, gs, Wg, Wu, mask, act, by_group ? (size_t)T * gs : (size_t)gs, by_group ? gs : ffn);
}

template <int NT>
static void launch_down(const float *act, int T, int d, int G, int gs, const float *Wd, const uint8_t *mask, float *y,
                        hipStream_t s)
{
    down_f32<NT><<<dim3((d + 15) / 16, (T + 16 * NT - 1) / (16 * NT)), dim3(kDownF32Waves * 64), 0, s>>>(act, G * gs, T, d, G,
                                                                                                   gs, Wd, mask, y);
}

// The weights are read once per range of tokens (from L2 after the first).  A range of down lies within one of gate/up, so the
// groups it walks have been written.  nt: token tiles of a workgroup in gate/up.
static hipError_t launch_blocks(const float *x, int T, int d, int G, int gs, const float *Wg, const float *Wu, const float *Wd,
                                const uint8_t *mask, float *y, float *act, int nt, bool ask, bool by_group, hipStream_t s)
{
    if (ask)
        launch_gate_up<1, true>(x, T, d, G, gs, Wg, Wu, mask, act, by_group, s);
    else if (nt == 1)
        launch_gate_up<1>(x, T, d, G, gs, Wg, Wu, mask, act, by_group, s);
    else if (nt == 2)
        launch_gate_up<2>(x, T, d, G, gs, Wg, Wu, mask, act, by_group, s);
    else
        launch_gate_up<4>(x, T, d, G, gs, Wg, Wu, mask, act, by_group, s);
    if (by_group)
        down_f32_128<<<dim3((d + 15) / 16, (T + 15) / 16), dim3(kDownF32Waves * 64), 0, s>>>(act, T, d, G, Wd, mask, y);
    else if (nt == 1)
        launch_down<1>(act, T, d, G, gs, Wd, mask, y, s);
    else
        launch_down<2>(act, T, d, G, gs, Wd, mask, y, s);
    return hipGetLastError();
}

// Up to five tokens leave groups unwanted, and what is asked for before the mask is known is wasted: both projections, groups of
// 128, half of them kept, us, asked for at once / after the mask: one token, d 256, 8 groups 10.3 / 8.4, d 1000, 24 groups 17.4 / 14.8,
// d 2048, 44 groups 37.9 / 25.3, d 8192, 64 groups 126 / 109; four tokens 10.8 / 10.2, 21.5 / 20.5, 46.4 / 43.5, 156 / 152.
static bool ask_after_mask(int T) { return T <= 5; }

// down_f32_128 asks for its first eight groups at once (up to eight groups it pays from nine tokens on: 128 wide, three tenths kept,
// five tokens 9.6 against 8.8 us, eight 9.5 / 9.6), and reads Wd once per 16 tokens, down_f32 once per 32: of many tokens it takes those
// that give no compute unit more than one workgroup (d 1000, 24 groups, 64 tokens 34 against 43 us, 128 57 / 55, 512 176 / 168;
// d 256, 8 groups, 256 tokens 14.3 / 17.4, 512 25.0 / 24.2; d 4096, 86 groups, 512 tokens 2299 / 2181).
static bool down_by_group(int T, int d, int G, int gs)
{
    return gs == 128 && !ask_after_mask(T) && (G > 8 || T > 8) && (T <= 64 || (long long)((d + 15) / 16) * ((T + 15) / 16) <= 256);
}

hipError_t launch_ffn_f32(const float *x, int T, int d, int G, int gs, const float *Wg, const float *Wu, const float *Wd,
                          const uint8_t *mask, float *y, float *act, hipStream_t s)
{
    // four token tiles to a workgroup read the weights least often, two where four would leave compute units without one
    const int nt = T <= 16 ? 1 : T <= 32 || (long long)((T + 63) / 64) * (G * gs / 16) < 256 ? 2 : 4;
    const bool ask = ask_after_mask(T), by_group = down_by_group(T, d, G, gs);
    constexpr int kRun = 1 << 20;                                // ranges of tokens are a grid's y, which ends at 65535
    for (int t0 = 0;; t0 += kRun) {
        const size_t t = (size_t)t0;
        const hipError_t e = launch_blocks(x + t * d, T - t0 < kRun ? T - t0 : kRun, d, G, gs, Wg, Wu, Wd, mask + t * G, y + t * d,
                                           act + t * G * gs, nt, ask, by_group, s);
        if (e != hipSuccess || T - t0 <= kRun) return e;
    }
}

// Whole pass in two launches, see hidden_gate_up_f32, against three or four, us in a graph of blocks, one block over and over, and (in brackets)
// blocks of 1.2 GB in all, whose weights come from HBM.  One group kept, the least there is to read, rank 256: d 1024, 24 groups, 1, 3, 4, 16 tokens
// 15.9 / 12.5 (16.6 / 15.6), 17.0 / 13.5 (17.8 / 16.5), 16.9 / 13.6 (18.6 / 16.7), 22.7 / 20.3 (25.9 / 24.3); d 1024, 32 groups 15.9 / 13.9 (16.8 /
// 17.9), 16.8 / 14.4 (17.8 / 17.9), 17.5 / 15.0 (18.4 / 18.0), 23.0 / 20.9 (26.7 / 26.0).  Half of the groups kept: d 1024, 24 groups 18.2 / 15.4
// (21.9 / 18.7), 21.7 / 18.8 (25.2 / 22.6), 23.4 / 19.1 (26.3 / 23.1), 26.2 / 22.7 (29.4 / 27.1); d 256, 8 groups, 1 and 16 tokens 13.6 / 9.3 (15.2 /
// 10.9), 15.7 / 11.0 (18.1 / 13.0).  Above the line d 2048, 32 groups, one group kept, 1, 4, 16 tokens 19.8 / 21.0 (21.6 / 24.8), 21.3 / 20.4 (23.6 /
// 25.3), 29.0 / 27.3 (32.5 / 32.4).  So the weights of all groups may be 24 Ki rows of 128 elements, 32 Ki from four tokens on, whatever share of the
// groups is kept.  64 tokens are still ahead (d 256, 12 groups 18.4 / 14.0 (20.3 / 15.5), d 1024, 24 groups, one kept 37.1 / 31.3 (39.8 / 33.7), d
// 2048, 8 groups 34.9 / 31.8 (38.2 / 35.6)); above, it depends on what is kept and on the rank (d 512, 24 groups, rank 256, 112 tokens 27.0 / 31.7
// with one group kept, 37.9 / 34.9 with seven; d 256, 8 groups, rank 512, 112 tokens 23.1 / 24.3).  Rows of up to 4096 (8 groups of them, rank 512,
// 1, 4, 16, 64 tokens 27.9 / 25.6 (32.9 / 29.4), 32.0 / 28.5 (35.4 / 33.0), 44.2 / 38.5 (47.0 / 47.3), 86.4 / 77.2 (90.8 / 80.3)); longer ones lose
// where their weights are not cached: d 8192, 4 groups, rank 512, 4 and 16 tokens 54.5 / 51.9 (58.3 / 60.1), 73.5 / 67.3 (77.5 / 84.9); 3 groups,
// rank 64, 32 tokens 83.2 / 82.8 (91.7 / 97.2); d 16384, 2 groups, rank 256, 16 tokens 119.1 / 119.9 (124.5 / 154.2).
bool forward_f32_supported(int T, int d, int G, int gs, int r, int n_dev)
{
    return gs == 128 && r <= 512 && f32_score_slots(G, r) <= kDownF32Waves && n_dev <= 64 && T <= 64 && d <= 4096 &&
           G * d <= (T < 4 ? 24 : 32) * 1024;
}

template <int NT>
static void launch_hidden_gate_up(const float *x, const float *x_pred, int T, int d, int r, int G, const float *At, const float *Wg,
                                  const float *Wu, float *h, float *act, hipStream_t s)
{
    const int n_gu = G * 8 * ((T + 16 * NT - 1) / (16 * NT)), n_hid = (T * r + kGateUpF32Waves - 1) / kGateUpF32Waves;
    launch_timed("hidden_gate_up_f32", hidden_gate_up_f32<NT>, dim3(n_gu + n_hid), dim3(kGateUpF32Waves * 64), s, x, T, d, G, Wg, Wu, act, x_pred, At, r, h, n_gu);
}

hipError_t launch_forward_f32(const float *x, const float *x_pred, int T, int d, int r, int G, const float *At, const float *Bt,
                              const float *Wg, const float *Wu, const float *Wd, float *h, float *act, float *scores, int K,
                              const int8_t *prio_dev, int n_dev, const uint8_t *drop, float *y, int32_t *order, int8_t *group_dev,
                              uint8_t *mask, int32_t *surv_idx, int32_t *n_surv, hipStream_t s)
{
    if (T <= 16)
        launch_hidden_gate_up<1>(x, x_pred, T, d, r, G, At, Wg, Wu, h, act, s);
    else
        launch_hidden_gate_up<2>(x, x_pred, T, d, r, G, At, Wg, Wu, h, act, s);
    const int slots = f32_score_slots(G, r), share = kDownF32Waves / slots;
    unsigned long long parts = 0;
    for (int w = 0; w < kDownF32Waves; ++w) parts |= (unsigned long long)(w / slots) << (4 * w);
    const PredictF32 pr{h, Bt, r, K, n_dev, share, parts, prio_dev, drop, scores, order, group_dev, mask, surv_idx, n_surv};
    const dim3 grid((d + 15) / 16, (T + 15) / 16), block(kDownF32Waves * 64);
    if (down_by_group(T, d, G, 128))
        predict_down_f32<true><<<grid, block, 0, s>>>(act, T, d, G, Wd, y, pr);
    else                                                         // (at most eight tokens)
        predict_down_f32<false><<<grid, block, 0, s>>>(act, T, d, G, Wd, y, pr);
    return hipGetLastError();
}

}  // namespace halo
