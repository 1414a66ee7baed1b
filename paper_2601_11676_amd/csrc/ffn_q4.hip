// Group-sparse SwiGLU FFN over 4-bit block-quantised weights (paper Sec. V-A: the evaluated
// models are quantised to 4-bit integers; Sec. II-A neuron groups, merge = sum).
//
// Storage format (the library's own; the paper fixes none): blocks of 128 consecutive elements
// along the reduction dimension share one bf16 scale s, an element is s * (c - 8) with a
// 4-bit code c.  Eight codes per 32-bit word: element 2i of the eight in bits [4i, 4i+3],
// element 2i+1 in bits [16+4i, 16+4i+3], so that (word >> 4i) & 0x000F000F holds the
// pair (2i, 2i+1) in the two halves of a register -- the shape of a packed bf16 pair.
//   gate/up : codes [ffn][d/8] words, scales [ffn][d/128]        (blocks along d)
//   down    : codes [G][d][gs/8] words, scales [G][d], gs = 128  (block = the group's neurons)
//
// One token (the hot path): a quarter of the bf16 bytes per group, so the kernels are built
// like the bf16 ones -- stream every surviving byte once with 16-byte loads -- and the
// arithmetic stays far below the memory time: or-ing 0x4300 over a code gives the bf16 value
// 128 + c exactly, the packed dot instruction multiplies two of those with two activations,
// and the constant offset is taken out once per 32 elements: sum (c-8) x = sum (128+c) x -
// 136 sum x.  Shapes that no tuned path takes go through plain kernels that dequantise element by element.
#include "kernels.hpp"
#include "mask_device.hpp"
#include "mask_words.hpp"
#include "q4_codes.hpp"
#include "row_stream.hpp"

namespace halo {

// sum over the 32 elements of one 16-byte code piece of (128 + c) * x, x as 16 packed bf16 pairs
__device__ __forceinline__ float q4_dot32(const u32x4 &c, const u32x4 (&x)[4])
{
    float a0 = 0.0f, a1 = 0.0f;
    const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a0 = dot2_bf16(q4_pair(w[j], 0), x[j].x, a0);
        a1 = dot2_bf16(q4_pair(w[j], 1), x[j].y, a1);
        a0 = dot2_bf16(q4_pair(w[j], 2), x[j].z, a0);
        a1 = dot2_bf16(q4_pair(w[j], 3), x[j].w, a1);
    }
    return a0 + a1;
}

// sum of 32 bf16 values held as 16 packed pairs
__device__ __forceinline__ float sum32(const u32x4 (&x)[4])
{
    float a = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a = dot2_bf16(0x3F803F80u, x[j].x, a);
        a = dot2_bf16(0x3F803F80u, x[j].y, a);
        a = dot2_bf16(0x3F803F80u, x[j].z, a);
        a = dot2_bf16(0x3F803F80u, x[j].w, a);
    }
    return a;
}

// ---------------------------------------------------------------------------
// one token, bf16 activations, d <= NH * 2048, group size 128, G <= 256
// ---------------------------------------------------------------------------
// gate/up: one wave per neuron at a time, NB neurons requested together.  A lane owns the 32
// elements 2048 h + 32 lane .. + 31 of every part h of the row: one 16-byte code piece per matrix row and
// part, one scale (block 16 h + lane / 4), and the matching 64 bytes of x kept in registers.
// Eight waves per workgroup, two per SIMD: unpacking the codes costs about three vector
// instructions per two weights, which is not negligible beside the memory time of a quarter
// of the bf16 bytes, so one wave's arithmetic has to overlap another's memory wait.
// WHOLE: rows of exactly NH * 2048 elements, activation in bf16.  Otherwise any multiple of 128 above
// (NH - 1) * 2048: lanes whose piece of the last part lies past the end read the row's first piece against zeros,
// and the activation stays in float32, as in the plain path that served these lengths (13B shape: gate/up
// 11.5 us and down 9.0 us per launch; the plain path took 19.7 and 44, and three more launches).
constexpr int kQ4GateUpThreads = 512;
constexpr int kQ4GateUpBlocks = 256;      // workgroups that do gate/up work (one per compute unit)

// a predictor row beside such a row: its 16-byte pieces as RowLanes deals them
template <int NH, bool WHOLE>
__device__ __forceinline__ void q4_pred_row(const bf16_t *__restrict__ x_next, const bf16_t *__restrict__ At_next,
                                            float *__restrict__ h_next, int d, int j, int lane)
{
    float p;
    if (WHOLE || d > (NH * 4 - 2) * 512) {                       // uniform
        const RowLanes<NH * 4, !WHOLE> rl(d, lane);
        p = dot_order64_row<NH * 4, !WHOLE>(x_next, At_next + rl.row(j), rl, lane);
    } else {
        const RowLanes<NH * 4 - 2, true> rl(d, lane);
        p = dot_order64_row<NH * 4 - 2, true>(x_next, At_next + rl.row(j), rl, lane);
    }
    if (lane == 0) h_next[j] = p > 0.0f ? p : 0.0f;
}

template <int NH, bool WHOLE, typename AT>
__global__ __launch_bounds__(kQ4GateUpThreads, (NH <= 2 ? 4 : 2)) void gate_up_q4_t1(
    const bf16_t *__restrict__ x, int G, const uint32_t *__restrict__ Gq, const bf16_t *__restrict__ Gs,
    const uint32_t *__restrict__ Uq, const bf16_t *__restrict__ Us, const uint8_t *__restrict__ mask,
    AT *__restrict__ act, const bf16_t *__restrict__ x_next, const bf16_t *__restrict__ At_next, int r,
    float *__restrict__ h_next, int n_pred, int pred_rows, int len)
{
    constexpr int gs = 128, NB = NH <= 2 ? 3 : 2, WPB = kQ4GateUpThreads / 64;
    const int d = WHOLE ? NH * 2048 : len;
    const int kWords = d / 8, kBlocks = d / kQ4Block;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // pred_rows > 0 (then n_pred == 0): the predictor's rows are dealt evenly, pred_rows of them to the last
    // waves of every workgroup, row vblock + 256 k to wave 7 - k.  A row of At is as many bytes as two
    // neurons' codes, and a workgroup of predictor rows alone carried three quarters more bytes than its
    // neighbours' share of the codes: the compute units that held one finished 2 us after the others.
    if (pred_rows > 0 && wave >= WPB - pred_rows)
        q4_pred_row<NH, WHOLE>(x_next, At_next, h_next, d, blockIdx.x + kQ4GateUpBlocks * (WPB - 1 - wave), lane);
    if ((int)blockIdx.x < n_pred) {
        // the first predictor layer of the NEXT block rides along (paper Sec. III-B.3, Pred beside
        // Load/Comp, one layer ahead): one row of At per wave, h_next = ReLU(x_next A)
        const int j = blockIdx.x * WPB + wave;
        if (j < r) q4_pred_row<NH, WHOLE>(x_next, At_next, h_next, d, j, lane);
        return;
    }
    const MaskWords mw = load_mask_words(mask, G, lane);
    // contiguous runs of the surviving neurons, wave by wave (lengths differ by at most one);
    // kQ4GateUpBlocks * WPB is a power of two, and a run is far shorter than a group, so it
    // touches at most two groups: the group ids are looked up twice, not once per neuron
    constexpr int nw = kQ4GateUpBlocks * WPB;
    const int total = mw.count * gs, w = (blockIdx.x - n_pred) * WPB + wave;
    int n0 = (int)((unsigned)total * (unsigned)w / nw), n1 = (int)((unsigned)total * (unsigned)(w + 1) / nw);
    const unsigned units = (unsigned)total + 2u * (unsigned)(pred_rows * kQ4GateUpBlocks);   // a row of At = two neurons
    if (pred_rows > 0 && units >= 2u * nw) {
        // runs cut by weight: a wave that has just done a predictor row gets two neurons fewer
        auto cut = [&](int ww) {
            const int v = ww / WPB, k = ww % WPB;
            const int rows_before = v * pred_rows + (k > WPB - pred_rows ? k - (WPB - pred_rows) : 0);
            return (int)(units * (unsigned)ww / nw) - 2 * rows_before;
        };
        n0 = cut(w);
        n1 = cut(w + 1);
    }
    if (n0 >= n1) return;
    const int u_first = n0 / gs, u_last = (n1 - 1) / gs;
    const int g_first = nth_group(mw, u_first, lane), g_last = nth_group(mw, u_last, lane);
    // this lane's piece of the last part of a row: in words from the row's start, and its scale
    const bool tail_ok = WHOLE || (NH - 1) * 2048 + lane * 32 < d;
    const int tail_word = tail_ok ? (NH - 1) * 256 + lane * 4 : 0, tail_block = tail_ok ? (NH - 1) * 16 + (lane >> 2) : 0;
    u32x4 xr[NH][4];
    float xs[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool tail = !WHOLE && h == NH - 1;
            xr[h][j] = *reinterpret_cast<const u32x4 *>(x + (tail ? tail_word * 8 : h * 2048 + lane * 32) + j * 8);
            if (tail && !tail_ok) xr[h][j] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    for (int nb = n0; nb < n1; nb += NB) {
        u32x4 cg[NB][NH], cu[NB][NH];
        uint16_t sg[NB][NH], su[NB][NH];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int n = nb + i < n1 ? nb + i : n1 - 1;            // past the end: an in-range duplicate
            const int u = n / gs;
            const size_t row = (size_t)(u == u_first ? g_first : g_last) * gs + (n - u * gs);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const bool tail = !WHOLE && h == NH - 1;
                const int word = tail ? tail_word : h * 256 + lane * 4, block = tail ? tail_block : h * 16 + (lane >> 2);
                cg[i][h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(Gq + row * kWords + word));
                cu[i][h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(Uq + row * kWords + word));
                sg[i][h] = Gs[row * kBlocks + block];
                su[i][h] = Us[row * kBlocks + block];
            }
        }
        if (nb == n0) {
#pragma unroll
            for (int h = 0; h < NH; ++h) xs[h] = 136.0f * sum32(xr[h]);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if (nb + i >= n1) break;                                // uniform: duplicates cost no arithmetic
            float ag = 0.0f, au = 0.0f;
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                ag = __builtin_fmaf(bf16_bits_to_float(sg[i][h]), q4_dot32(cg[i][h], xr[h]) - xs[h], ag);
                au = __builtin_fmaf(bf16_bits_to_float(su[i][h]), q4_dot32(cu[i][h], xr[h]) - xs[h], au);
            }
            ag = wave_sum_fast(ag);
            au = wave_sum_fast(au);
            const float v = WHOLE ? silu_mul_fast(ag, au) : silu_mul(ag, au);
            if (lane == 0) store_out(act + nb + i, v);
        }
    }
}

// down: four lanes share an output row j (16 bytes each = 32 of the group's 128 neurons), a
// wave covers 16 consecutive rows = 1 KiB of a group's codes, the workgroup's eight waves take
// every eighth surviving group and meet in LDS.  All of a wave's groups (up to eight at a time) are requested
// together: the codes and the rows' scales, and beside them the activations that face them, coalesced, which the
// wave then parks in LDS for itself -- no barrier stands between the mask and the codes -- and reads back in
// operand order.  What bounds it is the chain mask -> group ids -> codes -> sums, so it is built for few
// requests and one memory round trip per eight groups: with the activations fetched straight into every lane
// (four more requests per group, two batches of four groups, group ids from a search per group) it took 6.8 us per
// launch at the 7B shape, now 5.9; the same form in float32 at the 13B shape 30 us, now 9.0.
// AT: bf16, or float for row lengths other than 4096 and 8192.
constexpr int kDownQ4Batch = 8;

struct DownQ4Shared {
    float part[8][16];
};

// the 32 activations at LDS address a (bytes) against a lane's 32 codes: sum (c - 8) a.  The offset's sum comes from
// two of the 32 per lane, added over the 16 lanes (same lane % 4) that face the same 32.
__device__ __forceinline__ float q4_down_dot(const u32x4 &c, const bf16_t *a, int lane)
{
    u32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const u32x4 *>(a + k * 8);
    float sum = dot2_bf16(0x3F803F80u, *reinterpret_cast<const uint32_t *>(a + (lane >> 2) * 2), 0.0f);
    sum = xor_add<4>(sum);
    sum = xor_add<8>(sum);
    sum = xor_add<16>(sum);
    sum = xor_add<32>(sum);
    return q4_dot32(c, v) - 136.0f * sum;
}
__device__ __forceinline__ float q4_down_dot(const u32x4 &c, const float *a, int lane)
{
    const float2 own = *reinterpret_cast<const float2 *>(a + (lane >> 2) * 2);
    float sum = own.x + own.y;
    sum = xor_add<4>(sum);
    sum = xor_add<8>(sum);
    sum = xor_add<16>(sum);
    sum = xor_add<32>(sum);
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float4 v = *reinterpret_cast<const float4 *>(a + j * 4);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            // elements 4 j + 2 i and 4 j + 2 i + 1 as 128 + c
            const uint32_t pair = q4_pair(w[j >> 1], 2 * (j & 1) + i);
            acc[2 * i] = __builtin_fmaf(bf16_lo(pair), i ? v.z : v.x, acc[2 * i]);
            acc[2 * i + 1] = __builtin_fmaf(bf16_hi(pair), i ? v.w : v.y, acc[2 * i + 1]);
        }
    }
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) - 136.0f * sum;
}

// With ahead != 0 workgroup 0 is the mask workgroup of the NEXT block (second predictor layer,
// ranking, mask); it is dispatched first because it is the longest dependent chain.  A
// workgroup is one or the other, so the two LDS layouts share their bytes and two workgroups
// fit a compute unit (the mask workgroup must run beside a down-projection one, not after).
template <typename AT>
__global__ __launch_bounds__(512, 4) void down_q4_t1(int d, int G, const uint32_t *__restrict__ Dq,
                                                      const bf16_t *__restrict__ Ds,
                                                      const uint8_t *__restrict__ mask,
                                                      const AT *__restrict__ act, bf16_t *__restrict__ y,
                                                      int ahead, AheadDev nx)
{
    constexpr int gs = 128, kB = kDownQ4Batch;
    constexpr int kPer = 1024 / (gs * sizeof(AT)), kLoads = kB / kPer;     // groups per activation load, loads per batch
    constexpr size_t kActBytes = kB * gs * sizeof(AT);                     // a wave's activations of a batch
    constexpr size_t kProj = sizeof(DownQ4Shared) + 8 * kActBytes;
    constexpr size_t kLds = kProj > sizeof(MaskShared) ? kProj : sizeof(MaskShared);
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    if (ahead && blockIdx.x == 0) {
        mask_scores_block<512, bf16_t, true>(*reinterpret_cast<MaskShared *>(lds), tid, nx.h, nx.Bt, nx.r,
                                             nx.scores, G, nx.K, nx.prio_dev, nx.n_dev, nx.drop, nx.order,
                                             nx.group_dev, nx.mask, nx.surv_idx, nx.n_surv);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    DownQ4Shared &sh = *reinterpret_cast<DownQ4Shared *>(lds);
    AT *mine = reinterpret_cast<AT *>(lds + sizeof(DownQ4Shared) + wave * kActBytes);
    const int vblock = blockIdx.x - (ahead ? 1 : 0);
    const MaskWords mw = load_mask_words(mask, G, lane);
    // this wave's groups: positions wave, wave + 8, ... of the surviving list, at most 32 of them, one to a lane.
    // A lane that holds a surviving group knows its position and hands the group to lane position / 8 of this wave
    // if it is one of the wave's; the others hand theirs to lane 63, which nobody asks.
    int my_group = 0;
    {
        int base = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int pos = base + __popcll(mw.w[k] & ((1ull << lane) - 1ull));
            const bool ours = ((mw.w[k] >> lane) & 1ull) && (pos & 7) == wave;
            my_group |= __builtin_amdgcn_ds_permute((ours ? pos >> 3 : 63) * 4, ours ? k * kWave + lane : 0);
            base += __popcll(mw.w[k]);
        }
    }
    const int slots = (mw.count - wave + 7) >> 3;
    const int j = vblock * 16 + (lane >> 2);                       // output row of this lane
    const int p = lane & 3;                                        // which 32 neurons of the group
    float acc = 0.0f;
    const size_t gwords = (size_t)d * 16;                          // words per group
    for (int s0 = 0; s0 < slots; s0 += kB) {                       // uniform
        u32x4 c[kB], a[kLoads];
        uint16_t s[kB];
#pragma unroll
        for (int q = 0; q < kB; ++q) {
            if (s0 + q < slots) {
                const int g = __builtin_amdgcn_readlane(my_group, s0 + q);
                c[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(Dq + g * gwords + (size_t)j * 16) + p);
                s[q] = Ds[(size_t)g * d + j];
            }
        }
        // activation load n: groups s0 + n kPer .. of the wave, 16 bytes a lane (past the last one: repeats it)
        constexpr int kLanes = kWave / kPer;
#pragma unroll
        for (int n = 0; n < kLoads; ++n)
            if (s0 + n * kPer < slots) {
                const int u = wave + 8 * min(s0 + n * kPer + lane / kLanes, slots - 1);
                a[n] = *reinterpret_cast<const u32x4 *>(act + u * gs + (lane % kLanes) * (16 / (int)sizeof(AT)));
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < kLoads; ++n)
            if (s0 + n * kPer < slots) *reinterpret_cast<u32x4 *>(reinterpret_cast<unsigned char *>(mine) + n * 1024 + lane * 16) = a[n];
        // (the region is the wave's own, and a wave's LDS operations complete in order)
#pragma unroll
        for (int q = 0; q < kB; ++q) {
            if (s0 + q < slots) acc = __builtin_fmaf(bf16_bits_to_float(s[q]), q4_down_dot(c[q], mine + q * gs + p * 32, lane), acc);
        }
    }
    // the four lanes of a row, then the eight waves
    acc = dpp_add<0xB1>(acc);
    acc = dpp_add<0x4E>(acc);
    if (p == 0) sh.part[wave][lane >> 2] = acc;
    __syncthreads();
    if (wave == 0 && lane < 16) {
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) v += sh.part[k][lane];
        y[vblock * 16 + lane] = f32_to_bf16(v);
    }
}

// ---------------------------------------------------------------------------
// generic (any T, f32 or bf16 activations): dequantise element by element
// ---------------------------------------------------------------------------
__device__ __forceinline__ void q4_unpack8(uint32_t w, float s, float (&o)[8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[2 * i] = s * (float)((int)((w >> (4 * i)) & 15u) - 8);
        o[2 * i + 1] = s * (float)((int)((w >> (16 + 4 * i)) & 15u) - 8);
    }
}

template <typename XT, int TT>
__global__ __launch_bounds__(256) void gate_up_q4_generic(
    const XT *__restrict__ x, int T, int d, int G, int gs, const uint32_t *__restrict__ Gq,
    const bf16_t *__restrict__ Gs, const uint32_t *__restrict__ Uq, const bf16_t *__restrict__ Us,
    const uint8_t *__restrict__ mask, const int32_t *__restrict__ ulist, const int32_t *__restrict__ meta,
    float *__restrict__ act, int act_stride)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int total = meta[0] * gs;
    const int nwaves = gridDim.x * 4;
    const int words = d / 8, blocks = d / kQ4Block;
    for (int n = blockIdx.x * 4 + wave; n < total; n += nwaves) {
        const int u = n / gs, m = n - u * gs;
        const int g = ulist[u];
        const size_t row = (size_t)g * gs + m;
        for (int t0 = 0; t0 < T; t0 += TT) {
            float ag[TT], au[TT];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) ag[tt] = au[tt] = 0.0f;
            for (int c = lane; c < words; c += kWave) {
                float a[8], b[8];
                q4_unpack8(Gq[row * words + c], to_float(Gs[row * blocks + c / 16]), a);
                q4_unpack8(Uq[row * words + c], to_float(Us[row * blocks + c / 16]), b);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    if (t0 + tt < T) {
                        float xv[8];
                        load8(x + (size_t)(t0 + tt) * d + c * 8, xv);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            ag[tt] = __builtin_fmaf(a[e], xv[e], ag[tt]);
                            au[tt] = __builtin_fmaf(b[e], xv[e], au[tt]);
                        }
                    }
                }
            }
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const float vg = wave_sum(ag[tt]), vu = wave_sum(au[tt]);
                const int t = t0 + tt;
                if (lane == 0 && t < T)
                    act[(size_t)t * act_stride + n] = mask[(size_t)t * G + g] ? silu_mul(vg, vu) : 0.0f;
            }
        }
    }
}

// one wave per output row j; lanes take neurons lane and lane + 64 of every union group
template <typename XT, int TT>
__global__ __launch_bounds__(256) void down_q4_generic(
    const float *__restrict__ act, int act_stride, int T, int d, const uint32_t *__restrict__ Dq,
    const bf16_t *__restrict__ Ds, const int32_t *__restrict__ ulist, const int32_t *__restrict__ meta,
    XT *__restrict__ y)
{
    constexpr int gs = 128;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int j = blockIdx.x * 4 + wave;
    if (j >= d) return;
    const int n_u = meta[0];
    for (int t0 = 0; t0 < T; t0 += TT) {
        float acc[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[tt] = 0.0f;
        for (int u = 0; u < n_u; ++u) {
            const size_t blk = (size_t)ulist[u] * d + j;
            const float s = to_float(Ds[blk]);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int m = lane + half * kWave;
                const uint32_t w = Dq[blk * (gs / 8) + m / 8];
                const int k = m & 7;
                const int shift = (k & 1) ? 16 + 4 * (k >> 1) : 4 * (k >> 1);
                const float wv = s * (float)((int)((w >> shift) & 15u) - 8);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    if (t0 + tt < T)
                        acc[tt] = __builtin_fmaf(wv, act[(size_t)(t0 + tt) * act_stride + u * gs + m], acc[tt]);
            }
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const float v = wave_sum(acc[tt]);
            if (lane == 0 && t0 + tt < T) store_out(y + (size_t)(t0 + tt) * d + j, v);
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
template <typename XT>
static hipError_t q4_generic(const XT *x, int T, int d, int G, int gs, const Q4Weights &w,
                             const uint8_t *mask, XT *y, const DecodeScratch &ws, hipStream_t s)
{
    constexpr int TT = 4;
    const int ffn = G * gs;
    hipError_t e = launch_union(mask, T, G, ws.ulist, ws.meta, s);
    if (e != hipSuccess) return e;
    int blocks = (ffn + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    launch_timed("gate_up_q4_generic", gate_up_q4_generic<XT, TT>, dim3(blocks), dim3(256), s, x, T, d, G, gs,
                 w.gate_codes, w.gate_scales, w.up_codes, w.up_scales, mask, (const int32_t *)ws.ulist,
                 (const int32_t *)ws.meta, ws.act, ffn);
    down_q4_generic<XT, TT><<<dim3((d + 3) / 4), dim3(256), 0, s>>>(ws.act, ffn, T, d, w.down_codes,
                                                                  w.down_scales, ws.ulist, ws.meta, y);
    return hipGetLastError();
}

bool q4_shape_supported(int d, int gs) { return gs == kQ4Block && d % kQ4Block == 0; }

bool q4_expand_supported(int T, int dtype, int d, int G, int gs)
{
    return dtype == 1 && T > 16 && q4_shape_supported(d, gs) &&
           (mfma_path_supported(T, d, gs) || prefill_path_supported(T, d, gs));
}

// 4-bit codes and their scales -> bf16 values s * (c - 8), each rounded to nearest even: rows of K elements,
// one scale per 128 consecutive elements of a row (K = d for gate / up; K = 128 with one scale per row for
// the group-blocked down projection).  A thread takes one word of codes (8 elements) at a time and writes
// 16 bytes, so that a wave's store instruction covers 1 KiB of consecutive bytes (16 bytes of codes per
// thread made every store instruction touch 64 cache lines, 16 bytes of each).
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(256) void expand_q4_kernel(const uint32_t *__restrict__ codes,
                                                        const bf16_t *__restrict__ scales,
                                                        bf16_t *__restrict__ out, size_t words)
{
    constexpr int U = 4;                                    // words per thread and pass, all requested first
    const int words_per_block = kQ4Block / 8;
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t w0 = (size_t)blockIdx.x * 256 + threadIdx.x; w0 < words; w0 += stride * U) {
        uint32_t w[U];
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t i = w0 + u * stride < words ? w0 + u * stride : w0;
            w[u] = __builtin_nontemporal_load(codes + i);
            s[u] = bf16_bits_to_float(scales[i / words_per_block]);    // blocks follow each other row after row
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (w0 + u * stride < words) {
                const float off = -136.0f * s[u];
                uint32_t pr[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // the pair (2i, 2i+1) as the bf16 values 128 + c; s * (128 + c) - 136 s = s * (c - 8), exact
                    // in float (an 8-bit by 8-bit product and a difference of neighbours); one instruction
                    // rounds both
                    const uint32_t pair = ((w[u] >> (4 * i)) & 0x000F000Fu) | 0x43004300u;
                    const f32x2_t v = {__builtin_fmaf(bf16_lo(pair), s[u], off), __builtin_fmaf(bf16_hi(pair), s[u], off)};
                    pr[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
                }
                reinterpret_cast<u32x4 *>(out)[w0 + u * stride] = u32x4{pr[0], pr[1], pr[2], pr[3]};
            }
        }
    }
}

static hipError_t expand_q4(const uint32_t *codes, const bf16_t *scales, bf16_t *out, size_t rows, int K, hipStream_t s)
{
    const size_t words = rows * (size_t)(K / 8);
    const size_t want = (words + 1023) / 1024;
    const int blocks = (int)(want < 16384 ? want : 16384);
    expand_q4_kernel<<<dim3(blocks), dim3(256), 0, s>>>(codes, scales, out, words);
    return hipGetLastError();
}

template <typename AT>
static hipError_t q4_one_token(const bf16_t *x, int d, int G, const Q4Weights &w, const uint8_t *mask, bf16_t *y, AT *act,
                               hipStream_t s, const AheadArgs *ahead, bool *ahead_fused)
{
    constexpr bool kWhole = sizeof(AT) == 2;
    const AheadArgs *ah = (ahead && ahead_fused) ? ahead : nullptr;
    if (ah) *ahead_fused = true;
    // predictors of 256 or 512 rows: one or two rows in every gate/up workgroup; else workgroups of their own
    const int pred_rows = (ah && (ah->r == kQ4GateUpBlocks || ah->r == 2 * kQ4GateUpBlocks)) ? ah->r / kQ4GateUpBlocks : 0;
    const int n_pred = (ah && pred_rows == 0) ? (ah->r + 7) / 8 : 0;
    const bf16_t *xn = ah ? (const bf16_t *)ah->x_next : nullptr, *an = ah ? (const bf16_t *)ah->At : nullptr;
    float *hn = ah ? ah->h : nullptr;
    const int r = ah ? ah->r : 0;
#define HALO_Q4_T1(NH)                                                                                                  \
    launch_timed("gate_up_q4_t1", gate_up_q4_t1<NH, kWhole, AT>, dim3(kQ4GateUpBlocks + n_pred), dim3(kQ4GateUpThreads), \
                 s, x, G, w.gate_codes, w.gate_scales, w.up_codes, w.up_scales, mask, act, xn, an, r, hn, n_pred,       \
                 pred_rows, d)
    switch ((d + 2047) / 2048) {
    case 1: if constexpr (!kWhole) HALO_Q4_T1(1); break;
    case 2: HALO_Q4_T1(2); break;
    case 3: if constexpr (!kWhole) HALO_Q4_T1(3); break;
    default: HALO_Q4_T1(4); break;
    }
#undef HALO_Q4_T1
    const AheadDev nx = ah ? ahead_dev(*ah) : AheadDev{};
    down_q4_t1<AT><<<dim3(d / 16 + (ah ? 1 : 0)), dim3(512), 0, s>>>(d, G, w.down_codes, w.down_scales, mask, (const AT *)act,
                                                                 y, ah ? 1 : 0, nx);
    return hipGetLastError();
}

hipError_t launch_ffn_q4(int dtype, const void *x, int T, int d, int G, int gs, const Q4Weights &w,
                         const uint8_t *mask, void *y, const DecodeScratch &ws, hipStream_t s,
                         const AheadArgs *ahead, bool *ahead_fused)
{
    if (ahead_fused) *ahead_fused = false;
    if (dtype == 0)
        return q4_generic<float>((const float *)x, T, d, G, gs, w, mask, (float *)y, ws, s);
    const bf16_t *bx = (const bf16_t *)x;
    bf16_t *by = (bf16_t *)y;
    if (T == 1 && G <= 256 && d <= 8192)
        return d == 4096 || d == 8192
                   ? q4_one_token<bf16_t>(bx, d, G, w, mask, by, reinterpret_cast<bf16_t *>(ws.act), s, ahead, ahead_fused)
                   : q4_one_token<float>(bx, d, G, w, mask, by, ws.act, s, ahead, ahead_fused);
    if (stream_path_supported(T, d, G, gs)) return launch_ffn_q4_mfma(bx, T, d, G, w, mask, by, ws, s, ahead, ahead_fused);
    // The many-token kernels multiply by values rounded to bf16 (from 65 tokens on, and over rows of 128), the few-token kernels scale in
    // float: which of the two a call of many tokens gets is the caller's choice, by the workspace.
    if (ws.q4_w && prefill_q4_supported(T, d, G, gs)) return launch_ffn_prefill_q4(bx, T, d, G, w, mask, by, ws, s);
    if (ws.q4_w && q4_expand_supported(T, dtype, d, G, gs)) {
        // More tokens than the row table's 16 bits hold, and room for a block's weights as bf16: the weights are expanded once (a stream of
        // 0.5 + 2 bytes per element) and the bf16 matrix-core kernels do the rest, every weight used for
        // all the tokens that keep its group.
        const size_t ffn = (size_t)G * gs;
        bf16_t *Wg = ws.q4_w, *Wu = Wg + ffn * d, *Wd = Wu + ffn * d;
        hipError_t e = expand_q4(w.gate_codes, w.gate_scales, Wg, ffn, d, s);
        if (e == hipSuccess) e = expand_q4(w.up_codes, w.up_scales, Wu, ffn, d, s);
        if (e == hipSuccess) e = expand_q4(w.down_codes, w.down_scales, Wd, (size_t)G * d, gs, s);
        if (e != hipSuccess) return e;
        return launch_ffn_decode(dtype, x, T, d, G, gs, Wg, Wu, Wd, mask, y, ws, s);
    }
    if (T > 16 && stream_path_supported(16, d, G, gs)) {
        // Many tokens: the matrix-core kernels over tiles of up to 16 tokens, one tile after the other on
        // the stream (each streams the union of its own tokens' groups; the activation scratch is reused).
        // No kernel of its own for this case yet: a tile pair of launches is 30-90 us, where the plain path
        // below takes 50 us per TOKEN at the 7B shape.  A last tile of one token would leave the kernels'
        // range, so the last two tiles share their tokens.
        for (int t0 = 0; t0 < T;) {
            int n = T - t0 > 16 ? 16 : T - t0;
            if (T - t0 == 17) n = 15;
            const hipError_t e = launch_ffn_q4_mfma(bx + (size_t)t0 * d, n, d, G, w, mask + (size_t)t0 * G,
                                                    by + (size_t)t0 * d, ws, s, nullptr, nullptr);
            if (e != hipSuccess) return e;
            t0 += n;
        }
        return hipSuccess;
    }
    return q4_generic<bf16_t>(bx, T, d, G, gs, w, mask, by, ws, s);
}

}  // namespace halo
