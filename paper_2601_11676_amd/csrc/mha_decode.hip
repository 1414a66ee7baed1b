// Head-sparse multi-head attention for one new token (paper Sec. II-A: in the MHA one head
// and its slice of the output projection are one neuron group, the block output is the sum
// of the groups' partial results; Sec. III-B.3: every device keeps the full KV cache).
//
//   every head h     : k_h = Wk_h x, v_h = Wv_h x  -> row `pos` of the caches (storage type)
//   surviving heads  : q_h = Wq_h x,  p = softmax(q_h K_h^T / sqrt(dh)) over rows 0..pos,
//                      o_h = p V_h,   y = sum_h Wo_h o_h
//
// bf16, head dimension 128.  Three launches, or four (long caches, many heads):
//   qkv_rows     : a matrix-vector product over the rows that are needed -- all of Wk and Wv,
//                  and the rows of Wq of surviving heads only -- streamed like the FFN's
//                  gate/up rows (one wave per row, 16-byte non-temporal loads, two rows
//                  in flight while two are reduced).
//   attn_partial : one workgroup per (surviving head, 128 to 512 cached positions): scores, a local
//                  softmax (max, sum) and the weighted sum of the values of its positions.
//   merge_out_t1 : merges the heads' partial softmaxes and multiplies by Wo, which is stored head-blocked [H][d][128] exactly
//                  like Wd, heads in the role of groups; or
//   attn_combine : merges a head's partial softmaxes into o_h, and
//   out-proj     : the FFN's down-projection kernel, unchanged.
// Only surviving heads' query rows, cache rows and output-projection blocks are read.
#include <algorithm>
#include "down_t1.hpp"
#include "kernels.hpp"
#include "mask_device.hpp"
#include "mask_words.hpp"
#include "row_stream.hpp"

namespace halo {

constexpr int kHeadDim = 128;
constexpr int kAttnChunk = 128;      // cached positions per workgroup of attn_partial

// Maximum over the 64 lanes of a wave, in every lane, by the exchanges of the predictor's butterfly (xor_add): none goes through the LDS
// crossbar, on whose round trip each of six dependent steps would wait.  (With it and the value sums' two distances exchanged this way a
// block of 8 heads, 339 rows takes 12.9 us, 13.2 before; of 32 heads, 2048 rows 29.1, 29.25 before.)
__device__ __forceinline__ float wave_max(float v)
{
    auto as_f = [](unsigned u) { return __builtin_bit_cast(float, u); };
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned h = __builtin_bit_cast(unsigned, fmaxf(as_f(a[0]), as_f(a[1])));
    const auto b = __builtin_amdgcn_permlane16_swap(h, h, false, false);
    v = fmaxf(as_f(b[0]), as_f(b[1]));
    auto dpp = [&](auto ctrl) { return as_f((unsigned)__builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true)); };
    v = fmaxf(v, dpp(std::integral_constant<int, 0x128>{}));     // row_ror:8
    v = fmaxf(v, dpp(std::integral_constant<int, 0x141>{}));     // row_half_mirror: with distance 8 done, the lanes' other half of eight
    v = fmaxf(v, dpp(std::integral_constant<int, 0x4E>{}));      // quad_perm [2,3,0,1]
    return fmaxf(v, dpp(std::integral_constant<int, 0xB1>{}));   // quad_perm [1,0,3,2]
}

// ---------------------------------------------------------------------------
// q / k / v rows: grid = 256 workgroups of 256 threads
// ---------------------------------------------------------------------------
// Row v of the job list: v < H*dh -> Wk row v, < 2*H*dh -> Wv row, else a Wq row of the
// (v - 2*H*dh) / dh -th surviving head.  K/V rows do not depend on the mask, so every wave starts on its share of them at once and meets
// the mask only for its query rows.  They follow in the same sequence of loads and sums: with a sequence of its own for each, nothing was
// on its way while the last key or value row was summed up, and shares of both that were not whole numbers left some waves two pairs of
// rows more than others.  A block with half its heads and the next one's prediction, us, two sequences / one: d 1024, 8 heads 13.7 / 13.2;
// d 2048, 16 heads 16.8 / 15.8; d 3200, 25 heads 23.6 / 22.8; d 4096, 32 heads 29.8 / 29.3 (84 MB, this launch alone 16.1 / 15.6: 5.4 TB/s);
// d 5120, 40 heads 42.6 / 41.9; d 7168, 8192 level.
template <int NCH>
struct RowRegs {
    u32x4 a[NCH], b[NCH];            // two independent rows
};

template <int NCH, bool TAIL>
__device__ __forceinline__ void load_two(RowRegs<NCH> &r, const bf16_t *pa, const bf16_t *pb, const RowLanes<NCH, TAIL> &rl,
                                         int lane)
{
    const u32x4 *qa = reinterpret_cast<const u32x4 *>(pa), *qb = reinterpret_cast<const u32x4 *>(pb);
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        r.a[k] = __builtin_nontemporal_load(qa + rl.piece(k, lane));
        r.b[k] = __builtin_nontemporal_load(qb + rl.piece(k, lane));
    }
}

template <int NCH, bool TAIL>
__device__ __forceinline__ void dot_two(const RowRegs<NCH> &r, const u32x4 (&xr)[NCH], const RowLanes<NCH, TAIL> &rl,
                                        float &ra, float &rb)
{
    float a0 = 0.0f, b0 = 0.0f;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        const u32x4 a = rl.keep(r.a[k], k), b = rl.keep(r.b[k], k);
        a0 = dot2_bf16(a.x, xr[k].x, a0);
        b0 = dot2_bf16(b.x, xr[k].x, b0);
        a0 = dot2_bf16(a.y, xr[k].y, a0);
        b0 = dot2_bf16(b.y, xr[k].y, b0);
        a0 = dot2_bf16(a.z, xr[k].z, a0);
        b0 = dot2_bf16(b.z, xr[k].z, b0);
        a0 = dot2_bf16(a.w, xr[k].w, a0);
        b0 = dot2_bf16(b.w, xr[k].w, b0);
    }
    ra = wave_sum_fast(a0);
    rb = wave_sum_fast(b0);
}

struct QkvArgs {
    const bf16_t *x, *Wq, *Wk, *Wv;
    bf16_t *k_cache, *v_cache;       // [H][max_len][128]
    float *q;                        // [n_surv][128], compact by surviving-head slot
    const uint8_t *mask;             // [H]
    int H, max_len, pos;
    // the next block's first predictor layer, in the first n_pred workgroups (0 = none)
    const bf16_t *x_next, *At_next;
    float *h_next;
    int r, n_pred;
};

template <int NCH, bool TAIL>
__global__ __launch_bounds__(256) void qkv_rows(QkvArgs a, int len)
{
    constexpr int dh = kHeadDim;
    const int d = TAIL ? len : NCH * 512;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const RowLanes<NCH, TAIL> rl(d, lane);
    if ((int)blockIdx.x < a.n_pred) {
        // paper Sec. III-B.3, Pred beside Load/Comp, one layer ahead: h_next = ReLU(x_next A)
        const int j = blockIdx.x * 4 + wave;
        if (j < a.r) {
            const float p = dot_order64_row<NCH, TAIL>(a.x_next, a.At_next + (size_t)j * d, rl, lane);
            if (lane == 0) a.h_next[j] = p > 0.0f ? p : 0.0f;
        }
        return;
    }
    const int nw = (gridDim.x - a.n_pred) * 4, w = (blockIdx.x - a.n_pred) * 4 + wave;
    const MaskWords mw = load_mask_words(a.mask, a.H, lane);     // needed behind the first rows' loads
    u32x4 xr[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) xr[k] = rl.keep(reinterpret_cast<const u32x4 *>(a.x)[rl.piece(k, lane)], k);
    // this wave's pairs of rows in one sequence: n_kv of the 2*H*dh key and value rows, then those of the surviving heads' query rows
    // (count*dh rows, compact by slot)
    const int hd = a.H * dh, p0 = (int)((long long)hd * w / nw), n_kv = (int)((long long)hd * (w + 1) / nw) - p0;
    int q0 = 0, cur_u = -1, cur_g = 0;
    auto load = [&](RowRegs<NCH> &r, int i) __attribute__((always_inline)) {
        const bf16_t *src;
        if (i < n_kv) {
            const int v = 2 * (p0 + i);                          // hd is even: both rows on one side
            src = v < hd ? a.Wk + (size_t)v * d : a.Wv + (size_t)(v - hd) * d;
        } else {
            const int v = 2 * (q0 + i - n_kv), u = v / dh;
            if (u != cur_u) {
                cur_u = u;
                cur_g = nth_group(mw, u, lane);
            }
            src = a.Wq + ((size_t)cur_g * dh + (v - u * dh)) * d;
        }
        load_two<NCH, TAIL>(r, src, src + d, rl, lane);
    };
    auto finish = [&](const RowRegs<NCH> &r, int i) __attribute__((always_inline)) {
        float va, vb;
        dot_two<NCH, TAIL>(r, xr, rl, va, vb);
        if (lane != 0) return;
        if (i < n_kv) {
            const int v = 2 * (p0 + i), row = v < hd ? v : v - hd, h = row / dh;
            bf16_t *dst = (v < hd ? a.k_cache : a.v_cache) + ((size_t)h * a.max_len + a.pos) * dh + (row - h * dh);
            dst[0] = f32_to_bf16(va);
            dst[1] = f32_to_bf16(vb);
        } else {
            float *dst = a.q + 2 * (q0 + i - n_kv);
            dst[0] = va;
            dst[1] = vb;
        }
    };
    RowRegs<NCH> A, B;
    {
        // keys and values don't depend on the mask: their first rows are on their way while it arrives (a row that exists where this
        // wave has none)
        const int v = 2 * min(p0, hd - 1);
        const bf16_t *src = v < hd ? a.Wk + (size_t)v * d : a.Wv + (size_t)(v - hd) * d;
        load_two<NCH, TAIL>(A, src, src + d, rl, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the queries' share: as many as bring this wave's sum to its share of all pairs, where that takes none away from anyone
    const int qp = mw.count * (dh / 2);
    int q1;
    if (qp >= nw) {
        q0 = (int)((long long)(hd + qp) * w / nw) - p0;
        q1 = (int)((long long)(hd + qp) * (w + 1) / nw) - (p0 + n_kv);
    } else {
        q0 = (int)((long long)qp * w / nw);
        q1 = (int)((long long)qp * (w + 1) / nw);
    }
    const int n = n_kv + q1 - q0;
    if (n == 0) return;
    if (n_kv == 0) load(A, 0);
    int i = 0;
    while (i + 2 < n) {
        load(B, i + 1);
        finish(A, i);
        load(A, i + 2);
        finish(B, i + 1);
        i += 2;
    }
    if (i + 1 < n) {
        load(B, i + 1);
        finish(A, i);
        finish(B, i + 1);
    } else {
        finish(A, i);
    }
}

// any d that is a multiple of 8: one wave per row, one row at a time
__global__ __launch_bounds__(256) void qkv_rows_generic(QkvArgs a, int d, const int32_t *__restrict__ ulist,
                                                        const int32_t *__restrict__ meta)
{
    constexpr int dh = kHeadDim;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int hd = a.H * dh, total = 2 * hd + meta[0] * dh;
    for (int v = blockIdx.x * 4 + wave; v < total; v += gridDim.x * 4) {
        const bf16_t *src;
        if (v < hd) src = a.Wk + (size_t)v * d;
        else if (v < 2 * hd) src = a.Wv + (size_t)(v - hd) * d;
        else {
            const int r = v - 2 * hd, u = r / dh;
            src = a.Wq + ((size_t)ulist[u] * dh + (r - u * dh)) * d;
        }
        float p = 0.0f;
        for (int c = lane; c * 8 < d; c += kWave) {
            float xv[8], wv[8];
            load8(a.x + c * 8, xv);
            load8(src + c * 8, wv);
#pragma unroll
            for (int e = 0; e < 8; ++e) p = __builtin_fmaf(xv[e], wv[e], p);
        }
        p = wave_sum(p);
        if (lane == 0) {
            if (v < 2 * hd) {
                const int r = v < hd ? v : v - hd;
                const int h = r / dh, e = r - h * dh;
                (v < hd ? a.k_cache : a.v_cache)[((size_t)h * a.max_len + a.pos) * dh + e] = f32_to_bf16(p);
            } else {
                a.q[v - 2 * hd] = p;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// attention over the cache: grid (chunks, H), 2 CH threads
// ---------------------------------------------------------------------------
// Workgroup (c, u): surviving-head slot u (exits if u >= number of survivors), cached
// positions c*CH .. c*CH+CH-1 (rows beyond pos count as score -inf).  16 lanes share a
// cache row (16 bytes = 8 dimensions each), a wave covers 4 rows per instruction and 32 rows
// in all.  Output: part[(u*chunks + c)] = {128 weighted value sums, local max, local sum}.
// (CH = 128; with 256 or 512 positions to a workgroup of twice or four times the threads a head has few enough partial softmaxes
// for the output projection to merge them.)
constexpr int kPartStride = kHeadDim + 2;

template <int CH>
__global__ __launch_bounds__(CH * 2) void attn_partial(const float *__restrict__ q, const bf16_t *__restrict__ k_cache,
                                                    const bf16_t *__restrict__ v_cache,
                                                    const uint8_t *__restrict__ mask, int H, int max_len, int pos,
                                                    float *__restrict__ part)
{
    constexpr int dh = kHeadDim;
    constexpr int W = CH / 32;                                   // waves
    __shared__ float s_score[CH];
    __shared__ float s_o[W][dh];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c = blockIdx.x, u = blockIdx.y, chunks = gridDim.x;
    const int sub = lane >> 4, piece = (lane & 15) * 8;
    const MaskWords mw = load_mask_words(mask, H, lane);
    // in front of the rows, as the first scores need it (32 heads, half of them, 2048 rows: behind them 6.6 us, with keys and values in
    // turn; here 6.1)
    float qf[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[e] = q[u * dh + piece + e];
    if (u >= mw.count) return;                                   // uniform
    const int h = nth_group(mw, u, lane);
    const bf16_t *K = k_cache + (size_t)h * max_len * dh, *V = v_cache + (size_t)h * max_len * dh;
    const int j0 = c * CH + wave * 32;                   // this wave's first row
    // every load of the workgroup's (64 KiB for 128 positions) is requested before anything is reduced, the keys' in front: loads return
    // in order, and the scores are computed while the values arrive
    u32x4 kv[8], vv[8];
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        int j = j0 + it * 4 + sub;
        j = j <= pos ? j : pos;                                  // past the end: a valid duplicate, weight 0
        kv[it] = *reinterpret_cast<const u32x4 *>(K + (size_t)j * dh + piece);
    }
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        int j = j0 + it * 4 + sub;
        j = j <= pos ? j : pos;
        vv[it] = *reinterpret_cast<const u32x4 *>(V + (size_t)j * dh + piece);
    }
    __builtin_amdgcn_sched_barrier(0);
    const float scale = 0.08838834764831845f;                    // 1 / sqrt(128)
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        float kf[8], sdot = 0.0f;
        unpack8(kv[it], kf);
#pragma unroll
        for (int e = 0; e < 8; ++e) sdot = __builtin_fmaf(qf[e], kf[e], sdot);
        sdot = dpp_add<0xB1>(sdot);                              // the 16 lanes of a row
        sdot = dpp_add<0x4E>(sdot);
        sdot = dpp_add<0x141>(sdot);
        sdot = dpp_add<0x140>(sdot);
        const int j = j0 + it * 4 + sub;
        if ((lane & 15) == 0) s_score[wave * 32 + it * 4 + sub] = j <= pos ? sdot * scale : -INFINITY;
    }
    __syncthreads();
    // local softmax statistics (every wave computes them for itself from all scores)
    float m = s_score[lane];
#pragma unroll
    for (int k = 1; k < CH / 64; ++k) m = fmaxf(m, s_score[lane + 64 * k]);
    m = wave_max(m);
    // the chunk's first row always exists (chunks are launched only up to pos), so m is finite
    float l = 0.0f;
#pragma unroll
    for (int k = 0; k < CH / 64; ++k) l += __expf(s_score[lane + 64 * k] - m);
    l = wave_sum(l);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const float p = __expf(s_score[wave * 32 + it * 4 + sub] - m);
        float vf[8];
        unpack8(vv[it], vf);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(p, vf[e], acc[e]);
    }
    // the four row slots of a wave, then the four waves
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        acc[e] = xor_add<16>(acc[e]);
        acc[e] = xor_add<32>(acc[e]);
    }
    if (lane < 16) {
#pragma unroll
        for (int e = 0; e < 8; ++e) s_o[wave][piece + e] = acc[e];
    }
    __syncthreads();
    float *out = part + ((size_t)u * chunks + c) * kPartStride;
    if (tid < dh) {
        float v = s_o[0][tid];
#pragma unroll
        for (int w = 1; w < W; ++w) v += s_o[w][tid];
        out[tid] = v;
    }
    if (tid == 0) {
        out[dh] = m;
        out[dh + 1] = l;
    }
}

// grid = H workgroups of 128 threads: o_u = sum_c e^{m_c - M} o_c / sum_c e^{m_c - M} l_c.
// Thread tid owns dimension tid of the head and chunk tid's statistics.  Everything the first 32 chunks
// need -- the thread's chunk maximum and sum, and its 32 value sums -- is requested before anything is
// waited for, so a cache of up to 4096 positions costs one memory round trip (with the maxima, the
// sums and the values fetched in turn, in batches of eight, it was six).
constexpr int kMaxChunks = 1024;     // 131072 cached positions

template <typename OT>
__global__ __launch_bounds__(128) void attn_combine(const float *__restrict__ part, const uint8_t *__restrict__ mask,
                                                    int H, int chunks, OT *__restrict__ act)
{
    constexpr int dh = kHeadDim, kBatch = 32;
    __shared__ float s_w[kMaxChunks];
    __shared__ float s_red[2][2];
    const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const MaskWords mw = load_mask_words(mask, H, lane);
    if (u >= mw.count) return;
    const float *p = part + (size_t)u * chunks * kPartStride;
    // this thread's chunk statistics and the first batch of value sums, all in flight together, the statistics in front: loads return in
    // order, and the weights are computed from them while the values arrive
    const int c_own = tid < chunks ? tid : chunks - 1;
    const float m_own = p[(size_t)c_own * kPartStride + dh], l_own = p[(size_t)c_own * kPartStride + dh + 1];
    __builtin_amdgcn_sched_barrier(0);
    float v[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) v[i] = p[(size_t)(i < chunks ? i : chunks - 1) * kPartStride + tid];
    // pass 1: maximum of the chunk maxima
    float m_loc = tid < chunks ? m_own : -INFINITY;
    for (int c = tid + 128; c < chunks; c += 128) m_loc = fmaxf(m_loc, p[(size_t)c * kPartStride + dh]);
    m_loc = wave_max(m_loc);
    if (lane == 0) s_red[0][wave] = m_loc;
    __syncthreads();
    const float M = fmaxf(s_red[0][0], s_red[0][1]);
    // pass 2: chunk weights and the denominator
    float l_loc = 0.0f;
    if (tid < chunks) {
        const float w = __expf(m_own - M);
        s_w[tid] = w;
        l_loc = w * l_own;
    }
    for (int c = tid + 128; c < chunks; c += 128) {
        const float w = __expf(p[(size_t)c * kPartStride + dh] - M);
        s_w[c] = w;
        l_loc = __builtin_fmaf(w, p[(size_t)c * kPartStride + dh + 1], l_loc);
    }
    l_loc = wave_sum(l_loc);
    if (lane == 0) s_red[1][wave] = l_loc;
    __syncthreads();
    const float L = s_red[1][0] + s_red[1][1];
    float o = 0.0f;
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
        if (i < chunks) o = __builtin_fmaf(s_w[i], v[i], o);
    for (int c0 = kBatch; c0 < chunks; c0 += kBatch) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) v[i] = p[(size_t)(c0 + i < chunks ? c0 + i : chunks - 1) * kPartStride + tid];
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (c0 + i < chunks) o = __builtin_fmaf(s_w[c0 + i], v[i], o);
    }
    store_out(act + u * dh + tid, o / L);
}

// ---------------------------------------------------------------------------
// output projection that merges the heads' partial softmaxes itself: up to nine of them, up to 64 heads
// ---------------------------------------------------------------------------
// Every workgroup merges all surviving heads into LDS, n_surv * chunks * 520 bytes from L2, before it multiplies; that takes the place
// of a launch of its own.  A wave's loads return in order, so a thread asks for its first head's partials before the rows of Wo for the
// first heads, 48 loads of 16 bytes from HBM: behind them the merge began when the last of them had come.  A block with the next one's
// prediction, half the heads, us, us merged behind Wo's rows or in a launch of its own / merged in front of them: d 4096, 32 heads,
// 339 rows 27.9 / 27.5, 2048 rows 31.2 / 30.4, d 3200, 25 heads, 700 rows 24.8 / 23.5, d 7168, 56 heads, 700 rows 63.8 / 61.5.
// Up to 16 heads are merged here whenever nine chunks of up to 512 positions hold the cache (d 1024, 8 heads, 120 to 2000 rows
// 14.1 .. 14.9 in a launch of its own, 11.6 .. 13.7 here; d 2048, 16 heads, 2000 rows 18.3 / 17.2).  With more heads a thread has
// several heads' worth to merge one after the other, and there is a point from where the launch is the faster (own launch / here: d 3200,
// 25 heads, 8 chunks of 256 25.9 / 26.2; d 8192, 64 heads, 8 chunks of 128 77.4 / 77.9, 4 of 256 77.4 / 76.6; d 5120, 40 heads,
// 7 chunks of 256 40.4 / 39.6, 8 of 256 level; 32 heads, 9 chunks of 256 31.7 / 31.1; with chunks of 512 26.4 / 27.6 at 25 heads,
// 3000 rows).  So more than 16 heads are merged here while heads times chunks of up to 256 stay within 288 with the activations in
// bf16, and up to six chunks with them in float32.
constexpr int kMergeChunks = 9, kMergeHeads = 64;

template <typename AT>
struct MergedHeads {
    __attribute__((aligned(16))) AT act[kMergeHeads * kHeadDim];
};

template <int RQ, typename AT, bool EXACT>
__global__ __launch_bounds__(RQ * 128, 4) void merge_out_t1(int d, int H, const bf16_t *__restrict__ Wo,
                                                           const uint8_t *__restrict__ mask, const float *__restrict__ part,
                                                           int chunks, bf16_t *__restrict__ y, int ahead, AheadDev nx)
{
    constexpr int dh = kHeadDim, NT = RQ * 128;
    struct Proj {
        DownShared<RQ> down;
        MergedHeads<AT> o;
    };
    constexpr size_t kLds = sizeof(Proj) > sizeof(MaskShared) ? sizeof(Proj) : sizeof(MaskShared);
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    if (ahead && blockIdx.x == 0) {
        mask_scores_block<NT, bf16_t, true>(*reinterpret_cast<MaskShared *>(lds), tid, nx.h, nx.Bt, nx.r, nx.scores, H, nx.K,
                                            nx.prio_dev, nx.n_dev, nx.drop, nx.order, nx.group_dev, nx.mask, nx.surv_idx, nx.n_surv);
        return;
    }
    Proj &sh = *reinterpret_cast<Proj *>(lds);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), vblock = blockIdx.x - (ahead ? 1 : 0);
    const MaskWords mw = load_mask_words(mask, H, lane);
    if (wave == 0) write_group_list(mw, lane, sh.down.list);
    __syncthreads();
    const int count = mw.count;
    // rows and heads dealt as in down_t1_body, which adds up in the same order
    const int rq = wave % RQ, half = wave / RQ;                  // row quad, even/odd heads
    const int row = (vblock * RQ + rq) * 4 + (lane >> 4), piece = (lane & 15) * 8;
    const __amdgpu_buffer_rsrc_t bw = buffer_of(Wo), bp = buffer_of(part);
    const uint32_t at_w = (uint32_t)((EXACT ? row : min(row, d - 1)) * dh + piece) * 2;
    const int my_head = sh.down.list[lane];                      // at most 64: one to a lane
    // three batches in flight: 24 heads between the two halves, 18 with activations in float32 (with 24 that form spilled 19 registers:
    // d 1024, 8 heads, 339 rows 12.5 -> 11.9 us, d 7168, 56 heads, 300 rows 64.0 -> 59.6; d 3200, 40 heads, 300 rows 29.1 -> 29.5)
    constexpr int kB = sizeof(AT) == 4 ? 3 : 4;
    auto fetch = [&](u32x4 (&v)[kB], int u0) {
#pragma unroll
        for (int q = 0; q < kB; ++q) {
            const int u = u0 + 2 * q < count ? u0 + 2 * q : (count > 0 ? count - 1 : 0);   // an in-range duplicate
            v[q] = buffer_load16<kNt>(bw, at_w, (uint32_t)__builtin_amdgcn_readlane(my_head, u) * (uint32_t)d * (dh * 2));
        }
    };
    float acc0 = 0.0f, acc1 = 0.0f;
    auto mac = [&](const u32x4 (&v)[kB], int u0) {
#pragma unroll
        for (int q = 0; q < kB; ++q) {
            if (u0 + 2 * q < count) {
                ActPiece<AT> a;
                a.load(sh.o.act + (u0 + 2 * q) * dh + piece);
                a.dot(v[q], acc0, acc1);
            }
            if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // two heads' operands at a time: registers
        }
    };
    // the merge; a thread: four dimensions of a head, 32 threads a head.  Its loads go in front of Wo's, which are many bytes more, and
    // loads return in order; a wave that has no head asks for none (with few heads kept most of a large workgroup's: d 8192, 32 heads, one kept,
    // 1500 rows 34.4 us with duplicates asked for, 31.6).  Where threads have several heads' worth, all but the last are merged first if the chunks
    // are many (32 heads of d 4096, all kept, 2048 rows 38.2 -> 37.3; d 3200, 25 heads, 1500 rows 28.0 -> 26.9); with few the rows of Wo
    // would wait for nothing (64 heads of d 8192, 60 rows 91.3, that way 92.8).
    const int n_ids = count * (dh / 4);
    float2 pv[kMergeChunks][2], st[kMergeChunks];
    auto ask = [&](int id) __attribute__((always_inline)) {
        const int u = min(id, n_ids - 1) / (dh / 4), e = (id % (dh / 4)) * 4;
        const uint32_t head = (uint32_t)(u * chunks * kPartStride) * 4, at = head + e * 4;
        auto load2 = [&](uint32_t voff, uint32_t soff) { return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(bp, voff, soff, 0)); };
#pragma unroll
        for (int c = 0; c < kMergeChunks; ++c) {
            if (c < chunks) {                                    // uniform
                st[c] = load2(head, (c * kPartStride + dh) * 4);
                pv[c][0] = load2(at, c * kPartStride * 4);
                pv[c][1] = load2(at, c * kPartStride * 4 + 8);
            }
        }
    };
    auto merge = [&](int id) __attribute__((always_inline)) {
        float M = st[0].x;
#pragma unroll
        for (int c = 1; c < kMergeChunks; ++c)
            if (c < chunks) M = fmaxf(M, st[c].x);
        float L = 0.0f, o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int c = 0; c < kMergeChunks; ++c) {
            if (c < chunks) {
                const float w = __expf(st[c].x - M);
                L = __builtin_fmaf(w, st[c].y, L);
                o[0] = __builtin_fmaf(w, pv[c][0].x, o[0]);
                o[1] = __builtin_fmaf(w, pv[c][0].y, o[1]);
                o[2] = __builtin_fmaf(w, pv[c][1].x, o[2]);
                o[3] = __builtin_fmaf(w, pv[c][1].y, o[3]);
            }
        }
        if (id < n_ids) {
#pragma unroll
            for (int k = 0; k < 4; ++k) store_out(sh.o.act + id / (dh / 4) * dh + (id % (dh / 4)) * 4 + k, o[k] / L);
        }
    };
    u32x4 v0[kB], v1[kB], v2[kB];
    if (count > 0) {
        int id = tid;
        if (chunks > 4) {
#pragma unroll 1
            for (; id + NT < n_ids; id += NT) {
                ask(id);
                merge(id);
            }
        }
        const bool asks = wave * 64 < n_ids;                     // uniform
        if (asks) ask(id);
        __builtin_amdgcn_sched_barrier(0);
        fetch(v0, half);
        fetch(v1, half + 2 * kB);
        fetch(v2, half + 4 * kB);
        __builtin_amdgcn_sched_barrier(0);
        if (asks) merge(id);
#pragma unroll 1
        for (id += NT; id < n_ids; id += NT) {
            ask(id);
            merge(id);
        }
    }
    __syncthreads();
    if (count > 0) {
        int u0 = half;
        while (u0 + 6 * kB < count) {
            mac(v0, u0);
            fetch(v0, u0 + 6 * kB);
            mac(v1, u0 + 2 * kB);
            fetch(v1, u0 + 8 * kB);
            mac(v2, u0 + 4 * kB);
            fetch(v2, u0 + 10 * kB);
            u0 += 6 * kB;
        }
        if (u0 < count) mac(v0, u0);
        if (u0 + 2 * kB < count) mac(v1, u0 + 2 * kB);
        if (u0 + 4 * kB < count) mac(v2, u0 + 4 * kB);
    }
    float v = acc0 + acc1;
    v = dpp_add<0xB1>(v);    // the 16 lanes of a row: quad_perm, quad_perm, half mirror, mirror
    v = dpp_add<0x4E>(v);
    v = dpp_add<0x141>(v);
    v = dpp_add<0x140>(v);
    if (half == 1) sh.down.half[rq][lane] = v;
    __syncthreads();
    if (half == 0 && (lane & 15) == 0 && (EXACT || row < d)) y[row] = f32_to_bf16(v + sh.down.half[rq][lane]);
}

template <int RQ, typename AT, bool EXACT>
static void launch_merge_out(int blocks, int d, int H, const bf16_t *Wo, const uint8_t *mask, const float *part, int chunks,
                             bf16_t *y, const AheadArgs *ah, hipStream_t s)
{
    merge_out_t1<RQ, AT, EXACT><<<dim3(blocks + (ah ? 1 : 0)), dim3(RQ * 128), 0, s>>>(d, H, Wo, mask, part, chunks, y, ah ? 1 : 0,
                                                                                     ah ? ahead_dev(*ah) : AheadDev{});
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
bool mha_shape_supported(int d, int head_dim) { return head_dim == kHeadDim && d % 8 == 0; }

hipError_t launch_mha_decode(const void *x, int d, int H, const void *Wq, const void *Wk, const void *Wv,
                             const void *Wo, void *k_cache, void *v_cache, int max_len, int pos,
                             const uint8_t *mask, void *y, const MhaScratch &ws, hipStream_t s,
                             const AheadArgs *ahead, bool *ahead_fused)
{
    if (ahead_fused) *ahead_fused = false;
    if (H > 256) return hipErrorInvalidValue;                    // the mask-word helpers cover 256 heads
    const int chunks = pos / kAttnChunk + 1;
    if (chunks > kMaxChunks) return hipErrorInvalidValue;
    // row lengths up to 8192 are streamed; 4096, 5120 and 8192 by kernels without a clamped last part of the row and
    // with the merged head outputs in bf16, the others with those in float32 (2048 cached rows, d = 3200: 26 us of
    // kernels in four launches; the plain row kernels took 61 us in seven, d = 2048: 22 against 44)
    const bool whole = d == 4096 || d == 5120 || d == 8192, fast = d <= 8192;
    const AheadArgs *ah = (fast && ahead && ahead_fused) ? ahead : nullptr;
    if (ah) *ahead_fused = true;
    const int n_pred = ah ? (ah->r + 3) / 4 : 0;
    QkvArgs qa{(const bf16_t *)x, (const bf16_t *)Wq, (const bf16_t *)Wk, (const bf16_t *)Wv, (bf16_t *)k_cache,
               (bf16_t *)v_cache, ws.q, mask, H, max_len, pos,
               ah ? (const bf16_t *)ah->x_next : nullptr, ah ? (const bf16_t *)ah->At : nullptr,
               ah ? ah->h : nullptr, ah ? ah->r : 0, n_pred};
#define HALO_QKV(NCH, TAIL) launch_timed("qkv_rows", qkv_rows<NCH, TAIL>, dim3(256 + n_pred), dim3(256), s, qa, d)
    if (whole) {
        switch (d) {
        case 4096: HALO_QKV(8, false); break;
        case 5120: HALO_QKV(10, false); break;
        default: HALO_QKV(16, false); break;
        }
    } else if (fast) {
        switch ((d + 1023) / 1024) {
        case 1: HALO_QKV(2, true); break;
        case 2: HALO_QKV(4, true); break;
        case 3: HALO_QKV(6, true); break;
        case 4: HALO_QKV(8, true); break;
        case 5: HALO_QKV(10, true); break;
        case 6: HALO_QKV(12, true); break;
        case 7: HALO_QKV(14, true); break;
        default: HALO_QKV(16, true); break;
        }
    } else {
        hipError_t e = launch_union(mask, 1, H, ws.dec.ulist, ws.dec.meta, s);
        if (e != hipSuccess) return e;
        launch_timed("qkv_rows_generic", qkv_rows_generic, dim3(512), dim3(256), s, qa, d,
                     (const int32_t *)ws.dec.ulist, (const int32_t *)ws.dec.meta);
    }
#undef HALO_QKV
    // Few enough chunks, perhaps made so by longer ones, are merged by the output projection (see kMergeChunks).
    const int len = pos + 1;
    const int most = H <= 16 ? kMergeChunks : whole ? std::min(kMergeChunks, 288 / H) : 6, longest = H <= 16 ? 512 : 256;
    int ch = 128;
    while (ch < longest && len > ch * most) ch *= 2;
    const int few = (len + ch - 1) / ch;
    if (fast && H <= kMergeHeads && few <= most) {
        const bf16_t *kc = (const bf16_t *)k_cache, *vc = (const bf16_t *)v_cache, *wo = (const bf16_t *)Wo;
        if (ch == 128)
            attn_partial<128><<<dim3(few, H), dim3(256), 0, s>>>(ws.q, kc, vc, mask, H, max_len, pos, ws.part);
        else if (ch == 256)
            attn_partial<256><<<dim3(few, H), dim3(512), 0, s>>>(ws.q, kc, vc, mask, H, max_len, pos, ws.part);
        else
            attn_partial<512><<<dim3(few, H), dim3(1024), 0, s>>>(ws.q, kc, vc, mask, H, max_len, pos, ws.part);
        switch (whole ? d : 0) {
        case 4096: launch_merge_out<4, bf16_t, true>(256, d, H, wo, mask, ws.part, few, (bf16_t *)y, ah, s); break;
        case 5120: launch_merge_out<5, bf16_t, true>(256, d, H, wo, mask, ws.part, few, (bf16_t *)y, ah, s); break;
        case 8192: launch_merge_out<8, bf16_t, true>(256, d, H, wo, mask, ws.part, few, (bf16_t *)y, ah, s); break;
        default:                                                 // as launch_down_t1_any deals the rows
            if (d < 4096)
                launch_merge_out<2, float, false>((d + 7) / 8, d, H, wo, mask, ws.part, few, (bf16_t *)y, ah, s);
            else
                launch_merge_out<4, float, false>((d + 15) / 16, d, H, wo, mask, ws.part, few, (bf16_t *)y, ah, s);
        }
        return hipGetLastError();
    }
    // The merge kernel asks for 32 chunks at a time, one round trip after the other; up to 32 heads a chunk is longer where there would be
    // more than 36.  A block, us, chunks of 128 / of 256 or 512: 32 heads, 6000 rows 36.4 / 36.1, 15 000 51.1 / 49.3; 16 heads, 15 000 31.1 / 27.6;
    // 8 heads, 8000 19.0 / 18.3; 25 heads, 5000 28.1 / 27.7; but 32 heads, 4200 34.4 / 34.6,
    // and 40 heads, 10 000 57.7 / 58.3.
    ch = kAttnChunk;
    while (H <= 32 && ch < 512 && len > ch * 36) ch *= 2;
    const int n_chunks = (len + ch - 1) / ch;
    {
        const bf16_t *kc = (const bf16_t *)k_cache, *vc = (const bf16_t *)v_cache;
        if (ch == 128)
            attn_partial<128><<<dim3(n_chunks, H), dim3(256), 0, s>>>(ws.q, kc, vc, mask, H, max_len, pos, ws.part);
        else if (ch == 256)
            attn_partial<256><<<dim3(n_chunks, H), dim3(512), 0, s>>>(ws.q, kc, vc, mask, H, max_len, pos, ws.part);
        else
            attn_partial<512><<<dim3(n_chunks, H), dim3(1024), 0, s>>>(ws.q, kc, vc, mask, H, max_len, pos, ws.part);
    }
    // the output projection is the FFN's down projection with heads as groups
    if (whole) {
        attn_combine<bf16_t><<<dim3(H), dim3(128), 0, s>>>(ws.part, mask, H, n_chunks,
                                                           reinterpret_cast<bf16_t *>(ws.dec.act));
        return launch_down_t1((const bf16_t *)Wo, d, H, mask, reinterpret_cast<const bf16_t *>(ws.dec.act),
                              (bf16_t *)y, s, ah);
    }
    attn_combine<float><<<dim3(H), dim3(128), 0, s>>>(ws.part, mask, H, n_chunks, ws.dec.act);
    return launch_down_t1_any((const bf16_t *)Wo, d, H, mask, (const float *)ws.dec.act, (bf16_t *)y, s, ah);
}

}  // namespace halo
