// Few tokens (2 <= T <= 16) on the matrix cores, rows of any multiple of 128 up to 8192 (paper Sec. II-A neuron groups;
// Sec. V-A 4-bit models): the gate/up projection over bf16 or 4-bit weights, and the down projection over 4-bit weights
// with activations in float32.
//
// The block is bound by streaming the union of the tokens' surviving groups from HBM, so everything else is kept out
// of the way of that stream:
//   - The token side does not move.  In gate/up a wave owns a slice of the reduction range for ALL of its workgroup's
//     rows, so the tokens' values of that slice stay in registers as matrix operands and the loop has no LDS read of them.
//   - A load instruction covers whole cache lines, 128 bytes of each of eight rows: lane l = (q, c, r) = (l / 16, l / 8 % 2,
//     l % 8) holds row r, 16 bytes 4 c + q of the line.
//   - Loads that are past the end of something carry an offset out of the descriptor's range, or no descriptor: they move
//     nothing, so no load stands behind a condition and the compiler can count how many are in flight.
// v_mfma_f32_16x16x32_bf16: A lane l = row l % 16 (a token), elements 8 (l / 16) .. + 7; B lane l = column l % 16, same
// elements; D lane l = column l % 16, rows (tokens) 4 (l / 16) .. + 3.  Which 8 of the 32 elements a lane group holds is free
// as long as A and B agree.
#include <type_traits>

#include "kernels.hpp"
#include "mask_device.hpp"
#include "mask_words.hpp"
#include "q4_codes.hpp"

namespace halo {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kStreamWaves = 8, kStreamBlocks = 256, kStreamTokens = 16;

__device__ __forceinline__ f32x4_t mfma16s(const u32x4 &a, const u32x4 &b, const f32x4_t &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// Which tokens keep which groups, in LDS: bit i of bits[h][g] = token 2 i + h.  One byte load per token and thread, all
// in flight together.
struct KeepBits {
    uint8_t bits[2][256];
    __device__ __forceinline__ void load(const uint8_t *__restrict__ mask, int T, int G, int tid)
    {
        const int g = tid & 255, h = tid >> 8;
        uint8_t v[kStreamTokens / 2];
#pragma unroll
        for (int i = 0; i < kStreamTokens / 2; ++i) v[i] = mask[(size_t)min(2 * i + h, T - 1) * G + min(g, G - 1)];
        unsigned b = 0;
#pragma unroll
        for (int i = 0; i < kStreamTokens / 2; ++i) b |= (v[i] != 0 && 2 * i + h < T && g < G ? 1u : 0u) << i;
        bits[h][g] = (uint8_t)b;
    }
    // (after a barrier) the union of the tokens' groups
    __device__ __forceinline__ MaskWords any(int lane) const
    {
        MaskWords mw;
        mw.count = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int g = k * kWave + lane;
            mw.w[k] = __ballot((bits[0][g] | bits[1][g]) != 0);
            mw.count += __popcll(mw.w[k]);
        }
        return mw;
    }
    __device__ __forceinline__ bool keeps(int t, int g) const { return (bits[t & 1][g] >> (t >> 1)) & 1; }
};

// lane l's value of v + lane (l ^ 8)'s: the two half lines of a row
__device__ __forceinline__ f32x4_t add_halves(const f32x4_t &v)
{
    return f32x4_t{xor_add<8>(v[0]), xor_add<8>(v[1]), xor_add<8>(v[2]), xor_add<8>(v[3])};
}

// the fixed-order dot product of the predictor (dot_order64) for two rows of x against one of At, rows of up to NCH * 512
// elements, eight chunks of all three requested at a time
template <int NCH>
__device__ __forceinline__ void dot_order64_two(const bf16_t *__restrict__ x0, const bf16_t *__restrict__ x1,
                                                const bf16_t *__restrict__ wp, int d, int lane, float &p0, float &p1)
{
    constexpr int kPart = NCH < 8 ? NCH : 8;
    const __amdgpu_buffer_rsrc_t b0 = buffer_of(x0), b1 = buffer_of(x1), bw = buffer_of(wp);
    p0 = p1 = 0.0f;
    for (int k0 = 0; k0 < NCH; k0 += kPart) {
        u32x4 v0[kPart], v1[kPart], wv[kPart];
#pragma unroll
        for (int k = 0; k < kPart; ++k) {
            // past the end: zeros on both sides leave the chain as it is
            const uint32_t at = ((k0 + k) * kWave + lane) * 8, voff = at < (uint32_t)d ? at * 2 : kOutOfRange;
            wv[k] = buffer_load16<kNt>(bw, voff, 0);
            v0[k] = buffer_load16<0>(b0, voff, 0);
            v1[k] = buffer_load16<0>(b1, voff, 0);
        }
#pragma unroll
        for (int k = 0; k < kPart; ++k) {
            float w[8], a[8], b[8];
            unpack8(wv[k], w);
            unpack8(v0[k], a);
            unpack8(v1[k], b);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p0 = __builtin_fmaf(a[e], w[e], p0);
                p1 = __builtin_fmaf(b[e], w[e], p1);
            }
        }
    }
    p0 = wave_sum(p0);
    p1 = wave_sum(p1);
}

// ---------------------------------------------------------------------------
// gate/up: 256 workgroups of eight waves, one per compute unit
// ---------------------------------------------------------------------------
// The union's neurons are dealt evenly over the workgroups, by the row; a workgroup walks its rows in tiles of TR.
// Wave v multiplies units nu v / 8 .. of every row (a unit = 128 bytes of a row: 64 bf16 values, or two quantisation
// blocks of 128 codes), at most U of them, and leaves its sums of a tile in LDS; they meet there once, at the end.
// A ring of NS units of gate and up is in flight per wave, over TB tiles where a tile has few units.
// Measured (us per launch): 4-bit, 70B shape, 8 tokens 58 with the next block's prediction on board, 50.5 without (a plain read 34; the
// former kernel 62 with it); bf16, 70B shape, 8 tokens 140 (a plain read 126; the former 150), d 2432, 66 groups, 8 tokens 18.2 (26.1).
// What bounds it: bf16, HBM (6.1 TB/s at the 70B shape); 4-bit, the loads that a compute unit has in flight (64 KiB: two units of four
// load instructions a wave): 54 us without the prediction under the tracer, 58 with the codes not converted, 47 with every row from
// cache, 36 with both, 24 with loads that move nothing (timing-only builds).  By the counters a SIMD's two waves spend 0.44 of the time in
// vector and 0.13 in matrix instructions.
// 4-bit codes: a block's sum of products meets the scale in float.  Rows that are whole multiples of 1024 take a code as bf16
// 128 + c and start a block at -136 * (sum of the tokens' values).  The others keep float32's precision (EXACT: such rows have
// no other fast path): a code is c - 8, exactly, so that nothing has to cancel, and the activation is stored in float32.
enum class Weights { Bf16, Codes, CodesExact };

template <Weights W, int U>
struct GateUpRing {
    static constexpr bool Q4 = W != Weights::Bf16, EXACT = W == Weights::CodesExact;
    typedef std::conditional_t<EXACT, float, bf16_t> Act;
    static constexpr int TR = Q4 ? 16 : 8;                       // rows of a tile
    static constexpr int L = Q4 ? 2 : 1;                         // load instructions per unit and matrix
    static constexpr int TB = Q4 ? (U == 1 ? 4 : U == 2 ? 2 : 1) : (U == 1 ? 8 : U == 2 ? 4 : U <= 4 ? 12 / U : U <= 6 ? 2 : 1);
    static constexpr int NS = Q4 ? (U == 4 ? 2 : U * TB) : (U > 11 ? U / 2 : U * TB);
    static constexpr int kXF = Q4 ? 8 : 2;                       // operand registers (of 16 bytes) of x per unit
    static constexpr int kNCH = Q4 ? U * 4 : (U + 1) / 2 * 2;    // 512-element chunks of the longest row
    static constexpr int kSums = Q4 ? 8 : 4;                     // floats a lane leaves of a tile
};

// From the loaded layout (a: tile rows r, b: rows 8 + r; lanes with bit 3 clear hold the unit's first block, the others its
// second) to the operand layout (lane = 16 q + row): c0 = first block, c1 = second.  Row i < 8 of c0 is a's own lane, row
// 8 + r is b's lane across bit 3; c1 the other way round.  Crossing bit 3 is a rotation by 8 within a row of 16 lanes (DPP
// row_ror:8); the bank mask writes lanes 8..15 (0xC) or 0..7 (0x3) and leaves the others as they were.
__device__ __forceinline__ uint32_t cross8_hi(uint32_t keep, uint32_t take)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)take, 0x128, 0xf, 0xC, false);
}
__device__ __forceinline__ uint32_t cross8_lo(uint32_t keep, uint32_t take)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)take, 0x128, 0xf, 0x3, false);
}

template <Weights W, int U>
__global__ __launch_bounds__(kStreamWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gate_up_stream(
    const bf16_t *__restrict__ x, int T, int d, int G, const void *__restrict__ Wg, const void *__restrict__ Wu,
    const bf16_t *__restrict__ Sg, const bf16_t *__restrict__ Su, const uint8_t *__restrict__ mask,
    typename GateUpRing<W, U>::Act *__restrict__ act, int act_stride, AheadPredDev ap)
{
    using R = GateUpRing<W, U>;
    constexpr bool Q4 = R::Q4, EXACT = R::EXACT, kOffset = Q4 && !EXACT;
    constexpr int TR = R::TR, L = R::L, TB = R::TB, NS = R::NS, kXF = R::kXF, kNCH = R::kNCH, kSums = R::kSums, gs = 128;
    constexpr int kElems = Q4 ? 256 : 64;                        // row elements of a unit
    static_assert((TB * U) % NS == 0, "a slot serves the same unit in every turn");
    extern __shared__ __attribute__((aligned(16))) float part[]; // [tile][wave][64 lanes][kSums]
    __shared__ KeepBits keep;
    __shared__ __attribute__((aligned(16))) float s_off[kOffset ? kStreamWaves * U * 2 : 1][16];    // -136 * sum of x, [block][token]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, q = lane >> 4, r = lane & 7, c = (lane >> 3) & 1;
    const int wg = blockIdx.x;

    keep.load(mask, T, G, tid);

    // paper Sec. III-B.3, Pred beside Load/Comp, one layer ahead: rows of the next block's first predictor layer, dealt
    // over the workgroups; a workgroup's (row, two tokens) over its waves
    const int j_lo = (int)((long long)ap.r * wg / kStreamBlocks), two = (T + 1) / 2;
    const int n_pairs = ap.n_pred ? ((int)((long long)ap.r * (wg + 1) / kStreamBlocks) - j_lo) * two : 0;
    auto predict = [&](int p) {
        const int j = j_lo + p / two, t = (p - p / two * two) * 2, t1 = min(t + 1, T - 1);
        float v0, v1;
        dot_order64_two<kNCH>(ap.x_next + (size_t)t * d, ap.x_next + (size_t)t1 * d, ap.At + (size_t)j * d, d, lane, v0, v1);
        if (lane == 0) ap.h[(size_t)t * ap.r + j] = v0 > 0.0f ? v0 : 0.0f;
        if (lane == 1 && t1 > t) ap.h[(size_t)t1 * ap.r + j] = v1 > 0.0f ? v1 : 0.0f;
    };
    // this wave's units
    const int nu = (d + kElems - 1) / kElems;
    const int first = nu * wave / kStreamWaves, cnt = nu * (wave + 1) / kStreamWaves - first;
    __syncthreads();                                             // keep
    const MaskWords uw = keep.any(lane);
    const int total = uw.count * gs;
    const int n0 = total * wg / kStreamBlocks, n1 = total * (wg + 1) / kStreamBlocks;      // at most 128 rows: two groups
    const int ntile = (n1 - n0 + TR - 1) / TR;
    const int u_first = n0 / gs, u_last = n1 > n0 ? (n1 - 1) / gs : u_first;
    const int g_first = n1 > n0 ? nth_group(uw, u_first, lane) : 0, g_last = n1 > n0 ? nth_group(uw, u_last, lane) : 0;

    const uint32_t row_bytes = Q4 ? d / 2 : d * 2;
    const uint32_t at = first * 128 + c * 64 + q * 16;           // this lane's bytes of a row's first unit
    // 4-bit rows of an odd number of blocks end in half a unit
    const int whole = Q4 && (first + cnt) * 256 > d ? cnt - 1 : cnt;
    const __amdgpu_buffer_rsrc_t bg = buffer_of(Wg), bu = buffer_of(Wu), bsg = buffer_of(Sg), bsu = buffer_of(Su),
                                 none = buffer_of(Wg, 0);
    auto row_at = [&](int n) -> uint32_t {                       // row n of the union's, or kOutOfRange
        const int u = n / gs;
        return n < n1 ? (uint32_t)((u == u_first ? g_first : g_last) * gs + (n - u * gs)) : kOutOfRange;
    };
    struct Slot {
        u32x4 g[L], u[L];
    };
    struct TileRows {
        uint32_t at[L];                                          // this lane's bytes of its rows' first unit: rows r and (4-bit) 8 + r
    };
    struct TileScales {
        uint32_t g, u;                                           // scales of both blocks of a unit
    };
    Slot slot[NS];
    TileRows row[TB], row_next[TB];
    TileScales scale[TB], scale_next[TB];
    auto rows_of = [&](int tile) {
        TileRows t;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const uint32_t rw = row_at(n0 + tile * TR + 8 * l + r);
            t.at[l] = rw != kOutOfRange ? rw * row_bytes + at : kOutOfRange;
        }
        return t;
    };
    auto load = [&](Slot &s, const TileRows &t, int u) {
        // (a unit that does not exist has no descriptor: no vector instruction is spent on the question)
        const __amdgpu_buffer_rsrc_t rg = u < cnt ? bg : none, ru = u < cnt ? bu : none;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            uint32_t voff = t.at[l];
            if (Q4 && U - u <= 2) voff = u >= whole && c ? kOutOfRange : voff;           // (cnt is U or U - 1 where it counts)
            s.g[l] = buffer_load16<kNt>(rg, voff, u * 128);
            s.u[l] = buffer_load16<kNt>(ru, voff, u * 128);
        }
    };
    // the scales of a tile's row i16: lane group q brings those of unit q
    auto load_scales = [&](int tile) {
        const int nb = d / kQ4Block, b = (first + q) * 2;
        const uint32_t rw = row_at(n0 + tile * TR + i16);
        const uint32_t v0 = rw != kOutOfRange && q < cnt ? (rw * nb + b) * 2 : kOutOfRange, v1 = b + 1 < nb ? v0 : kOutOfRange;
        TileScales t;
        t.g = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bsg, v0, 0, 0);
        t.u = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bsu, v0, 0, 0);
        t.g |= (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bsg, v1, 2, 0) << 16;
        t.u |= (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bsu, v1, 2, 0) << 16;
        return t;
    };
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) row[tb] = rows_of(tb);
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
        if (Q4) scale[tb] = load_scales(tb);
#pragma unroll
    for (int j = 0; j < NS; ++j) load(slot[j], row[j / U], j % U);
    __builtin_amdgcn_sched_barrier(0);
    if (wave < n_pairs) predict(wave);
    __builtin_amdgcn_sched_barrier(0);
    // the tokens' values that face the wave's units
    u32x4 xf[U][kXF];
    {
        // rows >= T repeat the last token, unused.  Of unit u: bf16, half line f; 4-bit, words f % 4 of the lane group's four
        // in block f / 4 (the last unit may have one block only); past the end: zeros
        const __amdgpu_buffer_rsrc_t bx = buffer_of(x);
        const uint32_t voff = (uint32_t)(((i16 < T ? i16 : T - 1) * d + first * kElems + q * (Q4 ? 32 : 8)) * 2);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int f = 0; f < kXF; ++f)
                xf[u][f] = buffer_load16<0>(bx, u < (Q4 && f >= 4 ? whole : cnt) ? voff : kOutOfRange,
                                            u * (kElems * 2) + (Q4 ? (f >> 2) * 256 + (f & 3) * 16 : f * 64));
    }
    const Q4Consts qk = q4_consts();
    if (kOffset) {
        // -136 * the sum of a token's values in a block: a matrix product with -136 everywhere (every column is the sum)
        const u32x4 m136 = {0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u};
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 4; ++k) s = mfma16s(xf[u][(kOffset ? b * 4 + k : 0)], m136, s);
                if (i16 == 0) *reinterpret_cast<f32x4_t *>(&s_off[(kOffset ? (wave * U + u) * 2 + b : 0)][4 * q]) = s;
            }
        // (a wave reads back its own entries only, and its LDS operations complete in order)
    }
    for (int t0 = 0; t0 < ntile; t0 += TB) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) row_next[tb] = rows_of(t0 + TB + tb);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
            if (Q4) scale_next[tb] = load_scales(t0 + TB + tb);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            // The last turn's tiles that do not exist are left out: without this they were multiplied, all zeros (what they would
            // ask for does not exist either).  Both projections, 4-bit, d 1024, 27 groups, 2 tokens 16.0 -> 13.9 us, d 2048, 44 groups
            // 17.9 -> 16.2; bf16, d 1536, 20 groups, 5 tokens 15.7 -> 14.9.
            if (TB > 1 && t0 + tb >= ntile) break;
            f32x4_t ag[2], au[2];                                // 4-bit: [0] only
#pragma unroll
            for (int h = 0; h < 2; ++h) ag[h] = au[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = tb * U + u;
                Slot &s = slot[j % NS];
                if constexpr (Q4) {
                    const uint32_t sg = (uint32_t)__builtin_amdgcn_ds_bpermute((u * 16 + i16) * 4, (int)scale[tb].g);
                    const uint32_t su = (uint32_t)__builtin_amdgcn_ds_bpermute((u * 16 + i16) * 4, (int)scale[tb].u);
                    f32x4_t tg[2], tu[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        tg[h] = tu[h] = EXACT ? f32x4_t{0.f, 0.f, 0.f, 0.f} : *reinterpret_cast<const f32x4_t *>(&s_off[kOffset ? (wave * U + u) * 2 + h : 0][4 * q]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const uint32_t vg = h ? cross8_lo(s.g[1][k], s.g[0][k]) : cross8_hi(s.g[0][k], s.g[1][k]);
                            const uint32_t vu = h ? cross8_lo(s.u[1][k], s.u[0][k]) : cross8_hi(s.u[0][k], s.u[1][k]);
                            tg[h] = mfma16s(xf[u][h * 4 + k], EXACT ? q4_word_signed(vg) : q4_word_bf16(vg, qk), tg[h]);
                            tu[h] = mfma16s(xf[u][h * 4 + k], EXACT ? q4_word_signed(vu) : q4_word_bf16(vu, qk), tu[h]);
                        }
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float fg = h ? bf16_hi(sg) : bf16_lo(sg), fu = h ? bf16_hi(su) : bf16_lo(su);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            ag[0][e] = __builtin_fmaf(fg, tg[h][e], ag[0][e]);
                            au[0][e] = __builtin_fmaf(fu, tu[h][e], au[0][e]);
                        }
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        ag[h] = mfma16s(xf[u][h], s.g[0], ag[h]);
                        au[h] = mfma16s(xf[u][h], s.u[0], au[h]);
                    }
                }
                // the slot's next unit: NS further along
                const int jn = j + NS;
                if (jn < TB * U)
                    load(s, row[jn < TB * U ? jn / U : 0], jn % U);
                else
                    load(s, row_next[(jn - TB * U) / U], jn % U);
                __builtin_amdgcn_sched_barrier(0);
            }
            {
                float *dst = part + (((t0 + tb) * kStreamWaves + wave) * 64 + lane) * kSums;
                if (Q4) {
                    *reinterpret_cast<f32x4_t *>(dst) = ag[0];
                    *reinterpret_cast<f32x4_t *>(dst + 4) = au[0];
                } else {
                    f32x4_t vg = ag[0], vu = au[0];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        vg[e] = c ? ag[1][e] : vg[e];
                        vu[e] = c ? au[1][e] : vu[e];
                    }
                    vg = add_halves(vg);
                    vu = add_halves(vu);
                    // lanes with c = 0 keep the gate sums, the others the up sums
                    f32x4_t v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = c ? vu[e] : vg[e];
                    *reinterpret_cast<f32x4_t *>(dst) = v;
                }
            }
        }
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            row[tb] = row_next[tb];
            if (Q4) scale[tb] = scale_next[tb];
        }
    }
    for (int p = wave + kStreamWaves; p < n_pairs; p += kStreamWaves) predict(p);
    __syncthreads();
    // a thread finishes one row for four tokens
    for (int id = tid; id < ntile * TR * 4; id += kStreamWaves * 64) {
        const int tile = id / (TR * 4), rr = id & (TR - 1), tq = id / TR & 3, n = n0 + tile * TR + rr;
        if (n >= n1 || 4 * tq >= T) continue;
        f32x4_t gt = {0.f, 0.f, 0.f, 0.f}, up = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kStreamWaves; ++w) {
            const float *p = part + ((tile * kStreamWaves + w) * 64 + tq * 16 + rr) * kSums;
            gt += *reinterpret_cast<const f32x4_t *>(p);
            up += *reinterpret_cast<const f32x4_t *>(p + (Q4 ? 4 : 32));
        }
        const int g = n / gs == u_first ? g_first : g_last;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 4 * tq + e;
            const float f = EXACT ? kQ4Signed : 1.0f;
            if (t < T) store_out(act + (size_t)t * act_stride + n, keep.keeps(t, g) ? silu_mul(f * gt[e], f * up[e]) : 0.0f);
        }
    }
}

// ---------------------------------------------------------------------------
// down over 4-bit weights, activations in float32: n_mask + up to 256 workgroups of eight waves
// ---------------------------------------------------------------------------
// The output rows are dealt over the workgroups in eights, at most RT tiles of sixteen to a workgroup; the waves take every
// eighth of the union's groups and meet in LDS.  A tile's codes of a group are 1 KiB of consecutive bytes, one load, in operand
// order.  An activation is multiplied as the sum of three bf16 values, its leading, middle and trailing eight bits -- all 24 of them --
// with codes that are c - 8 exactly, so that float32 sums are the only rounding.
// TL > 0, up to 2 TL tokens: a wave's lanes share the split: a load brings two tokens' 512 bytes, a lane splits its four values, and the pieces
// go through the wave's own LDS region into operand order.  TL = 0: operand order from memory, a lane splits the 32 values of its token's
// that it multiplies; sixteen tokens have nothing to share.  (With that for every number of tokens two of them paid for sixteen: both
// projections, us, d 3200, 75 groups, 2 tokens 27.1 -> 22.3, 8 tokens 37.3 -> 33.8; d 8064, 256 groups, 2 tokens 100 -> 87.)
// The first n_mask workgroups do not project: each computes the next block's scores, ranking and mask for one token (paper
// Sec. III-B.3, one layer ahead; dispatched first, it is the longest dependent chain).  DEPTH groups are in flight per wave.
template <int RT, int TL>
struct DownStep {
    static constexpr int DEPTH = TL == 0 ? 2 : RT * TL == 8 ? 3 : 4, kLoads = TL == 0 ? 8 : TL;
    u32x4 w[RT];
    f32x4_t a[kLoads];
    uint32_t sc[RT];
};

// four floats as the sum of three times four bf16 values
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split3(f32x4_t v, u32x2 (&piece)[3])
{
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t top = __builtin_amdgcn_perm(__float_as_uint(v[2 * i + 1]), __float_as_uint(v[2 * i]), 0x07060302u);
            piece[p][i] = top;
            const float a = bf16_lo(top), b = bf16_hi(top);      // (of an infinity nothing is left)
            v[2 * i] = p == 0 && v[2 * i] == a ? 0.0f : v[2 * i] - a;
            v[2 * i + 1] = p == 0 && v[2 * i + 1] == b ? 0.0f : v[2 * i + 1] - b;
        }
}

template <int RT, int TL>
__global__ __launch_bounds__(kStreamWaves * 64, 4) void down_q4_f32(
    int T, int d, int G, const uint32_t *__restrict__ Dq, const bf16_t *__restrict__ Ds, const uint8_t *__restrict__ mask,
    const float *__restrict__ act, int act_stride, bf16_t *__restrict__ y, int n_mask, AheadDev nx)
{
    using Step = DownStep<RT, TL>;
    constexpr int gs = 128, DEPTH = Step::DEPTH;
    constexpr int kPitch = gs * 2 + 16, kPlane = 2 * TL * kPitch;           // bytes of a token's row of pieces, of all rows
    constexpr int kRegion = 3 * kPlane > RT * 1024 ? 3 * kPlane : RT * 1024;
    struct Proj {
        KeepBits keep;
        int list[256];
        __attribute__((aligned(16))) unsigned char region[kStreamWaves][kRegion];   // a wave's pieces; at the end its sums
        // [16 token quad + row][token in quad]
        __device__ __forceinline__ float (*sums(int wave))[64][4] { return reinterpret_cast<float(*)[64][4]>(region[wave]); }
    };
    constexpr size_t kLds = sizeof(Proj) > sizeof(MaskShared) ? sizeof(Proj) : sizeof(MaskShared);
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    if ((int)blockIdx.x < n_mask) {
        const int t = blockIdx.x;
        mask_scores_block<kStreamWaves * 64, bf16_t, true>(
            *reinterpret_cast<MaskShared *>(lds), tid, nx.h + (size_t)t * nx.r, nx.Bt, nx.r, nx.scores + (size_t)t * G, G,
            nx.K, nx.prio_dev, nx.n_dev, nx.drop ? nx.drop + (size_t)t * nx.n_dev : nullptr,
            nx.order ? nx.order + (size_t)t * G : nullptr, nx.group_dev ? nx.group_dev + (size_t)t * G : nullptr,
            nx.mask + (size_t)t * G, nx.surv_idx ? nx.surv_idx + (size_t)t * nx.K : nullptr,
            nx.n_surv ? nx.n_surv + t : nullptr);
        return;
    }
    Proj &sh = *reinterpret_cast<Proj *>(lds);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, q = lane >> 4;
    const int nwg = gridDim.x - n_mask, wg = blockIdx.x - n_mask, eights = d / 8;
    const int row0 = eights * wg / nwg * 8, nrows = eights * (wg + 1) / nwg * 8 - row0;       // <= 16 RT
    sh.keep.load(mask, T, G, tid);
    __syncthreads();
    const MaskWords uw = sh.keep.any(lane);
    if (wave == 0) write_group_list(uw, lane, sh.list);
    __syncthreads();
    const int n_u = uw.count;
    const __amdgpu_buffer_rsrc_t bw = buffer_of(Dq), bs = buffer_of(Ds), ba = buffer_of(act), none = buffer_of(Dq, 0);
    // rows past the last token repeat it, unused
    uint32_t at_act[TL == 0 ? 1 : TL];
#pragma unroll
    for (int n = 0; n < (TL == 0 ? 1 : TL); ++n)
        at_act[n] = TL == 0 ? (uint32_t)((i16 < T ? i16 : T - 1) * act_stride + q * 32) * 4
                            : (uint32_t)(min(2 * n + (lane >> 5), T - 1) * act_stride + (lane & 31) * 4) * 4;
    unsigned char *mine = sh.region[wave];
    uint32_t at_w[RT], at_s[RT];                                 // this lane's bytes of a group's block and of its scales
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int j = row0 + rt * 16 + i16;
        const bool ok = rt * 16 + i16 < nrows;
        at_w[rt] = ok ? (uint32_t)j * 64 + q * 16 : kOutOfRange;
        at_s[rt] = ok ? (uint32_t)j * 2 : kOutOfRange;
    }
    // the wave's groups (at most 32), one to a lane: a group's id comes out of this register into a scalar one, where a read of
    // the list would put an LDS round trip in front of every group's loads
    const int my_group = sh.list[wave + kStreamWaves * (lane & 31)];
    auto request = [&](Step &s, int u) {                         // past the end: activations of the last group, no weights
        const bool yes = u < n_u;
        const uint32_t g = yes ? (uint32_t)__builtin_amdgcn_readlane(my_group, u / kStreamWaves) : 0u;
        const __amdgpu_buffer_rsrc_t rw = yes ? bw : none, rs = yes ? bs : none;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            s.w[rt] = buffer_load16<kNt>(rw, at_w[rt], g * (uint32_t)d * 64);
            s.sc[rt] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, at_s[rt], g * (uint32_t)d * 2, 0);
        }
#pragma unroll
        for (int n = 0; n < Step::kLoads; ++n)
            s.a[n] = __builtin_bit_cast(f32x4_t, buffer_load16<0>(ba, at_act[TL == 0 ? 0 : n], (uint32_t)((yes ? u : n_u - 1) * gs) * 4 + (TL == 0 ? n * 16 : 0)));
    };
    f32x4_t acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](const Step &s) {
        f32x4_t t[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) t[rt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if constexpr (TL > 0) {
            // (the region is the wave's own and its LDS operations complete in order, so no barrier is needed)
#pragma unroll
            for (int n = 0; n < TL; ++n) {
                u32x2 piece[3];
                split3(s.a[n], piece);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    *reinterpret_cast<u32x2 *>(mine + p * kPlane + (2 * n + (lane >> 5)) * kPitch + (lane & 31) * 8) = piece[p];
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {                            // word k: eight elements
            u32x4 piece[3];
            if constexpr (TL > 0) {
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    piece[p] = *reinterpret_cast<const u32x4 *>(mine + p * kPlane + (i16 & (2 * TL - 1)) * kPitch + (q * 32 + k * 8) * 2);
            } else {
                u32x2 lo[3], hi[3];
                split3(s.a[TL == 0 ? 2 * k : 0], lo);
                split3(s.a[TL == 0 ? 2 * k + 1 : 0], hi);
#pragma unroll
                for (int p = 0; p < 3; ++p) piece[p] = u32x4{lo[p][0], lo[p][1], hi[p][0], hi[p][1]};
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const u32x4 v = q4_word_signed(s.w[rt][k]);
#pragma unroll
                for (int p = 0; p < 3; ++p) t[rt] = mfma16s(piece[p], v, t[rt]);
            }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const float f = bf16_lo(s.sc[rt]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[rt][e] = __builtin_fmaf(f, t[rt][e], acc[rt][e]);
        }
    };
    if (wave < n_u) {
        Step s[DEPTH];
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) request(s[k], wave + k * kStreamWaves);
        for (int u = wave; u < n_u; u += DEPTH * kStreamWaves) {
#pragma unroll
            for (int k = 0; k < DEPTH; ++k) {
                if (u + k * kStreamWaves < n_u) consume(s[k]);
                request(s[k], u + (k + DEPTH) * kStreamWaves);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) *reinterpret_cast<f32x4_t *>(sh.sums(wave)[rt][lane]) = acc[rt];
    __syncthreads();
    // a thread finishes one row for one token
    for (int id = tid; id < RT * 256; id += kStreamWaves * 64) {
        const int rt = id >> 8, t = (id >> 4) & 15, rr = id & 15;
        if (t >= T || rt * 16 + rr >= nrows) continue;
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < kStreamWaves; ++w) v += sh.sums(w)[rt][(t >> 2) * 16 + rr][t & 3];
        y[(size_t)t * d + row0 + rt * 16 + rr] = f32_to_bf16(kQ4Signed * v);
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
bool stream_path_supported(int T, int d, int G, int gs)
{
    return T >= 2 && T <= kStreamTokens && gs == 128 && d % 128 == 0 && d <= 8192 && G <= 256;
}

template <Weights W, int U>
static hipError_t launch_gate_up(const bf16_t *x, int T, int d, int G, const void *Wg, const void *Wu, const bf16_t *Sg,
                                 const bf16_t *Su, const uint8_t *mask, void *act, const AheadPredDev &ap, hipStream_t s)
{
    // room for the sums of every tile that a workgroup can have
    using R = GateUpRing<W, U>;
    const auto bytes = [](int groups) {
        return (size_t)((groups * 128 + kStreamBlocks - 1) / kStreamBlocks + R::TR - 1) / R::TR * kStreamWaves * 64 * R::kSums * sizeof(float);
    };
    const hipError_t lds_ok = allow_lds<gate_up_stream<W, U>>((int)bytes(256));
    if (lds_ok != hipSuccess) return lds_ok;
    launch_timed_lds(R::Q4 ? "gate_up_q4_stream" : "gate_up_stream", gate_up_stream<W, U>, dim3(kStreamBlocks), dim3(kStreamWaves * 64),
                     bytes(G), s, x, T, d, G, Wg, Wu, Sg, Su, mask, (typename R::Act *)act, G * 128, ap);
    return hipGetLastError();
}

hipError_t launch_gate_up_stream(const bf16_t *x, int T, int d, int G, const bf16_t *Wg, const bf16_t *Wu, const uint8_t *mask,
                                 bf16_t *act, hipStream_t s, const AheadPredDev &ap)
{
#define HALO_CASE(U) \
    case U: return launch_gate_up<Weights::Bf16, U>(x, T, d, G, Wg, Wu, nullptr, nullptr, mask, act, ap, s)
    const int units = (d / 64 + kStreamWaves - 1) / kStreamWaves;
    switch (units > 12 ? (units + 1) / 2 * 2 : units) {
        HALO_CASE(1);
        HALO_CASE(2);
        HALO_CASE(3);
        HALO_CASE(4);
        HALO_CASE(5);
        HALO_CASE(6);
        HALO_CASE(7);
        HALO_CASE(8);
        HALO_CASE(9);
        HALO_CASE(10);
        HALO_CASE(11);
        HALO_CASE(12);
        HALO_CASE(14);
        HALO_CASE(16);
    default: return hipErrorInvalidValue;
    }
#undef HALO_CASE
}

bool q4_few_tokens_exact(int d) { return d % 1024 != 0; }

hipError_t launch_gate_up_q4_stream(const bf16_t *x, int T, int d, int G, const Q4Weights &w, const uint8_t *mask, void *act,
                                    hipStream_t s, const AheadPredDev &ap)
{
#define HALO_CASE(W, U) \
    case U: return launch_gate_up<W, U>(x, T, d, G, w.gate_codes, w.up_codes, w.gate_scales, w.up_scales, mask, act, ap, s)
    const int units = (d + 2047) / 2048;
    if (q4_few_tokens_exact(d)) {
        switch (units) {
            HALO_CASE(Weights::CodesExact, 1);
            HALO_CASE(Weights::CodesExact, 2);
            HALO_CASE(Weights::CodesExact, 3);
            HALO_CASE(Weights::CodesExact, 4);
        default: return hipErrorInvalidValue;
        }
    }
    switch (units) {
        HALO_CASE(Weights::Codes, 1);
        HALO_CASE(Weights::Codes, 2);
        HALO_CASE(Weights::Codes, 3);
        HALO_CASE(Weights::Codes, 4);
    default: return hipErrorInvalidValue;
    }
#undef HALO_CASE
}

template <int RT, int TL>
static hipError_t launch_down_f32(int T, int d, int G, const Q4Weights &w, const uint8_t *mask, const float *act, bf16_t *y,
                                  const AheadArgs *ah, hipStream_t s)
{
    const int n_mask = ah ? T : 0, blocks = d / 8 < kStreamBlocks ? d / 8 : kStreamBlocks;
    down_q4_f32<RT, TL><<<dim3(blocks + n_mask), dim3(kStreamWaves * 64), 0, s>>>(
        T, d, G, w.down_codes, w.down_scales, mask, act, G * 128, y, n_mask, ah ? ahead_dev(*ah) : AheadDev{});
    return hipGetLastError();
}

template <int RT>
static hipError_t launch_down_f32_by_tokens(int T, int d, int G, const Q4Weights &w, const uint8_t *mask, const float *act, bf16_t *y,
                                            const AheadArgs *ah, hipStream_t s)
{
    if (T <= 2) return launch_down_f32<RT, 1>(T, d, G, w, mask, act, y, ah, s);
    if (T <= 4) return launch_down_f32<RT, 2>(T, d, G, w, mask, act, y, ah, s);
    if (T <= 8) return launch_down_f32<RT, 4>(T, d, G, w, mask, act, y, ah, s);
    return launch_down_f32<RT, 0>(T, d, G, w, mask, act, y, ah, s);
}

hipError_t launch_down_q4_f32(int T, int d, int G, const Q4Weights &w, const uint8_t *mask, const float *act, bf16_t *y,
                              const AheadArgs *ah, hipStream_t s)
{
    const bool one = (d / 8 + kStreamBlocks - 1) / kStreamBlocks <= 2;       // at most 16 rows to a workgroup
    return one ? launch_down_f32_by_tokens<1>(T, d, G, w, mask, act, y, ah, s) : launch_down_f32_by_tokens<2>(T, d, G, w, mask, act, y, ah, s);
}

}  // namespace halo
