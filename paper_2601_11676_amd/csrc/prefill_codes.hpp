// 17 to 64 tokens over 4-bit weights: the codes become matrix operands in registers.
//
// A code is c in 0..15, its value s * (c - 8) with one scale s per row and block of 128 elements.  A matrix instruction multiplies (c - 8) / 16,
// exact in bf16 (q4_word_signed), and the finished block is scaled in float on its way into the running sum: three and a half vector instructions per
// pair of codes, where a value that is scaled, rounded to bf16 and parked in LDS for all waves takes seven, an LDS write and reads of twice the
// bytes.  (128 + c, less 136 times the sum of the token's elements, is half the conversion and gained 1 to 4 %, but its sums carry 17 times what the
// block is made of: rows that cancel were up to 400 times further from 64 bits than here, blocks over codes of 8 alone were not 0, and sums of a
// block's elements from 2^121 on overflowed.)
//
// Workgroup tile: 128 weight rows x 64 tokens, eight waves: two halves of the blocks (a wave takes every other block) times four quarters
// of the rows, gate (or lower) and up (upper) rows alike; a wave owns 32 x 64, N of its four 16-token tiles existing.  A step is 64
// elements of each of two blocks, a unit the two steps of a pair of blocks.  In LDS: three steps of token rows (128 bytes each) and three
// units of codes (64 bytes a row, 16-byte piece p of row r at p ^ ((r >> 2) & 3)) and scales.
//
// What bounds it: the instructions of a wave, one per four cycles, more than half of them the conversion and the scaling, and the barrier of a step.
// Pass in us, codes rounded to bf16 on their way into LDS (as for more tokens) against this: 17 tokens 7B 68.2 / 50.1, 13B 84.0 / 62.0, 70B 224.5 /
// 144.2; 33 tokens 13B 89.1 / 67.3, 48 of 70B 226.8 / 158.7, 64 of 13B 91.4 / 74.6; d 2048, 44 groups, 40 tokens 46.6 / 38.3; d 256, 4 groups, 17
// tokens 23.0 / 18.8.  With 128 + c: two such workgroups to a compute unit (rings of two steps and two units, 128 registers) took 189 us at 70B, 17
// tokens, where one took 150, four units of codes instead of three 151.  The scalar address work is kept to an addition per load (157 -> 150 there),
// and the barrier stands in the middle of a step, where the fragments of its second half have long been read.
#pragma once
#include "prefill_tiles.hpp"

namespace halo {

constexpr int kCodesTokens = 64;
constexpr int kCodesX = 2 * kCodesTokens * 128, kCodesRaw = 2 * 8192, kCodesScale = 2 * 512;
constexpr int kCodesSteps = 3, kCodesUnits = 3;                  // ring buffers
constexpr int kCodesRawBase = kCodesSteps * kCodesX, kCodesScaleBase = kCodesRawBase + kCodesUnits * kCodesRaw;
constexpr int kCodesBytes = kCodesScaleBase + kCodesUnits * kCodesScale;
static_assert(kCodesBytes + kTabGroups * kTabBytes / 2 <= 160 * 1024, "fits a compute unit");

// The 16-byte piece of a token row's 128 bytes that is parked at position v ^ (row & 7): a lane group q multiplies pieces 2 q and
// 2 q + 1, and the four groups' pieces of one instruction share a half of the row (free of bank conflicts).
__device__ __forceinline__ int codes_piece(int v) { return (v & 3) * 2 + (v >> 2); }

// What a wave owns of the tile: half of the blocks, quarter of the rows; its 16-row tile m of the workgroup's eight.
struct CodesPart {
    int ks, rw;
    __device__ __forceinline__ explicit CodesPart(int wave) : ks(wave & 1), rw(wave >> 1) {}
    __device__ __forceinline__ int row_tile(int m) const { return 4 * m + rw; }
};

// The steps of a tile over n_units units: total[m][n] = sum over the wave's blocks, over kQ4Signed.
// load_x(half, buf): token rows of three steps on, that half of its unit, into ring buffer buf (two loads of every wave).  load_unit(): end of
// the first step of a unit; requests the next but one (EV loads of every wave), and load_x turns to it.
// upper(j): the scale of rows 4 q + j is the upper half of its word.
template <int N, int EV, typename LoadX, typename LoadUnit, typename Upper>
__device__ __forceinline__ void multiply_codes(f32x4_t (&total)[2][N], unsigned char *ring, int n_units, int wave, int lane,
                                               LoadX load_x, LoadUnit load_unit, Upper upper)
{
    const CodesPart part(wave);
    const int i16 = lane & 15, q = lane >> 4;
    const unsigned char *xbase = ring + part.ks * (kCodesTokens * 128) + i16 * 128;
    const int xoff[2] = {(q ^ (i16 & 7)) * 16, ((4 + q) ^ (i16 & 7)) * 16};
    auto read_b = [&](u32x4 &f, int n, int t, int buf) __attribute__((always_inline)) {
        f = *reinterpret_cast<const u32x4 *>(xbase + buf * kCodesX + n * 2048 + xoff[t]);
    };
    const unsigned char *cbase = ring + kCodesRawBase + part.ks * 8192 + i16 * 64 + (q & 1) * 8;
    const int coff[2] = {((q >> 1) ^ ((i16 >> 2) & 3)) * 16, ((2 + (q >> 1)) ^ ((i16 >> 2) & 3)) * 16};
    auto read_c = [&](uint2 &c, int m, int half, int ub) __attribute__((always_inline)) {
        c = *reinterpret_cast<const uint2 *>(cbase + ub * kCodesRaw + part.row_tile(m) * 1024 + coff[half]);
    };
    f32x4_t blk[2][N];
    u32x4 b0[N], b1[N], a, sc[2];
    uint2 c[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        read_c(c[m], m, 0, 0);
        sc[m] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int n = 0; n < N; ++n) total[m][n] = blk[m][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int n = 0; n < N; ++n) read_b(b0[n], n, 0, 0);
    a = q4_word_signed(c[0].x);
    uint32_t sel[2] = {0u, 0u};                                  // which half of a word of scales, rows 4 q + j with even and odd j
    auto fold = [&](int m) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // a half of the word, as float: bytes 3 2 or 1 0, above two zero bytes
            const float f = __uint_as_float(__builtin_amdgcn_perm(sc[m][j], 0u, sel[j & 1]));
#pragma unroll
            for (int n = 0; n < N; ++n) total[m][n][j] = __builtin_fmaf(f, blk[m][n][j], total[m][n][j]);
        }
    };
    int buf = 0, ub = 0;                                         // ring buffers of the step and of the unit
    // A step is cut in two: its first 32 elements of a block are multiplied while the fragments of the others are read, then, behind
    // the barrier, the others while the next step's are.  What a row tile's conversion and scaling need stands in front of
    // the matrix instructions of the one before or behind those of the one after.
    auto step = [&](auto second_c) __attribute__((always_inline)) {
        constexpr bool second = decltype(second_c)::value;       // second half of the unit's blocks
        const int nbuf = buf == kCodesSteps - 1 ? 0 : buf + 1, nub = ub == kCodesUnits - 1 ? 0 : ub + 1;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
#pragma unroll
            for (int n = m * N; n < (m + 1) * N && n < N; ++n) read_b(b1[n], n, 1, buf);
            const u32x4 w = a;
            a = q4_word_signed(m == 0 ? c[1].x : c[0].y);
            if (m == 0 && !second) fold(1);                      // (of the unit before; at first: nothing to scale)
#pragma unroll
            for (int n = 0; n < N; ++n) blk[m][n] = mfma16p(w, b0[n], second ? blk[m][n] : f32x4_t{0.f, 0.f, 0.f, 0.f});
            __builtin_amdgcn_sched_barrier(0);
        }
        // the rows of step s+2 may still be on their way, and the unit requested last (in step s-1 or s-2); everybody has read step s
        wait_loads<2 + EV>();
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            read_c(c[m], m, second ? 0 : 1, second ? nub : ub);
#pragma unroll
            for (int n = m * N; n < (m + 1) * N && n < N; ++n) read_b(b0[n], n, 0, nbuf);
            const u32x4 w = a;
            a = q4_word_signed(m == 0 ? c[1].y : c[0].x);
            if (m == 0) load_x(!second, buf);
            if (m == 0 && second) {
                sel[0] = upper(0) ? 0x07060c0cu : 0x05040c0cu;
                sel[1] = upper(1) ? 0x07060c0cu : 0x05040c0cu;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    sc[i] = *reinterpret_cast<const u32x4 *>(ring + kCodesScaleBase + ub * kCodesScale + part.row_tile(i) * 128 + part.ks * 64 + q * 16);
            }
            if (m == 1 && second) fold(0);
#pragma unroll
            for (int n = 0; n < N; ++n) blk[m][n] = mfma16p(w, b1[n], blk[m][n]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (second)
            ub = nub;
        else
            load_unit();
        buf = nbuf;
    };
    for (int e = 0; e < n_units; ++e) {
        step(std::false_type{});
        step(std::true_type{});
    }
    fold(1);
    wait_loads<0>();                                             // (of loads that move nothing)
    __syncthreads();                                             // every wave is done with the rings
}

// The two halves of the blocks meet in LDS: of token tiles by turns a wave keeps one and hands the other to its partner (wave ^ 1).
template <int N, int KS_HALF>
__device__ __forceinline__ void meet_codes(f32x4_t (&total)[2][N], unsigned char *ring, int wave, int lane)
{
    constexpr int H = (N + 1) / 2;
    unsigned char *mine = ring + wave * (2 * H * 1024) + lane * 16;
    const unsigned char *theirs = ring + (wave ^ 1) * (2 * H * 1024) + lane * 16;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < N; ++n)
            if ((n & 1) != KS_HALF) *reinterpret_cast<f32x4_t *>(mine + (m * H + (n >> 1)) * 1024) = total[m][n];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < N; ++n)
            if ((n & 1) == KS_HALF) total[m][n] += *reinterpret_cast<const f32x4_t *>(theirs + (m * H + (n >> 1)) * 1024);
}

// body(N) with as many 16-token tiles as `tokens` ask for
template <typename Body>
__device__ __forceinline__ void with_token_tiles(int tokens, Body body)
{
    if (tokens > 48)
        body(std::integral_constant<int, 4>{});
    else if (tokens > 32)
        body(std::integral_constant<int, 3>{});
    else if (tokens > 16)
        body(std::integral_constant<int, 2>{});
    else
        body(std::integral_constant<int, 1>{});
}

// Wg, Wu: code words [ffn][d/8].  T <= 64.
__device__ __forceinline__ void gate_up_codes(const bf16_t *__restrict__ x, int T, int d, int G, const unsigned char *__restrict__ Wg,
                                              const unsigned char *__restrict__ Wu, const bf16_t *__restrict__ Sg,
                                              const bf16_t *__restrict__ Su, const int32_t *__restrict__ tok_list,
                                              const int32_t *__restrict__ tok_cnt, bf16_t *__restrict__ act)
{
    constexpr int gs = 128, EV = 3;
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CodesPart part(wave);
    const int i16 = lane & 15, q = lane >> 4;
    // one or no tile per group, numbered as in gate_up_pf_ring
    auto tiles_of = [](int n) { return n > 0 ? 1 : 0; };
    const int n_items = 2 * count_tiles(tok_cnt, G, lane, tiles_of);
    const int per_die = (n_items + 7) >> 3;
    const int die = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int item = __builtin_amdgcn_readfirstlane(die * per_die + slot);
    if (slot >= per_die || item >= n_items) return;              // uniform for the workgroup
    const int nt = item & 1;
    const int2 tile = find_tile(tok_cnt, G, item >> 1, lane, tiles_of);
    const int g = __builtin_amdgcn_readfirstlane(tile.x);
    const int cnt = __builtin_amdgcn_readfirstlane(tok_cnt[g]);
    const int32_t *list = tok_list + (size_t)g * T;

    const int nb = d / kQ4Block, nu = (nb + 1) / 2;              // blocks, units
    const int unit0 = (die * nu) >> 3;                           // the dies start at different places, as in gate_up_pf_ring
    const int br = lane >> 3, piece = codes_piece((lane & 7) ^ br);
    // the wave loads rows 8 wave .. + 7 of the tile
    const int sl = wave * 8 + br;
    const uint32_t off_x = sl < cnt ? (uint32_t)(list[sl] * d + piece * 8) * 2u : kNoRow;
    // its 16 rows are gate rows (waves 0..3) or up rows; one load covers 16 rows x 64 bytes
    const size_t q_row0 = (size_t)g * gs + nt * 64 + (wave & 3) * 16;
    const uint32_t off_c = (uint32_t)((lane >> 2) * (d / 2) + ((lane & 3) ^ ((lane >> 4) & 3)) * 16);
    // the aligned pair of scales that holds the one of row (lane & 15) in block lane / 16 of a unit
    const uint32_t off_p = (uint32_t)(((lane & 15) * nb + (lane >> 4 & 1)) & ~1) * 2u;
    srd_t srd_x[2], srd_c[2];                                    // empty where there is no block
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        srd_x[ks] = make_srd(x, true);
        srd_c[ks] = make_srd((wave < 4 ? Wg : Wu) + q_row0 * (d / 2), true);
    }
    srd_t srd_s = make_srd((wave < 4 ? Sg : Su) + q_row0 * nb, true);
    const uint32_t ring0 = (uint32_t)(size_t)ring, xdst = ring0 + wave * 1024, cdst = ring0 + kCodesRawBase + wave * 1024;
    const uint32_t end = (uint32_t)nu * 512u;
    uint32_t at = (uint32_t)unit0 * 512u;                        // the unit's place in a row of x, bytes
    int left = nu, rb = 0;                                       // units from it on; buffer of the unit that is requested next
    auto load_x = [&](bool half, int b) __attribute__((always_inline)) {
        load_to_lds16_at<0>(srd_x[0], off_x, at + (half ? 128u : 0u), xdst + b * kCodesX);
        load_to_lds16_at<kCodesTokens * 128>(srd_x[1], off_x, at + (half ? 384u : 256u), xdst + b * kCodesX);
    };
    auto request = [&]() __attribute__((always_inline)) {
        const bool half_unit = at + 256u >= (uint32_t)nb * 256u;
        srd_x[0].z = srd_c[0].z = srd_s.z = (uint32_t)__builtin_amdgcn_readfirstlane(left > 0 ? kAnySize : 0u);
        srd_x[1].z = srd_c[1].z = (uint32_t)__builtin_amdgcn_readfirstlane(half_unit ? 0u : srd_x[0].z);
        load_to_lds16_at<0, true>(srd_c[0], off_c, at >> 2, cdst + rb * kCodesRaw);
        load_to_lds16_at<8192, true>(srd_c[1], off_c, (at >> 2) + 64u, cdst + rb * kCodesRaw);
        load_to_lds_lanes<4>(0xffffffffull, srd_s, half_unit && lane >= 16 ? kNoRow : off_p, (at >> 9) * 4u,
                             ring0 + kCodesScaleBase + rb * kCodesScale + wave * 128);
        rb = rb == kCodesUnits - 1 ? 0 : rb + 1;
    };
    auto load_unit = [&]() __attribute__((always_inline)) {
        at = at + 512u == end ? 0u : at + 512u;
        --left;
        request();
    };
    auto upper = [&](int j) { return ((((nb & j) & 1) + part.ks) & 1) != 0; };
    request();
    load_x(false, 0);
    load_x(true, 1);
    load_unit();
    load_x(false, 2);
    wait_loads<4 + EV>();
    __syncthreads();
    with_token_tiles(cnt, [&](auto n_c) __attribute__((always_inline)) {
        constexpr int N = decltype(n_c)::value;
        f32x4_t total[2][N];
        multiply_codes<N, EV>(total, ring, nu, wave, lane, load_x, load_unit, upper);
        bf16_t *act_row0 = act + (size_t)g * T * gs + nt * 64;
        auto put = [&](auto half) __attribute__((always_inline)) {
            constexpr int KH = decltype(half)::value;
            meet_codes<N, KH>(total, ring, wave, lane);
#pragma unroll
            for (int n = KH; n < N; n += 2) {
                const int s = n * 16 + i16;
                const f32x4_t gt = kQ4Signed * total[0][n], up = kQ4Signed * total[1][n];
                const uint32_t lo = (uint32_t)f32_to_bf16(silu_mul_fast(gt[0], up[0])) | ((uint32_t)f32_to_bf16(silu_mul_fast(gt[1], up[1])) << 16);
                const uint32_t hi = (uint32_t)f32_to_bf16(silu_mul_fast(gt[2], up[2])) | ((uint32_t)f32_to_bf16(silu_mul_fast(gt[3], up[3])) << 16);
                if (s < cnt) *reinterpret_cast<uint2 *>(act_row0 + (size_t)s * gs + part.rw * 16 + 4 * q) = make_uint2(lo, hi);
            }
        };
        if (part.ks == 0)
            put(std::integral_constant<int, 0>{});
        else
            put(std::integral_constant<int, 1>{});
    });
}

// Wd: code words [G][d][16]; rows: the row table.  T <= 64: one token tile.
__device__ __forceinline__ void down_codes(int T, int d, int G, int splits, const unsigned char *__restrict__ Wd,
                                           const bf16_t *__restrict__ Sd, const int16_t *__restrict__ rows,
                                           const bf16_t *__restrict__ act, float *__restrict__ partial, bf16_t *__restrict__ y)
{
    constexpr int EV = 4, kTab = kTabBytes / 2;                  // bytes of the table's entries of a unit
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CodesPart part(wave);
    const int i16 = lane & 15, q = lane >> 4;
    DownItem it;
    if (!down_item<true, kCodesTokens>(T, d, G, splits, it)) return;
    const int j0 = it.j0, g_lo = it.g_lo;
    const int ng = it.g_hi - g_lo, nu = (ng + 1) / 2;            // groups of the range, units: a block is a group
    const int br = lane >> 3, piece = codes_piece((lane & 7) ^ br);
    const uint32_t ring0 = (uint32_t)(size_t)ring;
    const int pitch = prefill_row_pitch(T);
    // the wave's eight entries of the row table for both groups of a unit, lane ks (past the table's end its last eight again; of a
    // group past the range none): requested three units before the unit's codes
    const uint32_t off_t = (uint32_t)(min(wave * 8, pitch - 8) + (lane & 1) * pitch) * 2u;
    srd_t srd_tab = make_srd(rows, true);
    uint32_t tab_at = (uint32_t)(g_lo * pitch) * 2u;
    int tab_left = ng;                                           // groups of the range from the unit's first on
    auto request_table = [&](int b) __attribute__((always_inline)) {
        srd_tab.z = (uint32_t)__builtin_amdgcn_readfirstlane(tab_left > 0 ? kAnySize : 0u);
        load_to_lds_lanes<16>(tab_left == 1 ? 1ull : 3ull, srd_tab, off_t, tab_at, ring0 + kCodesBytes + b * kTab + wave * 32);
        tab_at += (uint32_t)(2 * pitch) * 2u;
        tab_left -= 2;
    };
    auto entry = [&](int b, int ks, int r) -> int {              // table buffer b = unit % kTabGroups
        return reinterpret_cast<const int16_t *>(ring + kCodesBytes + b * kTab + wave * 32)[ks * 8 + r];
    };
    // the unit: where its groups' token rows and codes lie, their descriptors empty where there is no group
    uint32_t off_a[2];
    srd_t srd_a[2], srd_c[2];
    unsigned long long a_at = (unsigned long long)(act + (size_t)g_lo * T * 128);
    unsigned long long c_at = (unsigned long long)(Wd + ((size_t)g_lo * d + j0 + wave * 16) * 64);
    const unsigned long long a_step = (unsigned long long)T * 256u, c_step = (unsigned long long)d * 64u;
    const uint32_t off_c = (uint32_t)((lane >> 2) * 64 + ((lane & 3) ^ ((lane >> 4) & 3)) * 16);
    const uint32_t off_p = (uint32_t)((lane >> 4 & 1) * d + j0 + wave * 16 + (lane & 14)) * 2u;
    srd_t srd_s = make_srd(Sd, true);
    uint32_t s_at = (uint32_t)(g_lo * d) * 2u;
    int left = ng, rb = 0;                                       // groups from it on; buffer of the unit that is requested next
    const uint32_t xdst = ring0 + wave * 1024, cdst = ring0 + kCodesRawBase + wave * 1024;
    auto load_x = [&](bool half, int b) __attribute__((always_inline)) {
        load_to_lds16_at<0>(srd_a[0], off_a[0], half ? 128u : 0u, xdst + b * kCodesX);
        load_to_lds16_at<kCodesTokens * 128>(srd_a[1], off_a[1], half ? 128u : 0u, xdst + b * kCodesX);
    };
    auto request = [&](int tab) __attribute__((always_inline)) { // its table is in buffer tab
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            off_a[ks] = (uint32_t)(entry(tab, ks, br) * 128 + piece * 8) * 2u;
            srd_a[ks] = make_srd((const void *)(a_at + ks * a_step), left > ks);
            srd_c[ks] = make_srd((const void *)(c_at + ks * c_step), left > ks);
        }
        load_to_lds16_at<0>(srd_c[0], off_c, 0, cdst + rb * kCodesRaw);
        load_to_lds16_at<8192>(srd_c[1], off_c, 0, cdst + rb * kCodesRaw);
        srd_s.z = srd_c[0].z;
        load_to_lds_lanes<4>(0xffffffffull, srd_s, left == 1 && lane >= 16 ? kNoRow : off_p, s_at,
                             ring0 + kCodesScaleBase + rb * kCodesScale + wave * 128);
        rb = rb == kCodesUnits - 1 ? 0 : rb + 1;
    };
    int tb = 0;                                                  // the unit's table
    auto load_unit = [&]() __attribute__((always_inline)) {
        left -= 2;
        a_at += 2 * a_step;
        c_at += 2 * c_step;
        s_at += (uint32_t)(2 * d) * 2u;
        request_table(tb);                                       // the unit four on takes the place of the one that was
        tb = (tb + 1) & 3;
        request(tb);
    };
    auto upper = [&](int j) { return j != 0; };
#pragma unroll
    for (int e = 0; e < kTabGroups; ++e) request_table(e);
    wait_loads<0>();                                             // each wave its own entries
    request(0);
    load_x(false, 0);
    load_x(true, 1);
    load_unit();
    load_x(false, 2);
    wait_loads<4 + EV>();
    __syncthreads();
    float *out = partial ? partial + (size_t)it.split * T * d : nullptr;
    with_token_tiles(T, [&](auto n_c) __attribute__((always_inline)) {
        constexpr int N = decltype(n_c)::value;
        f32x4_t total[2][N];
        multiply_codes<N, EV>(total, ring, nu, wave, lane, load_x, load_unit, upper);
        auto put = [&](auto half) __attribute__((always_inline)) {
            constexpr int KH = decltype(half)::value;
            meet_codes<N, KH>(total, ring, wave, lane);
#pragma unroll
            for (int n = KH; n < N; n += 2) {
                const int t = n * 16 + i16;
                if (t < T) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const f32x4_t v = kQ4Signed * total[m][n];
                        const size_t at = (size_t)t * d + j0 + part.row_tile(m) * 16 + 4 * q;
                        if (out) {
                            *reinterpret_cast<f32x4_t *>(out + at) = v;
                        } else {
                            const uint32_t lo = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
                            const uint32_t hi = (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16);
                            *reinterpret_cast<uint2 *>(y + at) = make_uint2(lo, hi);
                        }
                    }
                }
            }
        };
        if (part.ks == 0)
            put(std::integral_constant<int, 0>{});
        else
            put(std::integral_constant<int, 1>{});
    });
}

}  // namespace halo
