// What the many-token kernels share: the numbering of their tiles and the row table.
#pragma once
#include <type_traits>

#include "kernels.hpp"
#include "lds_loads.hpp"
#include "q4_codes.hpp"

namespace halo {

constexpr int kRingWaves = 8;
constexpr int kTabGroups = 4, kTabBytes = 512;                   // entries of the row table in LDS: groups, or pairs of them; bytes of one

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4_t mfma16p(const u32x4 &a, const u32x4 &b, const f32x4_t &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                   __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// row table [G][row_pitch]: T rounded up to 8
__host__ __device__ inline int prefill_row_pitch(int T) { return (T + 7) & ~7; }

// Token tiles are numbered group by group (group g has ceil(cnt[g] / tile_tokens) of them), and only
// tiles that exist get a number, so the working workgroups are consecutive.  Called by whole waves;
// results are the same in every lane.
__device__ __forceinline__ int wave_inclusive_sum(int n, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(n, off);
        if (lane >= off) n += v;
    }
    return n;
}

// tiles(n): the tiles of a group that n tokens keep
template <typename Tiles>
__device__ __forceinline__ int count_tiles(const int32_t *__restrict__ tok_cnt, int G, int lane, Tiles tiles)
{
    int total = 0;
    for (int g0 = 0; g0 < G; g0 += 64) {
        const int g = g0 + lane;
        const int n = g < G ? tiles(tok_cnt[g]) : 0;
        total += __shfl(wave_inclusive_sum(n, lane), 63);
    }
    return total;
}

// group and tile within the group of tile number `target` (< count_tiles)
template <typename Tiles>
__device__ __forceinline__ int2 find_tile(const int32_t *__restrict__ tok_cnt, int G, int target, int lane, Tiles tiles)
{
    int base = 0;
    for (int g0 = 0; g0 < G; g0 += 64) {
        const int g = g0 + lane;
        const int n = g < G ? tiles(tok_cnt[g]) : 0;
        const int incl = wave_inclusive_sum(n, lane);
        const int total = __shfl(incl, 63);
        if (target < base + total) {
            const unsigned long long m = __ballot(target < base + incl);
            const int l = __ffsll((long long)m) - 1;
            const int excl = __shfl(incl - n, l);
            return make_int2(g0 + l, target - base - excl);
        }
        base += total;
    }
    return make_int2(-1, 0);
}

// a workgroup's part of the down projection: outputs j0 .. + 127, tokens t0 .. + NTOK - 1, groups g_lo .. g_hi - 1, which is range
// `split` of the groups; false: none
struct DownItem {
    int j0, t0, g_lo, g_hi, split;
};
template <bool Q4, int NTOK>
__device__ __forceinline__ bool down_item(int T, int d, int G, int splits, DownItem &it)
{
    // work items: (token tile, group range, output tile) triples; a die gets a consecutive run of them
    const int n_ot = d / 128;
    const int n_tt = (T + NTOK - 1) / NTOK;
    const int n_items = n_ot * n_tt * splits;
    const int per_die = (n_items + 7) >> 3;
    const int die = blockIdx.x & 7, dslot = blockIdx.x >> 3;
    const int item = die * per_die + dslot;
    if (dslot >= per_die || item >= n_items) return false;       // uniform for the workgroup
    // The items of a die are the token tiles of consecutive output tiles of one range: a tile of Wd is fetched from memory by the first
    // and found in the die's L2 by the others, which walk the groups beside it, and so are the act rows of a step, whatever the
    // number of token tiles.  (Where a die's items shared one token tile's act rows instead, above two token tiles, every die fetched Wd for
    // itself.  Pass in us: 600 tokens of the 70B shape 765 -> 705, 1000 910 -> 887, 1500 1297 -> 1260, 800 of 13B 296 -> 291, 900 of 7B 215 -> 209.)
    // A narrow layer's Wd, up to 6 MB in bf16, is mostly in a die's L2 anyhow: there its items share a token tile's act rows, above two token tiles
    // and where such rows, 64 KiB a group, fit beside it.  Wd / act rows shared, us a pass, half of the groups kept: d 512, 40 groups, 600, 800,
    // 1000, 1500, 2000 tokens 47.1 / 45.0, 54.4 / 51.7, 54.9 / 51.6, 58.6 / 58.9, 66.6 / 67.3; d 640, 24 groups, 800, 1000 54.5 / 51.3, 49.6 / 48.0;
    // d 1024, 24 groups, 800, 2000 57.3 / 56.4, 67.7 / 69.3 (a tenth kept 58.9 / 55.6, 66.2 / 67.0).  Past the line: d 256, 96 groups, 600, 800, 2000
    // 49.9 / 51.3, 52.5 / 53.9, 90.0 / 90.2; d 1536, 32 groups, 800, 1500 69.9 / 70.7, 81.9 / 82.6; d 2048, 24 groups, 600 70.6 / 72.1.  Over codes,
    // a quarter of the bytes, it is level at d 1024, 24 groups, and 77.1 / 77.9 at d 2048.
    int ttile;
    if (Q4 || n_tt <= 2 || G > 48 || G * d > 24 * 1024) {
        ttile = item % n_tt;
        const int rest = item / n_tt;
        it.split = rest / n_ot;
        it.j0 = (rest - it.split * n_ot) * 128;
    } else {
        const int pair = item / n_ot;
        it.j0 = (item - pair * n_ot) * 128;
        ttile = pair / splits;
        it.split = pair - ttile * splits;
    }
    it.t0 = ttile * NTOK;
    it.g_lo = (int)((long long)it.split * G / splits);
    it.g_hi = (int)((long long)(it.split + 1) * G / splits);
    return true;
}

}  // namespace halo
