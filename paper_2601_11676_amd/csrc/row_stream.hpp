// Weight rows held in registers as they were loaded, for the kernels that stream them one wave per row (bf16):
// a neuron's gate row and up row, or two independent rows.
#pragma once
#include "common.hpp"

namespace halo {

// Where a lane's pieces of a row lie: 16-byte piece 64 k + lane of the row, k = 0 .. NCH-1.
// TAIL = false: rows of exactly NCH * 512 elements.  TAIL = true: any length d (a multiple of 8) with
// (NCH - 2) * 512 < d <= NCH * 512: pieces past the end exist in the last two chunks only.  Their loads go to
// the row's first piece, and keep() puts zeros in their place where the registers are USED -- a select next to
// the load would wait for it.
template <int NCH, bool TAIL>
struct RowLanes {
    int len;
    int at[2] = {0, 0};                     // TAIL: piece index of the last two chunks
    bool ok[2] = {true, true};
    __device__ __forceinline__ RowLanes(int d, int lane) : len(TAIL ? d : NCH * 512)
    {
        if constexpr (TAIL) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int piece = (NCH - 2 + k) * kWave + lane;
                ok[k] = piece * 8 < d;
                at[k] = ok[k] ? piece : 0;
            }
        }
    }
    __device__ __forceinline__ int piece(int k, int lane) const
    {
        return TAIL && k >= NCH - 2 ? at[k - (NCH - 2)] : k * kWave + lane;
    }
    __device__ __forceinline__ u32x4 keep(const u32x4 &v, int k) const
    {
        return TAIL && k >= NCH - 2 && !ok[k - (NCH - 2)] ? u32x4{0u, 0u, 0u, 0u} : v;
    }
    __device__ __forceinline__ size_t row(size_t r) const { return r * (size_t)(TAIL ? len : NCH * 512); }
};

// the fixed-order dot product of the predictor (dot_order64_fixed) for such a row: pieces past the end are zeros on
// both sides and leave the chains as they are
template <int NCH, bool TAIL>
__device__ __forceinline__ float dot_order64_row(const bf16_t *__restrict__ xp, const bf16_t *__restrict__ wp,
                                                 const RowLanes<NCH, TAIL> &rl, int lane)
{
    if constexpr (!TAIL) {
        return dot_order64_fixed<NCH * 512>(xp, wp, lane);
    } else {
        u32x4 xv[NCH], wv[NCH];
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            xv[k] = reinterpret_cast<const u32x4 *>(xp)[rl.piece(k, lane)];
            wv[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(wp) + rl.piece(k, lane));
        }
        float p = 0.0f;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            float a[8], b[8];
            unpack8(rl.keep(xv[k], k), a);
            unpack8(rl.keep(wv[k], k), b);
#pragma unroll
            for (int e = 0; e < 8; ++e) p = __builtin_fmaf(a[e], b[e], p);
        }
        return wave_sum(p);
    }
}

template <int NCH>
struct RowPair {
    u32x4 g[NCH], u[NCH];
};

template <int NCH, bool TAIL = false>
__device__ __forceinline__ void load_rows(RowPair<NCH> &r, const bf16_t *__restrict__ Wg,
                                          const bf16_t *__restrict__ Wu, size_t row, int lane,
                                          const RowLanes<NCH, TAIL> &rl)
{
    const u32x4 *pg = reinterpret_cast<const u32x4 *>(Wg + rl.row(row));
    const u32x4 *pu = reinterpret_cast<const u32x4 *>(Wu + rl.row(row));
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        r.g[k] = __builtin_nontemporal_load(pg + rl.piece(k, lane));
        r.u[k] = __builtin_nontemporal_load(pu + rl.piece(k, lane));
    }
}

}  // namespace halo
