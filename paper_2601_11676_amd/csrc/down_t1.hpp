// What the one-token down projection and the attention block's output projection share.
#pragma once
#include "common.hpp"

namespace halo {

template <int RQ>
struct DownShared {
    int list[256];
    float half[RQ][64];
};

// the eight activations that face a lane's 16-byte piece of a row, as they are stored
template <typename AT> struct ActPiece;
template <> struct ActPiece<bf16_t> {
    u32x4 v;
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const u32x4 *>(p); }
    __device__ __forceinline__ void dot(const u32x4 &w, float &acc0, float &acc1) const
    {
        acc0 = dot2_bf16(w.x, v.x, acc0);
        acc1 = dot2_bf16(w.y, v.y, acc1);
        acc0 = dot2_bf16(w.z, v.z, acc0);
        acc1 = dot2_bf16(w.w, v.w, acc1);
    }
};
template <> struct ActPiece<float> {
    float4 a, b;
    __device__ __forceinline__ void load(const float *p)
    {
        a = *reinterpret_cast<const float4 *>(p);
        b = *reinterpret_cast<const float4 *>(p + 4);
    }
    __device__ __forceinline__ void dot(const u32x4 &w, float &acc0, float &acc1) const
    {
        acc0 = __builtin_fmaf(bf16_lo(w.x), a.x, acc0);
        acc1 = __builtin_fmaf(bf16_hi(w.x), a.y, acc1);
        acc0 = __builtin_fmaf(bf16_lo(w.y), a.z, acc0);
        acc1 = __builtin_fmaf(bf16_hi(w.y), a.w, acc1);
        acc0 = __builtin_fmaf(bf16_lo(w.z), b.x, acc0);
        acc1 = __builtin_fmaf(bf16_hi(w.z), b.y, acc1);
        acc0 = __builtin_fmaf(bf16_lo(w.w), b.z, acc0);
        acc1 = __builtin_fmaf(bf16_hi(w.w), b.w, acc1);
    }
};

}  // namespace halo
