// Loads that go straight from memory to LDS.
#pragma once
#include "common.hpp"

namespace halo {

// Direct memory -> LDS loads through a buffer descriptor: lane l's 16 bytes at base + voff + soff land at LDS
// address lds_addr + 16 l; m0 carries the LDS address.  A lane whose voff is kNoRow, and every lane of a
// descriptor of size 0, is out of range: it reads nothing (its place in LDS becomes zeros), but the load still
// counts as one of the wave's outstanding loads.  So rows that do not exist and stages past the end need no branch, no change of the
// active lanes and no other wait: a load is three instructions between two matrix instructions.  (With a branch
// and a masked exec around each load, eight more scalar instructions per load held the matrix instructions back:
// 512 tokens of the 7B
// shape, gate/up 80 -> 70 us, down 61 -> 51, with the loads dealt out between the matrix instructions)
// STREAM: the bytes are used once by this die (weight rows): the load carries the non-temporal hint, so
// that they do not push the rows that are used again (x, act) out of the die's L2.
typedef uint32_t srd_t __attribute__((ext_vector_type(4)));
constexpr uint32_t kNoRow = 0x80000000u, kAnySize = 0x7fffffffu;

__device__ __forceinline__ srd_t make_srd(const void *p, bool exists)
{
    const unsigned long long u = (unsigned long long)p;
    return srd_t{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)u),
                 (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(u >> 32) & 0xffffu),
                 (uint32_t)__builtin_amdgcn_readfirstlane(exists ? kAnySize : 0u), 0x00020000u};
}
template <bool STREAM = false>
__device__ __forceinline__ void load_to_lds16(const srd_t &srd, uint32_t voff, uint32_t soff, uint32_t lds_addr)
{
    if (STREAM)
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds" ::"v"(voff), "s"(srd),
                     "s"(__builtin_amdgcn_readfirstlane(soff)), "s"(__builtin_amdgcn_readfirstlane(lds_addr))
                     : "memory");           // m0 is reserved: the compiler sets it anew before each use of its own
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(srd),
                     "s"(__builtin_amdgcn_readfirstlane(soff)), "s"(__builtin_amdgcn_readfirstlane(lds_addr))
                     : "memory");
}
// the same with the LDS address lds_addr + AT: one scalar instruction
template <int AT, bool STREAM = false>
__device__ __forceinline__ void load_to_lds16_at(const srd_t &srd, uint32_t voff, uint32_t soff, uint32_t lds_addr)
{
    if (STREAM)
        asm volatile("s_add_u32 m0, %3, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds" ::"v"(voff), "s"(srd),
                     "s"(__builtin_amdgcn_readfirstlane(soff)), "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "n"(AT)
                     : "memory", "scc");
    else
        asm volatile("s_add_u32 m0, %3, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(srd),
                     "s"(__builtin_amdgcn_readfirstlane(soff)), "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "n"(AT)
                     : "memory", "scc");
}
// the same as load_to_lds16 for the lanes of `lanes` only: a lane out of range still writes zeros to its place in LDS, a lane that is
// switched off writes nothing.  BYTES: 16 or 4.
template <int BYTES>
__device__ __forceinline__ void load_to_lds_lanes(unsigned long long lanes, const srd_t &srd, uint32_t voff, uint32_t soff,
                                                  uint32_t lds_addr)
{
    unsigned long long saved_exec;
    if (BYTES == 16)
        asm volatile("s_mov_b32 m0, %4\n\ts_mov_b64 %0, exec\n\ts_mov_b64 exec, %5\n\t"
                     "buffer_load_dwordx4 %1, %2, %3 offen lds\n\ts_mov_b64 exec, %0"
                     : "=&s"(saved_exec)
                     : "v"(voff), "s"(srd), "s"(__builtin_amdgcn_readfirstlane(soff)),
                       "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "s"(lanes)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %4\n\ts_mov_b64 %0, exec\n\ts_mov_b64 exec, %5\n\t"
                     "buffer_load_dword %1, %2, %3 offen lds\n\ts_mov_b64 exec, %0"
                     : "=&s"(saved_exec)
                     : "v"(voff), "s"(srd), "s"(__builtin_amdgcn_readfirstlane(soff)),
                       "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "s"(lanes)
                     : "memory");
}

// wait until at most N of the wave's loads are outstanding
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace halo
