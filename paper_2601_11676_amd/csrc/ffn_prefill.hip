// Group-sparse SwiGLU FFN for many tokens (prefill) on the matrix cores, bf16.
//
// With hundreds of tokens the block is a dense contraction per neuron group, but only over
// the tokens that keep the group (paper Sec. II-A: groups are independent until the merge;
// Sec. III-B.3: each token has its own surviving set).  Kernels:
//
//   group_tokens : for every group, the ascending list of tokens that keep it, and for
//                  every (group, token) the row of the group's activations that the token reads: its
//                  position in that list, or the row of zeros kept behind the list's last row.
//   gate_up_pf_ring : one workgroup = 64 neurons of one group (64 gate + 64 up rows) x up to 256
//                  of the group's tokens (x rows gathered by the token list); the operands
//                  travel straight from memory into rings of K stages in LDS.
//                  act[g][slot][m] = SiLU(gate) * up in bf16.
//   gate_up_pf_big : the same with whole groups of rows and 256 tokens, where there are tiles enough (bf16).
//   down_pf_ring : one workgroup = 128 outputs x 256 tokens over a range of groups, same rings;
//                  a token that does not keep a group reads the group's zero row, so it
//                  contributes exactly nothing.  With several ranges the fp32 partial sums are
//                  added by reduce_partials in fixed order; every element has one writer.
//   down_pf      : the earlier output-stationary form (128 tokens x 64 outputs per workgroup,
//                  walking all groups), kept for more tokens than the row table's 16 bits hold.
//
// Both ring kernels take bf16 weights or 4-bit codes (Q4); the codes become the bf16 values s * (c - 8), rounded
// to nearest even, on their way into LDS, between the matrix instructions of the stage before.  Up to 64 tokens over codes have
// kernels of their own (prefill_codes.hpp).
//
// v_mfma_f32_16x16x32_bf16 operand layout as in ffn_mfma.hip: A lane l = row l%16, elements
// 8*(l/16)..+7; B lane l = column l%16, same elements; D lane l = column l%16, rows 4*(l/16)..+3.

#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "prefill_codes.hpp"

namespace halo {

// ---------------------------------------------------------------------------
// token lists: grid = G workgroups of 256 threads
// ---------------------------------------------------------------------------
// rows != nullptr: row table [G][row_pitch] (row_pitch = T rounded up to 8; the entries past T are 0).
// slot != nullptr instead (two or three tokens, or more than 32767): [T][G] positions in the list, -1 = not kept.
// A workgroup asks for the mask bytes of RUNS runs of 256 tokens at once and places them behind one barrier; where that is all of them
// the list's length comes from the same bytes.  (A run at a time, three barriers and a trip to memory
// each, after a pass over the bytes for the length: 1000 tokens, 224 groups 7.0 us, now 5.2; a pass of 5000 tokens, d 1024, 24 groups
// 120.9 / 115.2, of 2000 tokens of the 7B shape 376.9 / 372.6, of 300 tokens, d 2048 71.8 / 71.0,
// of 17 and 256 tokens, d 256, 6 groups 22.4 / 21.9 and 26.5 / 25.8.)
constexpr int kGroupRuns = 8;

template <int RUNS>
__global__ __launch_bounds__(256) void group_tokens_kernel(const uint8_t *__restrict__ mask, int T, int G,
                                                           int32_t *__restrict__ tok_list,
                                                           int32_t *__restrict__ tok_cnt, int16_t *__restrict__ rows,
                                                           int32_t *__restrict__ slot, bf16_t *__restrict__ act)
{
    __shared__ __attribute__((aligned(16))) int s_cnt[RUNS][4];
    __shared__ int s_wave[4];
    const int g = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int pitch = prefill_row_pitch(T);
    // the list's length is the zero row of the tokens that do not keep the group, so it is needed first
    int cnt = 0, base = 0;
    if (RUNS == kGroupRuns && T > RUNS * 256) {
        int mine = 0;
        for (int t = tid; t < T; t += 256) mine += mask[(size_t)t * G + g] != 0 ? 1 : 0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mine += __shfl_xor(mine, off, kWave);
        if (lane == 0) s_wave[wave] = mine;
        __syncthreads();
        cnt = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    }
    for (int t0 = 0; t0 < pitch; t0 += RUNS * 256) {
        uint8_t kept[RUNS];
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {
            const int t = t0 + i * 256 + tid;
            kept[i] = mask[(size_t)min(t, T - 1) * G + g];
        }
        unsigned long long b[RUNS];
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {
            b[i] = __ballot(t0 + i * 256 + tid < T && kept[i] != 0);
            if (lane == 0) s_cnt[i][wave] = __popcll(b[i]);
        }
        __syncthreads();
        int before[RUNS];
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {
            const int c0 = s_cnt[i][0], c1 = s_cnt[i][1], c2 = s_cnt[i][2], c3 = s_cnt[i][3];
            before[i] = base + (wave > 0 ? c0 : 0) + (wave > 1 ? c1 : 0) + (wave > 2 ? c2 : 0);
            base += c0 + c1 + c2 + c3;
        }
        if (T <= RUNS * 256) cnt = base;
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {
            const int t = t0 + i * 256 + tid;
            const bool keep = (b[i] >> lane & 1) != 0;
            const int pos = before[i] + __popcll(b[i] & ((1ull << lane) - 1ull));
            if (keep) tok_list[(size_t)g * T + pos] = t;
            if (rows) {
                if (t < pitch) rows[(size_t)g * pitch + t] = (int16_t)(t < T ? (keep ? pos : cnt) : 0);
            } else if (t < T) {
                slot[(size_t)t * G + g] = keep ? pos : -1;
            }
        }
        if (t0 + RUNS * 256 < pitch) __syncthreads();           // before s_cnt is written again
    }
    if (tid == 0) tok_cnt[g] = cnt;
    // the row after the group's last activation row is kept zero (group size 128): the down
    // projection points the tokens that do not keep the group at it
    if (cnt < T && tid < 64) reinterpret_cast<uint32_t *>(act + ((size_t)g * T + cnt) * 128)[tid] = 0u;
}

static void launch_group_tokens(const uint8_t *mask, int T, int G, int32_t *tok_list, int32_t *tok_cnt, int16_t *rows, int32_t *slot, bf16_t *act,
                                hipStream_t s)
{
    if (T <= 256)
        group_tokens_kernel<1><<<dim3(G), dim3(256), 0, s>>>(mask, T, G, tok_list, tok_cnt, rows, slot, act);
    else if (T <= 512)
        group_tokens_kernel<2><<<dim3(G), dim3(256), 0, s>>>(mask, T, G, tok_list, tok_cnt, rows, slot, act);
    else
        group_tokens_kernel<kGroupRuns><<<dim3(G), dim3(256), 0, s>>>(mask, T, G, tok_list, tok_cnt, rows, slot, act);
}

// ---------------------------------------------------------------------------
// gate/up through rings in LDS filled by direct global -> LDS loads
// grid: 8 * ceil(items / 8) workgroups of 512 threads, one per compute unit
// ---------------------------------------------------------------------------
// Workgroup tile: 128 weight rows (64 gate + 64 up neurons of one group) x NTOK (256 or 128) of the group's
// tokens; K advances 64 elements per stage.  In LDS a stage is 128 weight rows and NTOK gathered x
// rows of 128 bytes.  One load instruction moves 1 KiB = 8 rows x 128 bytes, lane l landing at byte
// 16 l of the block; to keep the operand reads free of bank conflicts the 16-byte piece p of tile row
// r is parked at position p ^ (r & 7) of its row, which the loading lane arranges by fetching piece
// (l & 7) ^ (l >> 3).  Nothing passes through registers on the way.
//
// The x ring (and with bf16 weights the weight ring) holds three stages, so a stage is requested three steps
// before the matrix instructions use it.  Each of the eight waves fetches an eighth of every stage.
//
// 4-bit weights: the codes of two stages -- one quantisation block of 128 elements, 64 bytes of each of 128
// rows -- and the rows' scales go to a ring of three such blocks in LDS the same way.  Step s turns the codes
// of stage s + 2 into bf16 (a thread 16 elements of a row) and parks them in one of two weight buffers.  A wave
// converts the rows it has fetched itself, so nothing but its own wait stands between the two.
//
// For the matrix work the eight waves are two halves of the stage's K range (elements
// 0..31 / 32..63) times four parts of the tile (256 tokens: four quarters of them; 128 or 64 tokens: two halves of the rows
// times two halves of the tokens), so a wave owns a 128 x 64 (64 x 64, 64 x 32) partial tile; the two K halves are
// added through LDS once at the end.
//
// Two waves share a SIMD, and that is what the kernels' speed comes from.  A wave issues one instruction at a time, and
// everything it issues beside its matrix instructions -- loads, LDS reads, address arithmetic, the conversion of codes --
// delays the next of them; with a wave of its own per SIMD (a 128 x 128 tile in 256 accumulation registers) all of that
// was added to the matrix time.  512 tokens of the 7B shape: gate/up 70 -> 64 us, down 51 -> 44 (bf16); 128 tokens of the
// 13B shape over codes: 63 -> 59 and 33.6 -> 32.  (32 x 32 x 16 instructions, which read half the operand registers per
// multiply-add, were no faster: 67 and 49 us.)
//
// What bounds them now, from builds with one thing taken out at a time (7B shape, 512 tokens): a launch, the tile
// lookup, the first stage and the exchange at the end 12 us; a stage 0.53 us of matrix work at what the chip sustains (46
// and 38 us with nothing else), 0.57 with the LDS reads, the barrier and loads that move nothing, 0.80 in gate/up when
// the 48 KiB come from memory, which is what a compute unit can have in flight; a stage of codes 0.8 us, the conversion
// being added to the matrix work.
constexpr int kRingStages = 3;
constexpr int kRawBlocks = 3;                                    // blocks of codes in LDS
constexpr int kRawBytes = 128 * 64 + 128 * 4;                    // codes, then a word with the scale of every row

template <bool Q4, int NTOK>
struct Ring {
    static constexpr int kMT = NTOK == 256 ? 8 : 4, kTT = NTOK == 64 ? 2 : 4;    // 16-row and 16-token tiles of a wave
    static constexpr int kXL = NTOK / 64;                        // x loads of a wave per stage
    static constexpr int kX = NTOK * 128;                        // bytes of a stage of token rows
    static constexpr int kW = 128 * 128;                         // bytes of a stage of weight rows
    static constexpr int kWBufs = Q4 ? 2 : kRingStages;
    static constexpr int kWBase = kRingStages * kX, kRawBase = kWBase + kWBufs * kW;
    static constexpr int kBytes = kRawBase + (Q4 ? kRawBlocks * kRawBytes : 0);
    static constexpr int kLoads = kXL + (Q4 ? 0 : 2);            // loads of a wave per stage
    static_assert(kBytes >= kRingWaves * kMT * (kTT / 2) * 1024, "the final exchange fits");
};

// the part of the workgroup's tile a wave multiplies
template <int MT>
struct WavePart {
    int ks, rh, tq;                                              // K half, half of the rows (MT == 4), part of the tokens
    __device__ __forceinline__ WavePart(int wave) : ks(wave & 1), rh(MT == 8 ? 0 : (wave >> 1) & 1), tq(MT == 8 ? wave >> 1 : wave >> 2) {}
    // 16-row tile of the workgroup that is the wave's tile m: gate rows first, then the up rows that face them
    __device__ __forceinline__ int row_tile(int m) const { return MT == 8 ? m : (m < 2 ? 2 * rh + m : 4 + 2 * rh + (m - 2)); }
};

// acc += a * b with the accumulator pinned to the accumulation registers and updated in place.
// (Left to itself the compiler gives the tiles of these kernels rotating destination registers and
// moves a few hundred registers between the two files per step to make that work.)  A statement the
// compiler cannot look into also gets none of its matrix-pipeline wait states, which is safe here:
// a wave goes through all of its tiles before it touches one again, 32 in the 256-token rings, 16 and 8 in the 128- and
// 64-token rings, 8 N in gate_up_pf_big (N = 1: seven matrix instructions lie between; ring_multiply asserts the 8).  A
// 16x16x32 bf16 instruction occupies the pipeline for 8 passes and they issue in order, so one instruction
// in between is already more than the few cycles a result takes after its last pass.  The first
// ordinary read of the accumulators comes after an explicit pause of 2 x 16 idle
// cycles, more than the 18 cycles the last instruction can still be in flight.
__device__ __forceinline__ void mfma16_inplace(f32x4_t &acc, const u32x4 &a, const u32x4 &b)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// Zeros in the accumulators.  (They are carried by the loop over the stages, so the writes stand in front of it, far from
// the first matrix instruction; in front of a peeled first step the compiler puts them right before the statements
// that read them, and it cannot know that those need a distance.)
template <int MT, int TT>
__device__ __forceinline__ void clear_accumulators(f32x4_t (&acc)[MT][TT])
{
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < TT; ++n) acc[m][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// The 4-bit side of a ring: this thread's row of the tile is 16 wave + lane / 4, and it converts elements
// 16 (lane & 3) .. + 15 of every stage: eight pairs, each in three parts of one or two vector instructions.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
struct Q4Stage {
    uint2 codes;
    u32x4 out;
    float scale, off, lo, hi;
    uint32_t word, pair, mask, base;
    // (the and-or's two constants in registers that the compiler cannot see through, as in q4_consts)
    __device__ __forceinline__ Q4Stage() { asm volatile("v_mov_b32 %0, 0x00F000F0\n\tv_mov_b32 %1, 0x54005400" : "=v"(mask), "=v"(base)); }
    // block slot `raw` (LDS bytes), second or first stage of the block
    __device__ __forceinline__ void read(const unsigned char *raw, int wave, int lane, bool second)
    {
        const int row = 16 * wave + (lane >> 2);
        codes = *reinterpret_cast<const uint2 *>(raw + row * 64 + (second ? 32 : 0) + (lane & 3) * 8);
        word = *reinterpret_cast<const uint32_t *>(raw + 128 * 64 + row * 4);
    }
    // upper: the scale is the upper half of the word
    __device__ __forceinline__ void set_scale(bool upper)
    {
        scale = __uint_as_float(upper ? word & 0xffff0000u : word << 16);
        off = -72.0f * scale;
    }
    // part 0, 1, 2 of pair p (0..7).  A code in bits 4..7 of the half float 64 is 64 + c, and the mixed multiply-add takes half floats as
    // they lie in the pair: s * (64 + c) - 72 s = s * (c - 8), exact in float (scales below 2^121.8); one instruction rounds both.  4.75
    // instructions per pair; as 128 + c in bf16, which has to be widened first, 6.75: a pass of 128 tokens at the 13B shape 105.8 -> 102.9
    // us, of 600 at 70B 763 -> 731, 97 tokens of d 3200, 75 groups 85.1 -> 81.2.  (As c 2^-24, a shift per pair less, it is no faster, and
    // 2^24 s overflows from 2^104 on.)
    __device__ __forceinline__ void part(int p, int which)
    {
        const int i = p & 3;
        if (which == 0) {
            const uint32_t w = p >> 2 ? codes.y : codes.x;
            const uint32_t at = i == 0 ? w << 4 : i == 1 ? w : w >> (4 * i - 4);
            asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(pair) : "v"(at), "v"(mask), "v"(base));
        } else if (which == 1) {
            const f16x2_t h = __builtin_bit_cast(f16x2_t, pair);
            lo = __builtin_fmaf((float)h[0], scale, off);
            hi = __builtin_fmaf((float)h[1], scale, off);
        } else {
            const f32x2_t v = {lo, hi};
            out[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
        }
    }
    // the eight elements of word j are complete
    __device__ __forceinline__ void park(unsigned char *wbuf, int wave, int lane, int j) const
    {
        const int row = 16 * wave + (lane >> 2), piece = (lane & 3) * 2 + j;
        *reinterpret_cast<u32x4 *>(wbuf + row * 128 + ((piece ^ (row & 7)) * 16)) = out;
    }
    __device__ __forceinline__ void all(unsigned char *wbuf, int wave, int lane, bool upper)
    {
        set_scale(upper);
#pragma unroll
        for (int p = 0; p < 8; ++p) {
#pragma unroll
            for (int which = 0; which < 3; ++which) part(p, which);
            if ((p & 3) == 3) park(wbuf, wave, lane, p >> 2);
        }
    }
    // what of the conversion goes in front of matrix instruction n of N (the first ones belong to the reads)
    template <int N>
    __device__ __forceinline__ void beside(int n, unsigned char *wbuf, int wave, int lane, bool upper)
    {
        constexpr int kFirst = N / 8 + 1, kLast = N - 1;
        if (n == kFirst - 1) set_scale(upper);
#pragma unroll
        for (int u = 0; u < 24; ++u) {                           // unit u = part u % 3 of pair u / 3
            if (n == kFirst + u * (kLast - kFirst) / 24) {
                part(u / 3, u % 3);
                if (u % 12 == 11) park(wbuf, wave, lane, u / 12);
            }
        }
    }
};

// The matrix work of a step, in the order it is issued: in front of matrix instruction n goes what beside(n) puts
// there, and as soon as a row tile's fragment has met the token tiles its registers are asked for the next stage's
// (refill(m)): it is used again a whole step later.
template <int MT, int TT, typename Beside, typename Refill>
__device__ __forceinline__ void ring_multiply(f32x4_t (&acc)[MT][TT], const u32x4 (&a)[MT], const u32x4 (&b)[TT], Beside beside,
                                              Refill refill)
{
    static_assert(MT * TT >= 8, "the distance that mfma16_inplace relies on");
#pragma unroll
    for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            beside(m * TT + tt);
            mfma16_inplace(acc[m][tt], a[m], b[tt]);
            __builtin_amdgcn_sched_barrier(0);
        }
        refill(m);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The two K halves of a tile meet in LDS: a wave keeps one half of its token tiles and hands the other to its partner
// (wave ^ 1).  put(m, j, v): element j of the kept half.
template <int KS_HALF, int MT, int TT, typename Put>
__device__ __forceinline__ void exchange_halves(f32x4_t (&acc)[MT][TT], unsigned char *ring, int wave, int lane, Put put)
{
    constexpr int H = TT / 2, own = H * KS_HALF, other = H - own;
    unsigned char *mine = ring + wave * (MT * H * 1024) + lane * 16;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < H; ++j) *reinterpret_cast<f32x4_t *>(mine + (m * H + j) * 1024) = acc[m][other + j];
    __syncthreads();
    const unsigned char *theirs = ring + (wave ^ 1) * (MT * H * 1024) + lane * 16;
#pragma unroll
    for (int j = 0; j < H; ++j)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m][own + j] += *reinterpret_cast<const f32x4_t *>(theirs + (m * H + j) * 1024);
    put(std::integral_constant<int, own>{});
}

// Wg, Wu: bf16 rows [ffn][d], or (Q4) code words [ffn][d/8] with scales Sg, Su [ffn][d/128]
template <bool Q4, int NTOK>
__global__ __launch_bounds__(kRingWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gate_up_pf_ring(
    const bf16_t *__restrict__ x, int T, int d, int G, const void *__restrict__ Wg, const void *__restrict__ Wu,
    const bf16_t *__restrict__ Sg, const bf16_t *__restrict__ Su, const int32_t *__restrict__ tok_list,
    const int32_t *__restrict__ tok_cnt, bf16_t *__restrict__ act)
{
    using R = Ring<Q4, NTOK>;
    constexpr int MT = R::kMT, TT = R::kTT, EV = Q4 ? 2 : 0;     // EV: loads of a wave per block of codes
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    constexpr int gs = 128;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WavePart<MT> part(wave);
    const int i16 = lane & 15, q = lane >> 4;
    // Workgroups are dealt to the eight dies round-robin by their index.  The work items (tile, half
    // of the group's neurons) are numbered so that a die gets a consecutive run of them: the two
    // halves of a tile share their x rows, the tiles of a group share its weight rows, and all
    // workgroups of a die walk K from the same starting stage, so those rows are found in the die's
    // own L2.  Numbering only the tiles that exist also spreads the work evenly over the dies (with
    // a (group, chunk) grid the empty chunks left some dies with more workgroups than compute units).
    auto tiles_of = [](int n) { return (n + NTOK - 1) / NTOK; };
    const int n_items = 2 * count_tiles(tok_cnt, G, lane, tiles_of);
    const int per_die = (n_items + 7) >> 3;
    const int die = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int item = __builtin_amdgcn_readfirstlane(die * per_die + slot);
    if (slot >= per_die || item >= n_items) return;              // uniform for the workgroup
    const int nt = item & 1;
    const int2 tile = find_tile(tok_cnt, G, item >> 1, lane, tiles_of);
    const int g = __builtin_amdgcn_readfirstlane(tile.x);
    const int cnt = __builtin_amdgcn_readfirstlane(tok_cnt[g]);
    const int c0 = __builtin_amdgcn_readfirstlane(tile.y) * NTOK;
    const int32_t *list = tok_list + (size_t)g * T;

    // The dies start at different K stages (rows are a power of two apart: with everybody at the same
    // K offset all requests of a moment would go to the same few memory channels).
    const int ns = d / 64, nd = ns / 2;                          // stages (even, >= 2), blocks of two
    const int block0 = (die * nd) >> 3;
    // loading role: the stage's blocks of 8 rows are dealt round-robin, wave w takes the x blocks w + 8 j, and (bf16)
    // the gate rows 8 w .. + 7 and the up rows 8 w .. + 7
    const int br = lane >> 3;
    const int piece = (lane & 7) ^ br;
    const uint32_t off_w = (uint32_t)((wave * 8 + br) * d + piece * 8) * 2u;
    uint32_t off_x[R::kXL];                                      // byte offset of the lane's piece of block j
#pragma unroll
    for (int j = 0; j < R::kXL; ++j) {
        const int sl = c0 + (wave + 8 * j) * 8 + br;
        off_x[j] = sl < cnt ? (uint32_t)(list[sl] * d + piece * 8) * 2u : kNoRow;
    }
    const uint32_t ring0 = (uint32_t)(size_t)ring;
    const uint32_t xdst0 = ring0 + wave * 1024, wdst0 = ring0 + R::kWBase + wave * 1024;
    const size_t row0 = (size_t)g * gs + nt * 64;                // first gate (or up) row of the tile
    const srd_t srd_g = make_srd((const bf16_t *)Wg + (Q4 ? 0 : row0 * d), true);
    const srd_t srd_u = make_srd((const bf16_t *)Wu + (Q4 ? 0 : row0 * d), true);
    const srd_t srd_x = make_srd(x, true);
    auto if_exists = [](srd_t v, bool yes) {
        v.z = (uint32_t)__builtin_amdgcn_readfirstlane(yes ? v.z : 0u);
        return v;
    };
    // load j (of kLoads) of stage s of the walk, into ring buffer b
    auto byte_of = [&](int s) { return (uint32_t)(2 * block0 + s >= ns ? 2 * block0 + s - ns : 2 * block0 + s) * 128u; };
    auto load = [&](int j, int s, int b) {
        const bool yes = s < ns;
        const uint32_t at = byte_of(yes ? s : 0);
        if (j < R::kXL)
            load_to_lds16(if_exists(srd_x, yes), off_x[j], at, xdst0 + b * R::kX + j * 8192);
        else
            load_to_lds16<true>(if_exists(j == R::kXL ? srd_g : srd_u, yes), off_w, at, wdst0 + b * R::kW + (j - R::kXL) * 8192);
    };
    // codes: this wave's 16 rows are gate rows (waves 0..3) or up rows; one load covers 16 rows x 64 bytes
    const size_t q_row0 = row0 + (wave & 3) * 16;
    const int nb = d / kQ4Block;
    const srd_t srd_c = make_srd((const unsigned char *)(wave < 4 ? Wg : Wu) + (Q4 ? q_row0 * (d / 2) : 0), true);
    const srd_t srd_s = make_srd((wave < 4 ? Sg : Su) + (Q4 ? q_row0 * nb : 0), true);
    const uint32_t off_c = (uint32_t)((lane >> 2) * (d / 2) + (lane & 3) * 16);
    auto block_of = [&](int e) { return block0 + e >= nd ? block0 + e - nd : block0 + e; };
    auto request_codes = [&](int e, bool yes) {                  // block e of the walk
        const int b = block_of(yes ? e : 0);
        const uint32_t dst = ring0 + R::kRawBase + (e % kRawBlocks) * kRawBytes;
        load_to_lds16<true>(if_exists(srd_c, yes), off_c, b * 64, dst + wave * 1024);
        // the aligned pair of scales that holds the row's
        load_to_lds_lanes<4>(0xffffull, if_exists(srd_s, yes), (uint32_t)((((lane & 15) * nb + b) & ~1) * 2), 0,
                             dst + 128 * 64 + wave * 64);
    };
    auto scale_upper = [&](int e) { return (((lane >> 2) * nb + block_of(e)) & 1) != 0; };
    auto raw_of = [&](int e) -> const unsigned char * { return ring + R::kRawBase + (e % kRawBlocks) * kRawBytes; };
    // operand reads: tile row (or token row) i16 of a tile, piece (4 ks + q) at its swizzled position
    const int loff = i16 * 128 + (((4 * part.ks + q) ^ (i16 & 7)) * 16);
    f32x4_t acc[MT][TT];
    clear_accumulators(acc);

    // Stage s lives in ring buffer s % 3 (converted weights: s % 2).  At the top of step s the fragments of stage s are
    // in registers.  The barrier of step s says: everybody's part of stage s+1 has landed and everybody
    // has finished reading stage s, whose buffer is then handed to stage s+3.  Whatever else a step does -- the loads of
    // stage s+3, the LDS reads of stage s+1's fragments, the conversion of stage s+2 -- is dealt out between its matrix
    // instructions: a burst of any of it holds them back for as long as the burst takes to issue.
    // (Waves whose part of the token tile is empty run the matrix work all the same, on rows of zeros: nothing they
    // compute is stored.)
    Q4Stage qs;
    if (Q4) {
#pragma unroll
        for (int e = 0; e < kRawBlocks; ++e) request_codes(e, e < nd);
    }
#pragma unroll
    for (int i = 0; i < kRingStages; ++i)
#pragma unroll
        for (int j = 0; j < R::kLoads; ++j) load(j, i, i);
    wait_loads<2 * R::kLoads>();                                 // the codes (they went first) and stage 0
    if (Q4) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            qs.read(raw_of(0), wave, lane, k == 1);
            qs.all(ring + R::kWBase + k * R::kW, wave, lane, scale_upper(0));
        }
        request_codes(0, false);                                 // nothing (block 0 is used up), but the waits below count on it
    }
    __syncthreads();
    u32x4 fa[MT], fb0[TT], fb1[TT];
    auto read_a = [&](int m, int wbuf) {
        fa[m] = *reinterpret_cast<const u32x4 *>(ring + R::kWBase + wbuf * R::kW + loff + part.row_tile(m) * 2048);
    };
    auto read_b = [&](u32x4 (&f)[TT], int n, int xbuf) {
        f[n] = *reinterpret_cast<const u32x4 *>(ring + xbuf * R::kX + part.tq * (TT * 2048) + loff + n * 2048);
    };
#pragma unroll
    for (int m = 0; m < MT; ++m) read_a(m, 0);
#pragma unroll
    for (int n = 0; n < TT; ++n) read_b(fb0, n, 0);
    int buf = 0;                                                 // ring buffer of stage s
    auto step = [&](const u32x4 (&cur)[TT], u32x4 (&next)[TT], int s, bool odd) __attribute__((always_inline)) {
        const int nbuf = buf == kRingStages - 1 ? 0 : buf + 1;
        // stage s+2 may still be on its way, and the block of codes requested last (in the even step s-1 or s-2)
        wait_loads<R::kLoads + EV>();
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        const int e = s / 2 + 1;                                 // block of stage s+2 (past the end: stale codes, unused)
        if (Q4) qs.read(raw_of(e), wave, lane, odd);
        unsigned char *wpark = ring + R::kWBase + (odd ? R::kW : 0);
        const bool upper = Q4 && scale_upper(e < nd ? e : 0);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int N = MT * TT, kEvery = N / (R::kLoads + 1);
        // (in the last step the fragments of a stage that does not exist, unused)
        ring_multiply<MT, TT>(
            acc, fa, cur,
            [&](int n) __attribute__((always_inline)) {
                if (n < TT) read_b(next, n, nbuf);
                if (n % kEvery == kEvery - 1 && n / kEvery < R::kLoads) load(n / kEvery, s + kRingStages, buf);
                if (Q4) qs.beside<N>(n, wpark, wave, lane, upper);
            },
            [&](int m) __attribute__((always_inline)) { read_a(m, Q4 ? (odd ? 0 : 1) : nbuf); });
        if (Q4 && !odd) request_codes(s / 2 + kRawBlocks, s / 2 + kRawBlocks < nd);
        buf = nbuf;
    };
    for (int s = 0; s < ns; s += 2) {
        step(fb0, fb1, s, false);
        step(fb1, fb0, s + 1, true);
    }
    wait_loads<0>();                                             // (of loads that move nothing)
    __syncthreads();                                             // every wave is done with the rings
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");           // the last matrix results are in the registers
    __builtin_amdgcn_sched_barrier(0);                           // (nothing that reads them moves above the pause)

    bf16_t *act_row0 = act + (size_t)g * T * gs + nt * 64;
    const int sl0 = c0 + part.tq * (TT * 16) + i16;
    auto put = [&](auto first) {
        constexpr int own = decltype(first)::value;
#pragma unroll
        for (int j = 0; j < TT / 2; ++j) {
            const int sl = sl0 + (own + j) * 16;
#pragma unroll
            for (int m = 0; m < MT / 2; ++m) {
                const f32x4_t gt = acc[m][own + j], up = acc[m + MT / 2][own + j];
                const uint32_t lo = (uint32_t)f32_to_bf16(silu_mul_fast(gt[0], up[0])) | ((uint32_t)f32_to_bf16(silu_mul_fast(gt[1], up[1])) << 16);
                const uint32_t hi = (uint32_t)f32_to_bf16(silu_mul_fast(gt[2], up[2])) | ((uint32_t)f32_to_bf16(silu_mul_fast(gt[3], up[3])) << 16);
                if (sl < cnt) *reinterpret_cast<uint2 *>(act_row0 + (size_t)sl * 128 + part.row_tile(m) * 16 + 4 * q) = make_uint2(lo, hi);
            }
        }
    };
    if (part.ks == 0)
        exchange_halves<0, MT, TT>(acc, ring, wave, lane, put);
    else
        exchange_halves<1, MT, TT>(acc, ring, wave, lane, put);
}

// codes of up to 64 tokens
template <>
__global__ __launch_bounds__(kRingWaves * 64, 2) void gate_up_pf_ring<true, 64>(
    const bf16_t *__restrict__ x, int T, int d, int G, const void *__restrict__ Wg, const void *__restrict__ Wu,
    const bf16_t *__restrict__ Sg, const bf16_t *__restrict__ Su, const int32_t *__restrict__ tok_list,
    const int32_t *__restrict__ tok_cnt, bf16_t *__restrict__ act)
{
    gate_up_codes(x, T, d, G, (const unsigned char *)Wg, (const unsigned char *)Wu, Sg, Su, tok_list, tok_cnt, act);
}

// ---------------------------------------------------------------------------
// the same over whole tiles of 256 weight rows x 256 tokens (bf16)
// ---------------------------------------------------------------------------
// What a compute unit can have in flight bounds gate_up_pf_ring: it moves 96 KiB into LDS per 256 x 256 x 64 of matrix
// work, this kernel 64.  (us per launch against gate_up_pf_ring, half of the tokens keeping a group: 1000 tokens of the 70B
// shape 495 against 525, of the 13B shape 135 against 168, 1024 tokens of the 7B shape 108 against 125.)  The eight waves are
// two halves of the rows times four shares of the 16-token tiles over the whole K range: no exchange at the end.
// Groups end in a tile of any length (their token counts differ widely), so a wave's tiles are every fourth one and a tile
// of one, two or three quarters runs with as many per wave: 1000 tokens of the 70B shape 523 -> 495.  (Taking all whole
// tiles first and the short ones behind them evened out the last round, but then no two tiles of a group share their
// weight rows in a die's L2: 13B shape 138 -> 192.)  So the weight rows carry the non-temporal hint, as gate_up_pf_ring's do, only where the tile is the
// group's one: with it they are gone when the next tile of the group comes (a pass of 600 tokens of the 70B shape, half kept, 775 us, without
// 719), without it a lone tile's push x out (200 tokens there, half kept 332 us, without 347; 512 tokens, a tenth kept 401 and 419; a pass as it is
// now 722, 333, 395).
// Two stages of 64 KiB fit, so a step is cut in two: half kk of the 64 elements of stage s is multiplied while the
// fragments of the next half are read.  The barrier sits in front of the second half, when everybody has read all of
// stage s: its buffers go to the stages that follow, token rows one step ahead, weight rows (three buffers: they come from
// memory, not from a neighbour's L2 lines) two.
constexpr int kBigStage = 256 * 128;                             // bytes of a stage of weight rows, or of token rows

__global__ __launch_bounds__(kRingWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gate_up_pf_big(
    const bf16_t *__restrict__ x, int T, int d, int G, const bf16_t *__restrict__ Wg, const bf16_t *__restrict__ Wu,
    const int32_t *__restrict__ tok_list, const int32_t *__restrict__ tok_cnt, bf16_t *__restrict__ act)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];      // two stages of token rows, three of weight rows
    constexpr int gs = 128, kWBase = 2 * kBigStage;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rh = wave & 1, tq = wave >> 1;
    const int i16 = lane & 15, q = lane >> 4;
    // one item per token tile; numbered as in gate_up_pf_ring
    auto tiles_of = [](int n) { return (n + 255) / 256; };
    const int n_items = count_tiles(tok_cnt, G, lane, tiles_of);
    const int per_die = (n_items + 7) >> 3;
    const int die = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int item = __builtin_amdgcn_readfirstlane(die * per_die + slot);
    if (slot >= per_die || item >= n_items) return;              // uniform for the workgroup
    const int2 tile = find_tile(tok_cnt, G, item, lane, tiles_of);
    const int g = __builtin_amdgcn_readfirstlane(tile.x);
    const int cnt = __builtin_amdgcn_readfirstlane(tok_cnt[g]);
    const int c0 = __builtin_amdgcn_readfirstlane(tile.y) * 256;
    const int quarters = min((cnt - c0 + 63) / 64, 4);
    const int32_t *list = tok_list + (size_t)g * T;

    const int ns = d / 64, stage0 = (die * ns) >> 3;
    const int br = lane >> 3, piece = (lane & 7) ^ br;
    // a stage's 32 blocks of 8 token rows and 32 of weight rows (gate rows, then up rows): wave w takes blocks w + 8 j
    uint32_t off_x[4], off_w[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int sl = c0 + (wave + 8 * j) * 8 + br;
        off_x[j] = sl < cnt ? (uint32_t)(list[sl] * d + piece * 8) * 2u : kNoRow;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) off_w[j] = (uint32_t)(((wave + 8 * j) * 8 + br) * d + piece * 8) * 2u;
    const uint32_t ring0 = (uint32_t)(size_t)ring + wave * 1024;
    const srd_t srd_g = make_srd(Wg + (size_t)g * gs * d, true), srd_u = make_srd(Wu + (size_t)g * gs * d, true);
    const srd_t srd_x = make_srd(x, true);
    auto if_exists = [](srd_t v, bool yes) {
        v.z = (uint32_t)__builtin_amdgcn_readfirstlane(yes ? v.z : 0u);
        return v;
    };
    auto byte_of = [&](int s) { return (uint32_t)(stage0 + s >= ns ? stage0 + s - ns : stage0 + s) * 128u; };
    auto load_x = [&](int j, int s) {
        const bool yes = s < ns;
        load_to_lds16(if_exists(srd_x, yes), off_x[j], byte_of(yes ? s : 0), ring0 + (s & 1) * kBigStage + j * 8192);
    };
    auto load_w = [&](auto lone, int j, int s, int b) {          // b = s % 3; lone: the only tile of its group
        const bool yes = s < ns;
        load_to_lds16<decltype(lone)::value>(if_exists(j < 2 ? srd_g : srd_u, yes), off_w[j & 1], byte_of(yes ? s : 0),
                                             ring0 + kWBase + b * kBigStage + j * 8192);
    };
    // the wave's row tiles: four of the gate rows and the four of the up rows that face them; its 16-token tiles: tq + 4 n
    auto row_tile = [&](int m) { return m < 4 ? 4 * rh + m : 8 + 4 * rh + (m - 4); };

    auto first_stages = [&](auto lone) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int j = 0; j < 4; ++j) load_x(j, s);
#pragma unroll
            for (int j = 0; j < 4; ++j) load_w(lone, j, s, s);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) load_w(lone, j, 2, 2);
        wait_loads<12>();                                        // stage 0
        __syncthreads();
    };
    auto tile_of = [&](auto quarters_c, auto lone) __attribute__((always_inline)) {
        constexpr int N = decltype(quarters_c)::value;           // 16-token tiles of a wave
        int loff0 = i16 * 128 + ((q ^ (i16 & 7)) * 16);          // piece 4 kk + q
        asm volatile("" : "+v"(loff0));                          // (worked out here: kept from the kernel's head it is spilled)
        const int loff1 = loff0 ^ 64;
        f32x4_t acc[8][N];
        clear_accumulators(acc);
        u32x4 fa[8], f0[N], f1[N];
        int wb = 0;                                              // weight buffer of stage s
        auto wbuf = [&](int ahead) { return wb + ahead >= 3 ? wb + ahead - 3 : wb + ahead; };
        auto read_a = [&](int m, int b, int off) __attribute__((always_inline)) {
            fa[m] = *reinterpret_cast<const u32x4 *>(ring + kWBase + b * kBigStage + off + row_tile(m) * 2048);
        };
        auto read_b = [&](u32x4 (&f)[N], int n, int s, int off) __attribute__((always_inline)) {
            f[n] = *reinterpret_cast<const u32x4 *>(ring + (s & 1) * kBigStage + off + (tq + 4 * n) * 2048);
        };
#pragma unroll
        for (int m = 0; m < 8; ++m) read_a(m, 0, loff0);
#pragma unroll
        for (int n = 0; n < N; ++n) read_b(f0, n, 0, loff0);
        for (int s = 0; s < ns; ++s) {
            ring_multiply<8, N>(
                acc, fa, f0, [&](int n) __attribute__((always_inline)) { if (n < N) read_b(f1, n, s, loff1); },
                [&](int m) __attribute__((always_inline)) { read_a(m, wb, loff1); });
            wait_loads<4>();                                     // all but stage s+2's weight rows
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            // (in the last step the fragments of a stage that does not exist, unused)
            ring_multiply<8, N>(
                acc, fa, f1,
                [&](int n) __attribute__((always_inline)) {
                    if (n < N) read_b(f0, n, s + 1, loff0);
                    constexpr int every = N < 3 ? N : 3;
                    const int k = n / every;
                    if (n % every == every - 1 && k < 8) {
                        if (k < 4)
                            load_x(k, s + 2);
                        else
                            load_w(lone, k - 4, s + 3, wb);
                    }
                },
                [&](int m) __attribute__((always_inline)) { read_a(m, wbuf(1), loff0); });
            wb = wbuf(1);
        }
        wait_loads<0>();                                         // (of loads that move nothing)
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");       // the last matrix results are in the registers
        __builtin_amdgcn_sched_barrier(0);                       // (nothing that reads them moves above the pause)

        bf16_t *act_row0 = act + (size_t)g * T * gs;
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int sl = c0 + (tq + 4 * n) * 16 + i16;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const f32x4_t gt = acc[m][n], up = acc[m + 4][n];
                const uint32_t lo = (uint32_t)f32_to_bf16(silu_mul_fast(gt[0], up[0])) | ((uint32_t)f32_to_bf16(silu_mul_fast(gt[1], up[1])) << 16);
                const uint32_t hi = (uint32_t)f32_to_bf16(silu_mul_fast(gt[2], up[2])) | ((uint32_t)f32_to_bf16(silu_mul_fast(gt[3], up[3])) << 16);
                if (sl < cnt) *reinterpret_cast<uint2 *>(act_row0 + (size_t)sl * 128 + (4 * rh + m) * 16 + 4 * q) = make_uint2(lo, hi);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto run_tile = [&](auto lone) __attribute__((always_inline)) {
        first_stages(lone);
        if (quarters == 4)
            tile_of(std::integral_constant<int, 4>{}, lone);
        else if (quarters == 3)
            tile_of(std::integral_constant<int, 3>{}, lone);
        else if (quarters == 2)
            tile_of(std::integral_constant<int, 2>{}, lone);
        else
            tile_of(std::integral_constant<int, 1>{}, lone);
    };
    if (cnt <= 256)                                              // uniform
        run_tile(std::true_type{});
    else
        run_tile(std::false_type{});
}

// ---------------------------------------------------------------------------
// down: grid (d/64, ceil(T/128)), 256 threads; group size 128
// ---------------------------------------------------------------------------
// A workgroup owns 128 tokens x 64 outputs and walks the groups.  The group's 64 x 128 tile of
// Wd is 16 KiB of consecutive bytes: it is fetched once per workgroup with coalesced loads,
// staged through LDS and shared by the four waves (each wave loading its own operand pieces
// cost four times the L1 traffic and ran at 8 % of the matrix peak).  The activation rows are
// private to a wave (its 32 tokens), gathered by slot straight into registers; a token that
// does not keep the group gets a zero fragment and so contributes exactly nothing.
constexpr int kWdRow = 128 + 8;     // padded LDS row of the Wd tile, elements

struct ActFrags {
    u32x4 b[4][2];                  // [k step][token tile]
};

__global__ __launch_bounds__(256) void down_pf(
    int T, int d, int G, const bf16_t *__restrict__ Wd, const int32_t *__restrict__ slot,
    const bf16_t *__restrict__ act, bf16_t *__restrict__ y)
{
    constexpr int gs = 128;
    __shared__ __attribute__((aligned(16))) bf16_t sWd[2][64 * kWdRow];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i16 = lane & 15, q = lane >> 4;
    const int j0 = blockIdx.x * 64;
    const int t0 = blockIdx.y * 128 + wave * 32;       // may be >= T for the last workgroup's upper waves:
                                                        // those waves still stage Wd and meet the barriers
    const int32_t *sl0, *sl1;
    {
        const int ta = t0 + i16, tb = t0 + 16 + i16;
        sl0 = slot + (size_t)(ta < T ? ta : T - 1) * G;          // duplicates of a valid token, never stored
        sl1 = slot + (size_t)(tb < T ? tb : T - 1) * G;
    }
    f32x4_t acc[4][2];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) acc[mt][tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const size_t gstride = (size_t)d * gs;
    // staging role: the tile is 1024 pieces of 16 bytes; this thread moves pieces tid + 256 n
    const bf16_t *wsrc = Wd + (size_t)j0 * gs + tid * 8;
    int wdst[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int p = tid + 256 * n;
        wdst[n] = (p >> 4) * kWdRow + (p & 15) * 8;
    }
    auto load_w = [&](u32x4 (&r)[4], int g) {
#pragma unroll
        for (int n = 0; n < 4; ++n)
            r[n] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(wsrc + g * gstride + n * 2048));
    };
    auto store_w = [&](bf16_t *buf, const u32x4 (&r)[4]) {
#pragma unroll
        for (int n = 0; n < 4; ++n) *reinterpret_cast<u32x4 *>(buf + wdst[n]) = r[n];
    };
    auto load_act = [&](ActFrags &f, int g, int s0, int s1) {
        const bf16_t *pb0 = act + ((size_t)g * T + (s0 < 0 ? 0 : s0)) * gs + q * 8;
        const bf16_t *pb1 = act + ((size_t)g * T + (s1 < 0 ? 0 : s1)) * gs + q * 8;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const u32x4 v0 = *reinterpret_cast<const u32x4 *>(pb0 + ks * 32);
            const u32x4 v1 = *reinterpret_cast<const u32x4 *>(pb1 + ks * 32);
            f.b[ks][0] = s0 < 0 ? u32x4{0u, 0u, 0u, 0u} : v0;
            f.b[ks][1] = s1 < 0 ? u32x4{0u, 0u, 0u, 0u} : v1;
        }
    };
    auto multiply = [&](const bf16_t *buf, const ActFrags &f) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            u32x4 a[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                a[mt] = *reinterpret_cast<const u32x4 *>(buf + (mt * 16 + i16) * kWdRow + ks * 32 + q * 8);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                acc[mt][0] = mfma16p(a[mt], f.b[ks][0], acc[mt][0]);
                acc[mt][1] = mfma16p(a[mt], f.b[ks][1], acc[mt][1]);
            }
        }
    };
    // groups in pairs.  A group's Wd tile travels global -> registers -> LDS two groups ahead of its
    // use, its activation fragments one group ahead, the slots (which the fragment addresses depend
    // on) one group further.  Loads past the last group repeat the last group (harmless).
    // Top of an even step g: sWd[0] holds W(g); rw1 = W(g+1) and F0 = act(g) are in flight;
    // (s0, s1) are the slots of group g+1.
    auto cl = [&](int g) { return g < G ? g : G - 1; };
    u32x4 rw0[4], rw1[4];
    ActFrags F0, F1;
    int s0 = sl0[0], s1 = sl1[0];
    load_w(rw0, 0);
    load_act(F0, 0, s0, s1);
    load_w(rw1, cl(1));
    s0 = sl0[cl(1)]; s1 = sl1[cl(1)];
    int n0 = sl0[cl(2)], n1 = sl1[cl(2)];       // slots of group g+2
    store_w(sWd[0], rw0);
    __syncthreads();
    int g = 0;
    for (; g + 1 < G; g += 2) {
        load_act(F1, cl(g + 1), s0, s1);
        load_w(rw0, cl(g + 2));
        s0 = n0; s1 = n1;                       // slots of group g+2
        n0 = sl0[cl(g + 3)]; n1 = sl1[cl(g + 3)];
        multiply(sWd[0], F0);
        store_w(sWd[1], rw1);
        __syncthreads();
        load_act(F0, cl(g + 2), s0, s1);
        load_w(rw1, cl(g + 3));
        s0 = n0; s1 = n1;                       // slots of group g+3
        n0 = sl0[cl(g + 4)]; n1 = sl1[cl(g + 4)];
        multiply(sWd[1], F1);
        store_w(sWd[0], rw0);
        __syncthreads();
    }
    if (g < G) multiply(sWd[0], F0);            // an odd number of groups: the last one
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
        const int t = t0 + tt * 16 + i16;
        if (t < T) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                uint32_t lo = (uint32_t)f32_to_bf16(acc[mt][tt][0]) | ((uint32_t)f32_to_bf16(acc[mt][tt][1]) << 16);
                uint32_t hi = (uint32_t)f32_to_bf16(acc[mt][tt][2]) | ((uint32_t)f32_to_bf16(acc[mt][tt][3]) << 16);
                *reinterpret_cast<uint2 *>(y + (size_t)t * d + j0 + mt * 16 + 4 * q) = make_uint2(lo, hi);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// down projection through the same kind of rings, groups split over workgroups
// grid: 8 * ceil(items / 8) workgroups of 512 threads
// ---------------------------------------------------------------------------
// Workgroup tile: 128 outputs x NTOK tokens, over a contiguous range of the groups (the K
// dimension): with 128 x 256 tiles alone a 512-token call would occupy 64 compute units, so the
// groups are cut into `splits` ranges and every range goes to its own workgroup, which leaves its
// fp32 partial sums in partial[split][t][j]; reduce_partials adds the ranges in fixed order.  With a
// single range the workgroup writes y itself.
//
// A stage is half a group (64 of its 128 neurons): 128 rows of Wd (the group's 128 x 128 tile is 32
// KiB of consecutive bytes, a stage takes alternate halves of its 256-byte rows; as codes it is 8 KiB, one block of
// the ring of codes) and the token rows of act, found through the row table: the table's entries of a
// group for the tile's tokens travel like everything else, four groups ahead, each wave's own to itself
// (a table of all groups built in LDS up front cost 4 us and held 32 groups: a block of 224 groups needed seven ranges and
// their partial sums, 1000 tokens 509 + 43 us; one range takes 370).
// A token that does not keep the group is pointed at the group's row of zeros (written by group_tokens), so
// it contributes exactly nothing.  Everything else is as in gate_up_pf_ring.
constexpr int kDownMaxSplits = 8;

template <bool Q4, int NTOK>
__host__ __device__ constexpr int down_ring_bytes() { return Ring<Q4, NTOK>::kBytes + kTabGroups * kTabBytes; }
static_assert(down_ring_bytes<true, 256>() <= 160 * 1024 && down_ring_bytes<false, 256>() <= 160 * 1024, "fits a compute unit");

// Number of group ranges, the cheapest by a plain account in us: rounds of one workgroup per compute unit, each 10 and 1.3
// per group, and with several ranges the reduction's launch, write and read.
// 1000 tokens of the 13B shape in three ranges 130 + 12 us against 166 + 9 in two, 600 tokens of the 70B shape in four
// 309 + 15 against 318 in one.
static int down_splits(int T, int d, int G)
{
    const long long tiles = (long long)(d / 128) * ((T + 255) / 256);
    int best = 1;
    float least = 0.f;
    for (int n = 1; n <= kDownMaxSplits && n <= G; ++n) {
        const float rounds = (float)((tiles * n + 255) / 256), reduce = n > 1 ? 5.f + 1.2e-6f * n * T * d : 0.f;
        const float us = rounds * (10.f + 1.3f * ((G + n - 1) / n)) + reduce;
        if (n == 1 || us < least) best = n, least = us;
    }
    return best;
}

// the row table holds 16 bits, and x is addressed with 32-bit byte offsets
int prefill_ring_tokens(int d) { return (int)std::min<long long>(32767, ((1ll << 31) - 1) / ((long long)d * 2)); }

// the ranges that this shape is cut into where the scratch has room for their sums, 0 = shape not covered by
// the ring kernels.  With the tiles fixed it falls as T grows (the reduction's part of the account is n T d), never rises.
int prefill_down_splits(int T, int d, int G) { return d % 128 != 0 || T > 32767 ? 0 : down_splits(T, d, G); }

// The ranges whose sums every workspace has room for.  They give a workspace its size, and so decide which calls the fixed
// scratch array takes: the line is an agreed one (ranges of at most 32 groups, none for shapes that would need
// more than kDownMaxSplits to fill the chip) and does not follow the kernels.
int prefill_down_splits_reserved(int T, int d, int G)
{
    if (d % 128 != 0 || T > 32767) return 0;
    const int tiles = (d / 128) * ((T + 255) / 256), need = (G + 31) / 32;
    int splits = (256 + tiles / 2) / tiles;
    splits = splits < need ? need : splits;
    splits = splits < 1 ? 1 : splits;
    splits = splits > G ? G : splits;
    return splits > kDownMaxSplits || (G + splits - 1) / splits > 32 ? 0 : splits;
}

// the wanted ranges, or as many as the call's scratch holds (a small workspace of a narrow layer)
static int splits_in_room(int splits, int T, int d, const DecodeScratch &ws)
{
    const size_t room = ws.partial_elems / ((size_t)T * d);
    return room >= (size_t)splits ? splits : room < 1 ? 1 : (int)room;
}

// Wd: bf16 [G][d][128], or (Q4) code words [G][d][16] with scales Sd [G][d]; rows: the row table.  SCALED: codes of up to 64 tokens
// (down_codes), with the sums of the activations
template <bool Q4, int NTOK, bool SCALED>
__global__ __launch_bounds__(kRingWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void down_pf_ring(
    int T, int d, int G, int splits, const void *__restrict__ Wd, const bf16_t *__restrict__ Sd,
    const int16_t *__restrict__ rows, const bf16_t *__restrict__ act, float *__restrict__ partial, bf16_t *__restrict__ y)
{
    using R = Ring<Q4, NTOK>;
    constexpr int MT = R::kMT, TT = R::kTT, EV = Q4 ? 3 : 1;     // EV: loads of a wave per group besides the stages'
    extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WavePart<MT> part(wave);
    const int i16 = lane & 15, q = lane >> 4;
    DownItem it;
    if (!down_item<Q4, NTOK>(T, d, G, splits, it)) return;
    const int t0 = it.t0, j0 = it.j0, g_lo = it.g_lo, split = it.split;
    const int ng = it.g_hi - g_lo;                               // >= 1
    const int ns = 2 * ng;

    // loading role: the stage's blocks of 8 rows are dealt round-robin, wave w takes the act blocks w + 8 j and (bf16)
    // the Wd rows 8 w .. + 7 and 64 + 8 w .. + 7
    const int br = lane >> 3;
    const int piece = (lane & 7) ^ br;
    const uint32_t ring0 = (uint32_t)(size_t)ring;
    const uint32_t off_w = (uint32_t)((wave * 8 + br) * 128 + piece * 8) * 2u;
    uint32_t off_a[R::kXL];
    // what travels once per group: the wave's entries of the row table, four groups ahead (a piece of eight entries for
    // each of its blocks; pieces past the table's end repeat its last one), and with 4-bit weights its 16 rows of
    // codes and their scales, three groups ahead
    const int pitch = prefill_row_pitch(T);
    const uint32_t off_t = (uint32_t)min(t0 + (wave + 8 * (lane & (R::kXL - 1))) * 8, pitch - 8) * 2u;
    auto request_table = [&](int gi, bool yes) {
        const size_t gg = (size_t)(g_lo + (yes ? gi : 0));
        load_to_lds_lanes<16>((1ull << R::kXL) - 1ull, make_srd(rows + gg * pitch, yes), off_t, 0,
                              ring0 + R::kBytes + (gi % kTabGroups) * kTabBytes + wave * (R::kXL * 16));
    };
    auto request_codes = [&](int gi, bool yes) {
        const size_t gg = (size_t)(g_lo + (yes ? gi : 0)) * d + j0 + wave * 16;
        const uint32_t dst = ring0 + R::kRawBase + (gi % kRawBlocks) * kRawBytes;
        load_to_lds16(make_srd((const unsigned char *)Wd + gg * 64, yes), lane * 16u, 0, dst + wave * 1024);
        load_to_lds_lanes<4>(0xffffull, make_srd(Sd + gg, yes), ((lane & 15) >> 1) * 4u, 0, dst + 128 * 64 + wave * 64);
    };
    auto raw_of = [&](int gi) -> const unsigned char * { return ring + R::kRawBase + (gi % kRawBlocks) * kRawBytes; };
    const bool upper = (lane >> 2) & 1;                          // row 16 wave + lane / 4 of an even first row
    auto entry = [&](int gi, int j) -> int {
        return reinterpret_cast<const int16_t *>(ring + R::kBytes + (gi % kTabGroups) * kTabBytes + wave * (R::kXL * 16))[j * 8 + br];
    };
    auto offset_of = [&](int row) { return (uint32_t)(row * 128 + piece * 8) * 2u; };
    const uint32_t xdst0 = ring0 + wave * 1024, wdst0 = ring0 + R::kWBase + wave * 1024;
    // load j (of kLoads) of stage s, half of group s / 2 of the range, into ring buffer b
    srd_t srd_a, srd_w;
    auto group_srds = [&](int gi) {
        const bool yes = gi < ng;
        const size_t gg = (size_t)(g_lo + (yes ? gi : 0));
        srd_a = make_srd(act + gg * T * 128, yes);
        if (!Q4) srd_w = make_srd((const bf16_t *)Wd + (gg * d + j0) * 128, yes);
    };
    auto load = [&](int j, int s, int b) {
        const uint32_t at = (s & 1) * 128u;
        if (j < R::kXL)
            load_to_lds16(srd_a, off_a[j], at, xdst0 + b * R::kX + j * 8192);
        else
            load_to_lds16(srd_w, off_w, at + (j - R::kXL) * 16384u, wdst0 + b * R::kW + (j - R::kXL) * 8192);
    };
    const int loff = i16 * 128 + (((4 * part.ks + q) ^ (i16 & 7)) * 16);
    f32x4_t acc[MT][TT];
    clear_accumulators(acc);

#pragma unroll
    for (int gi = 0; gi < kTabGroups; ++gi) request_table(gi, gi < ng);
    if (Q4) {
#pragma unroll
        for (int gi = 0; gi < kRawBlocks; ++gi) request_codes(gi, gi < ng);
    }
    wait_loads<0>();                                             // the table of the first groups (each wave its own entries)
#pragma unroll
    for (int i = 0; i < kRingStages; ++i) {
        if (i != 1) {                                            // stages 0 and 1 are group 0's, 2 and 3 group 1's
#pragma unroll
            for (int j = 0; j < R::kXL; ++j) off_a[j] = offset_of(entry(i / 2 < ng ? i / 2 : 0, j));
            group_srds(i / 2);
        }
#pragma unroll
        for (int j = 0; j < R::kLoads; ++j) load(j, i, i);
    }
    Q4Stage qs;
    if (Q4) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            qs.read(raw_of(0), wave, lane, k == 1);
            qs.all(ring + R::kWBase + k * R::kW, wave, lane, upper);
        }
    }
    wait_loads<2 * R::kLoads>();
    request_table(0, false);                                     // nothing (group 0 is used up), but the waits below count on it
    if (Q4) request_codes(0, false);
    __syncthreads();
    u32x4 fa[MT], fb0[TT], fb1[TT];
    auto read_a = [&](int m, int wbuf) {
        fa[m] = *reinterpret_cast<const u32x4 *>(ring + R::kWBase + wbuf * R::kW + loff + part.row_tile(m) * 2048);
    };
    auto read_b = [&](u32x4 (&f)[TT], int n, int xbuf) {
        f[n] = *reinterpret_cast<const u32x4 *>(ring + xbuf * R::kX + part.tq * (TT * 2048) + loff + n * 2048);
    };
#pragma unroll
    for (int m = 0; m < MT; ++m) read_a(m, 0);
#pragma unroll
    for (int n = 0; n < TT; ++n) read_b(fb0, n, 0);
    int buf = 0;                                                 // ring buffer of stage s
    int row[R::kXL];
    auto step = [&](const u32x4 (&cur)[TT], u32x4 (&next)[TT], int s, bool odd) __attribute__((always_inline)) {
        const int nbuf = buf == kRingStages - 1 ? 0 : buf + 1;
        // stage s+2 may still be on its way, and the loads of the group requested last (in the even step s-1 or s-2)
        wait_loads<R::kLoads + EV>();
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        if (Q4) qs.read(raw_of(s / 2 + 1), wave, lane, odd);     // stage s+2 (past the end: stale codes, unused)
        unsigned char *wpark = ring + R::kWBase + (odd ? R::kW : 0);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int N = MT * TT, kEvery = N / (R::kLoads + 1);
        // (in the last step the fragments of a stage that does not exist, unused)
        ring_multiply<MT, TT>(
            acc, fa, cur,
            [&](int n) __attribute__((always_inline)) {
                if (n < TT) read_b(next, n, nbuf);
                if (n % kEvery == kEvery - 1 && n / kEvery < R::kLoads) load(n / kEvery, s + kRingStages, buf);
                // an even step requests the second half of a group; behind its loads, the next group's rows
                // (s + 4 is their first stage; past the end whatever the table holds, unused)
                if (!odd && n >= 4 && n < 4 + R::kXL) row[n - 4] = entry(s / 2 + 2, n - 4);
                if (!odd && n >= N - R::kXL) off_a[n - (N - R::kXL)] = offset_of(row[n - (N - R::kXL)]);
                if (Q4) qs.beside<N>(n, wpark, wave, lane, upper);
            },
            [&](int m) __attribute__((always_inline)) { read_a(m, Q4 ? (odd ? 0 : 1) : nbuf); });
        if (!odd) {
            request_table(s / 2 + kTabGroups, s / 2 + kTabGroups < ng);
            if (Q4) request_codes(s / 2 + kRawBlocks, s / 2 + kRawBlocks < ng);
            group_srds(s / 2 + 2);
        }
        buf = nbuf;
    };
    for (int s = 0; s < ns; s += 2) {
        step(fb0, fb1, s, false);
        step(fb1, fb0, s + 1, true);
    }
    wait_loads<0>();                                             // (of loads that move nothing)
    __syncthreads();                                             // every wave is done with the rings
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");           // the last matrix results are in the registers
    __builtin_amdgcn_sched_barrier(0);                           // (nothing that reads them moves above the pause)

    float *out = partial ? partial + (size_t)split * T * d : nullptr;
    auto put = [&](auto first) {
        constexpr int own = decltype(first)::value;
#pragma unroll
        for (int j = 0; j < TT / 2; ++j) {
            const int t = t0 + part.tq * (TT * 16) + (own + j) * 16 + i16;
            if (t < T) {
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const f32x4_t v = acc[m][own + j];
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
        exchange_halves<0, MT, TT>(acc, ring, wave, lane, put);
    else
        exchange_halves<1, MT, TT>(acc, ring, wave, lane, put);
}

template <>
__global__ __launch_bounds__(kRingWaves * 64, 2) void down_pf_ring<true, 64, true>(
    int T, int d, int G, int splits, const void *__restrict__ Wd, const bf16_t *__restrict__ Sd,
    const int16_t *__restrict__ rows, const bf16_t *__restrict__ act, float *__restrict__ partial, bf16_t *__restrict__ y)
{
    down_codes(T, d, G, splits, (const unsigned char *)Wd, Sd, rows, act, partial, y);
}

// y = sum of the ranges' partial sums, added in the order of the ranges; n = T * d, a multiple of 8
__global__ __launch_bounds__(256) void reduce_partials(const float *__restrict__ partial, int splits, size_t n,
                                                       bf16_t *__restrict__ y)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    float v[8];
    load8(partial + i, v);
    for (int k = 1; k < splits; ++k) {
        float w[8];
        load8(partial + (size_t)k * n + i, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += w[e];
    }
    store8(y + i, v);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
bool prefill_path_supported(int T, int d, int gs)
{
    // (the ring kernel addresses x rows with 32-bit byte offsets)
    return T > 1 && d % 128 == 0 && gs == 128 && (size_t)T * d * sizeof(bf16_t) < (1ull << 31);
}

// Up to 64 tokens over codes (rows of at least 256: pairs of blocks): prefill_codes.hpp, the scale applied in float as for fewer tokens.  Above that
// the values are rounded to bf16 and the results are those of the bf16 kernels on the expanded weights, bit for bit, which callers may count on (the
// same kernel in a 128-token tile, codes as 128 + c, would run 100 tokens of d 3200, 75 groups and 128 of 13B in 70 us instead of 85 and 98 instead
// of 109).
static bool codes_path(int T, int d) { return T <= 64 && d >= 256; }

template <bool Q4, int NTOK>
static hipError_t launch_gate_up_ring(const bf16_t *x, int T, int d, int G, const void *Wg, const void *Wu, const bf16_t *Sg,
                                      const bf16_t *Su, const DecodeScratch &ws, bf16_t *act, hipStream_t s)
{
    constexpr int bytes = Q4 && NTOK == 64 ? kCodesBytes : Ring<Q4, NTOK>::kBytes;
    const hipError_t lds_ok = allow_lds<gate_up_pf_ring<Q4, NTOK>>(bytes);
    if (lds_ok != hipSuccess) return lds_ok;
    const int items_max = 2 * G * ((T + NTOK - 1) / NTOK);                  // every group kept by every token
    launch_timed_lds("gate_up_pf_ring", gate_up_pf_ring<Q4, NTOK>, dim3((items_max + 7) / 8 * 8), dim3(kRingWaves * 64),
                     bytes, s, x, T, d, G, Wg, Wu, Sg, Su, (const int32_t *)ws.tok_list, (const int32_t *)ws.tok_cnt, act);
    return hipSuccess;
}

static void launch_reduce(const float *partial, int splits, int T, int d, bf16_t *y, hipStream_t s)
{
    const size_t n = (size_t)T * d;
    reduce_partials<<<dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, s>>>(partial, splits, n, y);
}

template <bool Q4, int NTOK, bool SCALED = false>
static hipError_t launch_down_ring(int T, int d, int G, int splits, const void *Wd, const bf16_t *Sd, const DecodeScratch &ws,
                                   const bf16_t *act, bf16_t *y, hipStream_t s)
{
    constexpr int bytes = SCALED ? kCodesBytes + kTabGroups * kTabBytes / 2 : down_ring_bytes<Q4, NTOK>();
    const hipError_t lds_ok = allow_lds<down_pf_ring<Q4, NTOK, SCALED>>(bytes);
    if (lds_ok != hipSuccess) return lds_ok;
    const int items = (d / 128) * ((T + NTOK - 1) / NTOK) * splits;
    down_pf_ring<Q4, NTOK, SCALED><<<dim3((items + 7) / 8 * 8), dim3(kRingWaves * 64), bytes, s>>>(
        T, d, G, splits, Wd, Sd, reinterpret_cast<const int16_t *>(ws.slot), act, splits > 1 ? ws.partial : (float *)nullptr, y);
    if (splits > 1) launch_reduce(ws.partial, splits, T, d, y, s);
    return hipSuccess;
}

// Whole tiles of 256 x 256 in gate/up when half of the tokens keeping a group (the lists are not known here; each
// ends in half a tile on average) gives more than 150 of them: gate_up_pf_ring's half rows then take a second round.
// Whole FFN in us, ring against whole tiles, half of the tokens keeping a group: below the line 7B 500 tokens 115 against 138,
// 13B 400 148 against 175; above it 7B 700 196 against 163, 13B 600 260 against 221, 70B 256 385 against 294.  With other
// shares the line lies elsewhere: at 0.3 these three run in 157 (ring 133), 197 (171) and 275 (286), at 0.7 the two below
// the line in 170 (whole tiles 143) and 234 (194).
static bool gate_up_big_tiles(int T, int G) { return (long long)G * (T + 256) > 512 * 150; }

static hipError_t launch_gate_up_big(const bf16_t *x, int T, int d, int G, const bf16_t *Wg, const bf16_t *Wu,
                                     const DecodeScratch &ws, bf16_t *act, hipStream_t s)
{
    const hipError_t lds_ok = allow_lds<gate_up_pf_big>(5 * kBigStage);
    if (lds_ok != hipSuccess) return lds_ok;
    launch_timed_lds("gate_up_pf_big", gate_up_pf_big, dim3((G * ((T + 255) / 256) + 7) / 8 * 8),
                     dim3(kRingWaves * 64), 5 * kBigStage, s, x, T, d, G, Wg, Wu, (const int32_t *)ws.tok_list, (const int32_t *)ws.tok_cnt, act);
    return hipSuccess;
}

// Half tiles of tokens where they hold (gate/up: nearly) all of a group's tokens: half the matrix work of a stage, and
// the next tile of a group's weights is found in the die's L2.  7B shape, bf16,
// 128 tokens 44.7 us in gate/up and 25.7 us in down against 50.8 and 28.2 with whole tiles; 256 tokens 49.8 against 60.1
// in gate/up, but 32.9 against 31.8 in down; 400 tokens 85 against 63 and 56 against 45.
// In the down projection also where whole tiles times ranges would fill less than half of the chip: 200 tokens of d 2048, one
// range, 41.7 us against 63.4; 200 tokens of d 1024 10.0 against 13.6.
//
// Quarter tiles where they hold all of a group's tokens, whatever the mask: up to 64 tokens, in the down projection (and over codes, see
// codes_path).  Not in gate/up: it waits for memory, and a stage of fewer bytes keeps fewer in flight.  Pass in us, half tiles against quarter
// tiles in gate/up alone and in both projections: 17 tokens, 7B 78.5 / 78.4 / 76.4, 70B 267 / 273 / 270.
// In the down projection also where half tiles times ranges would fill less than half of the chip.  Half against quarter, bf16
// and codes: 256 tokens of d 2048 77.4 / 68.4 and 96.1 / 89.2, 200 of d 2560 101.5 / 94.2 and 119.6 / 111.3, 100 of d 3072
// 79.6 / 76.7 and 83.3 / 79.6, 600 of d 768 54.0 / 49.3 and 62.9 / 59.2; where they fill more than that, 100 tokens of 13B
// 122 against 157.  So it is down to the shortest rows and the fewest groups.  The FFN on its own, bf16 and codes: d 256, 2 groups, 65 tokens
// 16.3 / 15.1 and 19.4 / 18.1, 256 tokens 17.6 / 16.0 and 20.6 / 18.9; d 640, 40 groups, 128 tokens 28.3 / 25.9 and 32.4 / 30.5; d 1024,
// 6 groups, 256 tokens 28.7 / 26.4 and 32.8 / 30.6; over d 256 .. 1024, 2 .. 40 groups, 65 .. 400 tokens 1.00 to 1.12 times as fast, never
// slower.  Rows of one output tile stay as they are.
static bool down_quarter_tiles(int T, int d, int splits)
{
    return d >= 256 && (T <= 64 || (long long)(d / 128) * ((T + 127) / 128) * splits < 128);
}

template <bool Q4>
static hipError_t launch_rings(const bf16_t *x, int T, int d, int G, const void *Wg, const void *Wu, const void *Wd,
                               const bf16_t *Sg, const bf16_t *Su, const bf16_t *Sd, const DecodeScratch &ws, bf16_t *act,
                               bf16_t *y, hipStream_t s)
{
    hipError_t e;
    if (!Q4 && gate_up_big_tiles(T, G))
        e = launch_gate_up_big(x, T, d, G, (const bf16_t *)Wg, (const bf16_t *)Wu, ws, act, s);
    else if (Q4 && codes_path(T, d))
        e = launch_gate_up_ring<Q4, Q4 ? 64 : 128>(x, T, d, G, Wg, Wu, Sg, Su, ws, act, s);   // (no bf16 form is built)
    else if (T <= 256)
        e = launch_gate_up_ring<Q4, 128>(x, T, d, G, Wg, Wu, Sg, Su, ws, act, s);
    else
        e = launch_gate_up_ring<Q4, 256>(x, T, d, G, Wg, Wu, Sg, Su, ws, act, s);
    if (e != hipSuccess) return e;
    const int splits = splits_in_room(down_splits(T, d, G), T, d, ws);
    if (Q4 && codes_path(T, d))
        e = launch_down_ring<Q4, 64, Q4>(T, d, G, splits, Wd, Sd, ws, act, y, s);
    else if (down_quarter_tiles(T, d, splits))
        e = launch_down_ring<Q4, 64>(T, d, G, splits, Wd, Sd, ws, act, y, s);
    else if (T <= 128 || (d / 128) * ((T + 255) / 256) * splits < 128)
        e = launch_down_ring<Q4, 128>(T, d, G, splits, Wd, Sd, ws, act, y, s);
    else
        e = launch_down_ring<Q4, 256>(T, d, G, splits, Wd, Sd, ws, act, y, s);
    return e == hipSuccess ? hipGetLastError() : e;
}

// the row table takes the place of the slots: [G][prefill_row_pitch(T)] of 2 bytes in a buffer of [T][G] of 4
static bool row_table_fits(int T) { return T <= 32767 && 2 * prefill_row_pitch(T) <= 4 * T; }

hipError_t launch_ffn_prefill(const bf16_t *x, int T, int d, int G, int gs, const bf16_t *Wg,
                              const bf16_t *Wu, const bf16_t *Wd, const uint8_t *mask, bf16_t *y,
                              const DecodeScratch &ws, hipStream_t s)
{
    bf16_t *act = reinterpret_cast<bf16_t *>(ws.act);
    const bool ring = prefill_down_splits(T, d, G) > 0 && row_table_fits(T);
    launch_group_tokens(mask, T, G, ws.tok_list, ws.tok_cnt, ring ? reinterpret_cast<int16_t *>(ws.slot) : nullptr, ws.slot, act, s);
    if (ring) return launch_rings<false>(x, T, d, G, Wg, Wu, Wd, nullptr, nullptr, nullptr, ws, act, y, s);
    const hipError_t e = launch_gate_up_ring<false, 256>(x, T, d, G, Wg, Wu, nullptr, nullptr, ws, act, s);
    if (e != hipSuccess) return e;
    down_pf<<<dim3(d / 64, (T + 127) / 128), dim3(256), 0, s>>>(T, d, G, Wd, ws.slot, act, y);
    return hipGetLastError();
}

// The same over 4-bit weights: the codes are expanded on their way into LDS, or in registers (codes_path).
bool prefill_q4_supported(int T, int d, int G, int gs)
{
    return T > 16 && prefill_path_supported(T, d, gs) && prefill_down_splits(T, d, G) > 0 && row_table_fits(T);
}

hipError_t launch_ffn_prefill_q4(const bf16_t *x, int T, int d, int G, const Q4Weights &w, const uint8_t *mask, bf16_t *y,
                                 const DecodeScratch &ws, hipStream_t s)
{
    bf16_t *act = reinterpret_cast<bf16_t *>(ws.act);
    launch_group_tokens(mask, T, G, ws.tok_list, ws.tok_cnt,
                        reinterpret_cast<int16_t *>(ws.slot), ws.slot, act, s);
    return launch_rings<true>(x, T, d, G, w.gate_codes, w.up_codes, w.down_codes, w.gate_scales, w.up_scales, w.down_scales,
                              ws, act, y, s);
}

}  // namespace halo
