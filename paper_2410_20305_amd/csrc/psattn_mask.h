// How kernels read the block mask: from device memory, or, where it is small, from their own arguments.
//
// A step of a few hundred tokens is bound by launches and by chains of dependent loads.  Bringing its mask onto the device took a
// kernel of its own: 2.6 us, which is PCIe latency, 2.6 us of host time to launch it and 1.5 us to record the event that guards
// its buffers.  Masks of samples of up to 1 024 tokens travel with the arguments of each kernel, packed into 136 bytes because
// every 64 bytes of arguments take time to arrive.  Measured, in device memory / in the arguments: fp32 step of 168 tokens on one head
// 25.5 / 21.3 us, bf16 step of 221 tokens on 32 / 8 heads 46.6 / 39.4.  A mask that is kept over many calls costs the kernels the
// same from either place: forward and backward together 18.0 / 18.0 on those 168 tokens, 33.2 / 33.2 on 180, 38.4 / 38.5 on 221,
// 47.4 / 47.4 on 500, 66.1 / 65.7 on 900.
//
// The arguments are read by scalar loads through the argument segment's address, so that indexing them does not make the compiler
// copy them to scratch memory: kernels take AttnArgs as their first argument.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "psattn_internal.h"

namespace psattn {

typedef const __attribute__((address_space(4))) uint32_t ArgWord;
__device__ __forceinline__ ArgWord* small_mask(size_t field) {
    return (ArgWord*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(AttnArgs, meta.small) + field);
}
// A word of the arguments in a scalar register.  (Left to itself the compiler turns a choice between words into vector loads at a
// chosen address, each as far away as memory.)
__device__ __forceinline__ uint32_t arg_word(ArgWord* p) {
    uint32_t x = *p;
    asm volatile("" : "+s"(x));
    return x;
}

// Loads the arguments that a kernel starts with in one go instead of one by one as they are needed.
__device__ __forceinline__ void fetch_args(const AttnArgs& a) {
    ArgWord* const row = small_mask(offsetof(SmallMask, row));
    asm volatile("" ::"s"(a.Hq), "s"(a.Hkv), "s"(a.Q), "s"(a.K), "s"(a.V), "s"(a.dO), "s"(a.O), "s"(a.LSE), "s"(a.rope), "s"(a.meta.T), "s"(a.meta.in_args),
                 "s"(a.meta.list.tok), "s"(a.meta.list.launch[0]), "s"(a.meta.list.launch[1]), "s"(row[-(2 * kSmallRows)]), "s"(row[0]));
}

__device__ __forceinline__ Tok4 unpack_run(uint32_t lo, uint32_t hi) {
    const uint64_t x = (static_cast<uint64_t>(hi) << 32) | lo;
    const auto field = [&](int i) { return static_cast<int>(static_cast<uint32_t>(x >> (kSmallField * i)) & kSmallNone); };
    return Tok4{field(1) == static_cast<int>(kSmallNone) ? kPadStart : field(1), field(2), field(3), field(4)};
}

// Descriptor of token t (padding from T on) in three steps, so that what a kernel issues in between hides the wait: the load from
// device memory is started, a mask in the arguments is searched, and the one that holds is chosen where the load has come back.
// Each has registers of its own.  (Where both ways wrote the same ones, the compiler let the way through the arguments wait for the
// load that it does not make, and with it for all copies issued since, which it does not count: the search then stood
// behind the first tile's arrival.  Forward / backward of 180 tokens, 32 / 8 heads, on a kept mask: 7.9 / 7.8 us, 25.9 / 25.5.)
typedef int TokenLoad __attribute__((ext_vector_type(4)));
__device__ __forceinline__ TokenLoad token_begin(const DeviceMeta& m, int t) {
    TokenLoad x = {kPadStart, 0, 0, 0};
    if (!m.in_args && t < m.T) x = *reinterpret_cast<const TokenLoad*>(m.list.tok + t);
    return x;
}
__device__ __forceinline__ Tok4 token_search(const DeviceMeta& m, int t) {
    Tok4 x = {kPadStart, 0, 0, 0};
    if (m.in_args) {  // a token's run is the last that starts at or before it
        typedef uint32_t Runs __attribute__((ext_vector_type(2 * kSmallRuns)));
        typedef Runs RunWords __attribute__((aligned(4)));
        Runs run = *(const __attribute__((address_space(4))) RunWords*)small_mask(offsetof(SmallMask, run));
        asm volatile("" : "+s"(run));
        uint32_t lo = run[0], hi = run[1];
#pragma unroll
        for (int i = 1; i < kSmallRuns; ++i) {
            const bool past = t >= static_cast<int>(run[2 * i] & kSmallNone);
            lo = past ? run[2 * i] : lo;
            hi = past ? run[2 * i + 1] : hi;
        }
        if (t < m.T) x = unpack_run(lo, hi);
    }
    return x;
}
__device__ __forceinline__ Tok4 token_choose(const DeviceMeta& m, TokenLoad loaded, const Tok4& found) {
    asm volatile("" : "+v"(loaded));  // waited for here and not earlier
    return m.in_args ? found : Tok4{loaded.x, loaded.y, loaded.z, loaded.w};
}
// the same at once, 0 <= t < T, from any control flow: one run after the other
__device__ inline Tok4 token(const DeviceMeta& m, int t) {
    if (!m.in_args) return m.list.tok[t];
    ArgWord* const run = small_mask(offsetof(SmallMask, run));
    uint32_t lo = 0, hi = 0;
#pragma nounroll
    for (int i = 0; i < kSmallRuns; ++i) {
        const uint32_t l = arg_word(run + 2 * i), h = arg_word(run + 2 * i + 1);
        if (t >= static_cast<int>(l & kSmallNone)) { lo = l; hi = h; }
    }
    return unpack_run(lo, hi);
}

// What a workgroup starts with: row `i` of the launch order, one scalar load.
template <int GRID>
__device__ __forceinline__ RowLaunch row_launch(const DeviceMeta& m, int i) {
    ArgWord* p = m.in_args ? small_mask(offsetof(SmallMask, tiles)) + GRID * kSmallRows + i
                           : (ArgWord*)reinterpret_cast<uintptr_t>(m.list.launch[GRID]) + 4 * static_cast<ptrdiff_t>(i);
    RowLaunch rl{static_cast<int>(p[0]), static_cast<int>(p[1]), static_cast<int>(p[2]), static_cast<int>(p[3])};
    if (m.in_args) {  // `begin` keeps the row's word of tiles
        const uint32_t tiles = static_cast<uint32_t>(rl.row), listed = tiles & 0xffffu;
        const int first = listed == 0 ? 0 : GRID == kGridQ ? __builtin_ctz(listed) : 31 - __builtin_clz(listed);
        rl.row = static_cast<int>(arg_word(small_mask(offsetof(SmallMask, row)) + GRID) >> (4 * i) & 15u);
        rl.begin = static_cast<int>(tiles);
        rl.count = __builtin_popcount(listed);
        rl.first_entry = first << 2 | (tiles >> (16 + first) & 1u ? PSATTN_TILE_FULL : PSATTN_TILE_PARTIAL);
    }
    return rl;
}

// The list of a row in the arguments, from its word of tiles: entry l to lane l, l < n, read backwards if `step` is -1.  Lane i looks
// at tile i, which is as many entries into the list as listed tiles lie below it, and sends it there.
__device__ __forceinline__ int small_entries(uint32_t tiles, int step, int n) {
    const int i = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    const bool listed = i < kSmallTiles && (tiles >> (i & 15) & 1u);
    const int at = __builtin_amdgcn_mbcnt_lo(tiles & 0xffffu, 0), e = i << 2 | (tiles >> (16 + (i & 15)) & 1u ? PSATTN_TILE_FULL : PSATTN_TILE_PARTIAL);
    return __builtin_amdgcn_ds_permute((listed ? step > 0 ? at : n - 1 - at : 63) << 2, e);
}

// entry `k` of a row's list, the same in all lanes
template <int GRID>
__device__ __forceinline__ int tile_entry(const DeviceMeta& m, const RowLaunch& rl, int k) {
    if (!m.in_args) return m.list.entry[GRID][rl.begin + k];
    return __builtin_amdgcn_readlane(small_entries(static_cast<uint32_t>(rl.begin), 1, rl.count), k);
}

}  // namespace psattn
