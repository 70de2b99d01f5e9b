// bf16 flash-attention kernels for gfx950 (MI355X), head_dim 128 and 64.
//
// What is computed is ordinary softmax attention on the pairs allowed by the
// prefix-sharing mask (paper Algorithm 1 / Algorithm 3); tiles of the block mask
// without an allowed pair are never visited (Section 3.1).  How it is computed is
// this file's own design:
//
//  * 64-wide wavefronts, v_mfma_f32_32x32x16_bf16.  Every product is arranged so
//    that the quantity the wave owns (its 32 queries in forward / dQ, its 32 keys
//    in dK/dV) is the MFMA *column*: scores come out with one query (or key) per
//    lane, softmax statistics are per-lane scalars, and the probabilities feed the
//    next MFMA as a B operand straight from the accumulator registers (the
//    accumulator's row order is absorbed into the order in which the other
//    operand's rows are fetched).
//  * K/V (or Q/dO) tiles are staged in LDS, rows of 2 d bytes, with the 16-byte chunk
//    index XOR-swizzled by the row so that both row-wise 128-bit reads and the
//    transposing 64-bit reads (ds_read_b64_tr_b16) are bank-conflict free without
//    padding (Rows::put, which writes accumulators, is not).  Tiles are copied global -> LDS asynchronously, one tile ahead, into
//    the buffer the previous tile has just vacated; one barrier per tile.
//  * dK/dV are owned by one workgroup per (k-tile, kv-head), which walks the G
//    query heads of the group and the k-major tile list, so the prompt's keys
//    collect the contributions of prompt, chosen and rejected queries without
//    atomics.  dQ is a separate q-major pass.  Both are deterministic.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "psattn_exact.h"

namespace psattn {
namespace mma {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// LDS tile rows are the head dimension: 256 bytes (d = 128) or 128 bytes (d = 64).
template <int D>
constexpr int kRowBytesOf = 2 * D;
constexpr int kRowBytes = kRowBytesOf<128>;

// compile-time loop: f(std::integral_constant<int, I>) for I in [B, E)
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// x, and nothing that the compiler knows of it: what is computed from it stays where it stands instead of living in
// registers throughout the loop before it
__device__ __forceinline__ int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

union Frag8 {
    bf16x8 v;
    bf16x4 h[2];
    bf16x2 p[4];
    uint4 u;
};

// XOR on the 16-byte chunk index of row `row`.  Sixteen consecutive rows at one logical chunk cover all 64 banks
// (row-wise 128-bit reads), and so do four consecutive rows at four neighbouring chunks (transposing reads).  A
// 128-byte row is half the width of the banks: the row's lowest bit selects the half, the next three make the XOR.
template <int D>
__device__ inline int row_swizzle(int row) {
    if constexpr (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
    else return ((row & 2) << 1) | ((row >> 2) & 3);
}

// byte offset of 16-byte chunk `chunk` of row `row` in a swizzled tile
template <int D>
__device__ inline int tile_off(int row, int chunk) {
    return row * kRowBytesOf<D> + ((chunk ^ row_swizzle<D>(row)) << 4);
}

// Per-lane LDS byte offsets of the two operand fetch patterns, relative to the first
// row of a 32-row block.  Because the swizzle is an XOR on the 16-byte chunk index,
// the offset for step t (row-wise operand) or head-dim block db (transposed operand)
// is one lane constant XOR a compile-time constant:
//   row-wise, step t:        nat ^ (t << 5)     row l % 32, chunk 2 t + l / 32
//   transposed, block db:    tr1 ^ (db << 6)    rows 4 (l / 32) + (l % 16) / 4, first four
//                            tr2 ^ (db << 6)    the same, eight rows further down
// A tile base that is a multiple of 256 bytes may be added to the lane constant first.
// MFMA operands: row-wise, a lane holds 8 consecutive bf16 of one row; transposed, lane l holds column
// col0 + l % 32, stored rows r0 + {0..3} and r0 + 8 + {0..3} with r0 = row0 + 4 * (l / 32), which is the
// row order in which a 32x32 accumulator hands its values to the next MFMA.
struct LaneOffsets {
    int nat, tr1, tr2;
};

template <int D = 128>
__device__ inline LaneOffsets lane_offsets(int l) {
    LaneOffsets o;
    const int c32 = l & 31, g = l >> 5, i16 = l & 15;
    o.nat = tile_off<D>(c32, g);
    const int row = 4 * g + (i16 >> 2);
    const int col = 16 * ((l >> 4) & 1) + 4 * (i16 & 3);
    o.tr1 = tile_off<D>(row, col >> 3) + (col & 7) * 2;
    o.tr2 = tile_off<D>(row + 8, col >> 3) + (col & 7) * 2;
    return o;
}

// row-wise MFMA operand, step t, of the 32-row block at `blk` (blk: multiple of 256 bytes)
template <int T>
__device__ __forceinline__ bf16x8 ld_rows(const char* blk, int nat) {
    return *reinterpret_cast<const bf16x8*>(blk + (nat ^ (T << 5)));
}

// transposed MFMA operand: head-dim block DB, stored rows 16 HALF + {0..15} of the block
template <int DB, int HALF, int D = 128>
__device__ __forceinline__ bf16x8 ld_cols(const char* blk, int tr1, int tr2) {
    Frag8 f;
    f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(blk + (tr1 ^ (DB << 6)) + 16 * HALF * kRowBytesOf<D>));
    f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(blk + (tr2 ^ (DB << 6)) + 16 * HALF * kRowBytesOf<D>));
    return f.v;
}

// Mask arithmetic of PARTIAL tiles.  A lane's 32 score elements of a 64-row tile are
// numbered e = 16 b + i (b = 32-row block, i = accumulator register); element e belongs to
// tile row 32 b + acc_row(i, g), so the elements ordered by e are also ordered by row.
// elems_below(x, g): how many of them lie in rows below x, 0 <= x <= 64.
__device__ inline int elems_below(int x, int g) {
    return 4 * (x >> 3) + min(max((x & 7) - 4 * g, 0), 4);
}

// bit e set <=> element e lies in tile rows [lo, hi) (any integers; clamped to the tile)
__device__ inline uint32_t elem_range_bits(int lo, int hi, int g) {
    const int a = elems_below(min(max(lo, 0), 64), g), b = elems_below(min(max(hi, 0), 64), g);
    return static_cast<uint32_t>(((1ull << b) - 1) & ~((1ull << a) - 1));
}

// x if bit e of `bits` is set, otherwise -inf (two instructions: bit -> word mask, select)
template <int E>
__device__ __forceinline__ float keep_or_neg_inf(float x, uint32_t bits) {
    const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(bits << (31 - E)) >> 31);
    return __uint_as_float((__float_as_uint(x) & m) | (~m & 0xff800000u));
}

__device__ inline f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// values of accumulator registers [8*half, 8*half + 8) as a bf16 B operand
__device__ inline bf16x8 pack8(const f32x16& x, int half) {
    Frag8 f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f32x2 v = {x[8 * half + 2 * j], x[8 * half + 2 * j + 1]};
        f.p[j] = __builtin_convertvector(v, bf16x2);
    }
    return f.v;
}

// The second factor of the second products (probabilities, score gradients) is held in fp32 and the matrix cores take
// bf16.  head_dim 128 rounds it to one bf16 operand.  head_dim 64 loses nothing: three operands, each the upper 16 bits
// (8 of the 24 significant bits) of what the ones before leave, add up to the fp32 value exactly.  Measured on head_dim 64
// against 64-bit sums, 32 / 8 heads, 4 758 tokens: O / dQ / dK / dV off by 1.97 / 2.51 / 2.47 / 2.30e-3 with one operand,
// 1.60 / 1.82 / 1.80 / 1.66e-3 with three, which is the rounding of the outputs (and of O, in delta) and the same as with
// fp32 products throughout; the step takes 176 us instead of 126.
template <int D>
constexpr int kPartsOf = D == 128 ? 1 : 3;

template <int D>
struct Operand {
    bf16x8 part[kPartsOf<D>];
};

// values of accumulator registers [8*half, 8*half + 8)
template <int D>
__device__ __forceinline__ Operand<D> make_operand(const f32x16& x, int half) {
    Operand<D> o;
    if constexpr (kPartsOf<D> == 1) {
        o.part[0] = pack8(x, half);
    } else {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = x[8 * half + j];
        Frag8 f[kPartsOf<D>];
#pragma unroll
        for (int p = 0; p < kPartsOf<D>; ++p) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = __builtin_amdgcn_perm(__float_as_uint(v[2 * j + 1]), __float_as_uint(v[2 * j]), 0x07060302);
            f[p].u = make_uint4(w[0], w[1], w[2], w[3]);
            o.part[p] = f[p].v;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] -= __uint_as_float(__float_as_uint(v[j]) & 0xffff0000u);
        }
    }
    return o;
}

// acc + a b, the smallest part of b first
template <int D>
__device__ __forceinline__ f32x16 mfma_parts(bf16x8 a, const Operand<D>& b, f32x16 acc) {
#pragma unroll
    for (int p = kPartsOf<D> - 1; p >= 0; --p) acc = mfma(a, b.part[p], acc);
    return acc;
}

// max / sum across the two half-waves that share a column: what either of them holds, the same in both
struct Halves {
    float lo, hi;
};
__device__ inline Halves halves(float x) {
    const uint32_t u = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// row of the 32x32 accumulator that register i of lane-half g holds
__device__ inline int acc_row(int i, int g) { return (i >> 2) * 8 + 4 * g + (i & 3); }

// Asynchronous global -> LDS copies (global_load_lds_*): no staging registers.
// One wave instruction writes lane l's 16 (or 4) bytes at LDS base + 16 (4) * l, the
// base being wave-uniform (M0).  The copies are issued from inline assembly on
// purpose: the compiler's wait-count bookkeeping treats every LDS read that follows a
// copy it knows of as dependent on it and waits for vmcnt(0) there, which would
// serialise each copy with the arithmetic it is meant to overlap.  Completion is
// therefore tracked by hand: copies retire in issue order, dma_wait_barrier<N>()
// waits until at most N of this wave's copies are in flight and then joins the
// workgroup barrier.  Compiler-issued vector memory loads stay correct (its waits can
// only be stricter than needed); inside the tile loops there are none except the tile
// list refills, which are consumed right after a full wait.
// The copies also write M0 (the LDS base).  The compiler refuses M0 in a clobber list (it is
// a reserved register), so the statements cannot declare it; what makes this sound is that
// compiled code for gfx950 keeps nothing alive in M0 in these kernels, which a test on the
// compiled ISA pins (no instruction outside the assembly statements names M0).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) char*)p));
}

__device__ __forceinline__ void dma4(const void* src, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(src) : "memory");
}
// the same from a wave-uniform address plus a lane's offset
__device__ __forceinline__ void dma4(const void* base, uint32_t lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(lane_off), "s"(base) : "memory");
}

template <int N>
__device__ __forceinline__ void dma_wait_barrier() {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Copy of a 64-row tile (rows `row_bytes` apart in global memory) into a swizzled LDS tile.
// A wave instruction fills 1024 bytes, four tile rows (d = 128) or eight (d = 64), so the
// swizzle is applied on the global side: lane l fetches the logical chunk that belongs at its
// physical chunk.  Each of the four waves of a workgroup copies 16 rows in D / 32
// instructions; DmaLaneOf holds the lane's byte offsets for them, so that a copy costs no
// vector ALU work: the address is a scalar tile base plus that 32-bit lane offset.
template <int D>
struct DmaLaneOf {
    uint32_t off[D / 32];
};

// `w` (wave index in the workgroup) must be wave-uniform; rows past `last_row` re-read it
template <int D = 128>
__device__ __forceinline__ DmaLaneOf<D> dma_lane(uint32_t row_bytes, int w, int l, int last_row = 63) {
    DmaLaneOf<D> d;
    constexpr int kChunks = D / 8, kRows = 64 / kChunks;  // 16-byte chunks of a row, rows per instruction
#pragma unroll
    for (int i = 0; i < D / 32; ++i) {
        const int row = 16 * w + kRows * i + l / kChunks;
        d.off[i] = static_cast<uint32_t>(min(row, last_row)) * row_bytes + (((l % kChunks) ^ row_swizzle<D>(row)) << 4);
    }
    return d;
}

__device__ __forceinline__ void dma16(const void* base, uint32_t lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_base)), "v"(lane_off), "s"(base) : "memory");
}

// Copy of a pair of tiles (K and V of one key block, or Q and dO of one query block) as
// eight separate instructions per lane, so that a kernel can spread them over its MFMA
// slots: issued back to back they hold the wave for about a thousand cycles (the CU's
// address unit takes one such instruction per ~16 cycles and the waves of a workgroup issue
// theirs at the same moment).  One piece every other slot keeps the unit's queue short.
// The first D / 32 pieces belong to the first tile, the rest to the second.
template <int D = 128>
struct PairCopyOf {
    const char* a;  // first row of the first tile (wave-uniform)
    const char* b;  // first row of the second tile
    DmaLaneOf<D> lane;
};

// Lane offsets of a kernel's tiles.  Rows past the end of the buffer re-read its last one, in the one clipped tile of a list, which
// stands at its end: the offsets are made again where the last row changes, by a branch that is taken once or twice in a
// kernel, and not chosen for every tile (eight moves per tile, with nothing to cover them).
template <typename Offsets>
__device__ __forceinline__ void tile_rows(int last, int& cp_last, Offsets&& make) {
    if (last == cp_last) return;
    cp_last = last;
    asm volatile("; clipped tile" : "+s"(last));  // keeps the clamped offsets' arithmetic in this branch
    make(last);
}

template <int P, int D>
__device__ __forceinline__ void pair_copy_piece(const PairCopyOf<D>& c, const char* tile_a, const char* tile_b, int w) {
    constexpr int n = D / 32;
    if constexpr (P < n) dma16(c.a, c.lane.off[P], lds_addr(tile_a) + 16 * w * kRowBytesOf<D> + 1024 * P);
    else dma16(c.b, c.lane.off[P - n], lds_addr(tile_b) + 16 * w * kRowBytesOf<D> + 1024 * (P - n));
}

__device__ __forceinline__ uint32_t pack2(float a, float b) {
    f32x2 v = {a, b};
    union { bf16x2 p; uint32_t u; } o;
    o.p = __builtin_convertvector(v, bf16x2);
    return o.u;
}

// Stores one 32-wide block (head dims 32 db ..) of the wave's 32 output rows: `x` is an accumulator whose column is
// the lane's row.  A lane holds pieces of four head dims, 8 bytes in bf16, of one row; stored like that, every store
// instruction would scatter 32 pieces of 16 bytes.  Two rounds of lane swaps first: between the half-waves (the two
// pieces of 8 bytes that make 16), then between the 16-lane halves of each (rows r and r + 16 trade 16-byte chunks),
// after which an instruction writes 64 contiguous bytes of each of 16 rows.
// `base`: row 0 of the wave's 32; `row_elems`: elements between rows; rows from n_rows on are not stored.
__device__ __forceinline__ void store_block(uint16_t* base, size_t row_elems, int n_rows, int db, const f32x16& x, float factor, int l) {
    uint32_t c[2][4];  // 16-byte chunks 2 k + g of the block, k = 0, 1
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = 8 * k + 2 * j;
            const auto r = __builtin_amdgcn_permlane32_swap(pack2(x[i] * factor, x[i + 1] * factor), pack2(x[i + 4] * factor, x[i + 5] * factor), false, false);
            c[k][j] = r[0];
            c[k][2 + j] = r[1];
        }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const auto r = __builtin_amdgcn_permlane16_swap(c[0][j], c[1][j], false, false);
        c[0][j] = r[0];
        c[1][j] = r[1];
    }
    const int row = l & 15;
    uint16_t* p = base + row * row_elems + 32 * db + 16 * ((l >> 4) & 1) + 8 * (l >> 5);
    if (row < n_rows) *reinterpret_cast<uint4*>(p) = make_uint4(c[0][0], c[0][1], c[0][2], c[0][3]);
    if (row + 16 < n_rows) *reinterpret_cast<uint4*>(p + 16 * row_elems) = make_uint4(c[1][0], c[1][1], c[1][2], c[1][3]);
}

// Between LDS accesses by which the lanes of a wave hand values to each other.  LDS takes a wave's instructions in order; the
// compiler keeps that order only where one lane's own addresses may meet, which is not where the values go.  No instruction.
__device__ __forceinline__ void lds_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A wave's 32 rows of a tensor on their way through LDS, so that memory is read and written in whole rows.  Operands loaded
// straight into their registers take 32 bytes of each of 32 rows at a time: a line is asked for by four instructions, by which
// time the eight waves of a CU have pushed it out of their 32 KB of L1.  (Taking the same loads non-temporally, so that every
// one of the four goes to memory, slows dQ of packed short samples from 680 to 912 us, which is what gave it away; fetching the rows into
// L2 beforehand changes nothing.)  Accumulators stored straight from theirs write 64 bytes of each of 16 rows.  In LDS the rows stand
// as in a tile, 0 - 15 at `a` and 16 - 31 at `b`: the two places that the wave itself fills when it copies its share of a pair
// of tiles.  Measured, straight / through LDS, in us: 65 536 tokens of packed samples of 450, 32 / 8 heads, forward 490 / 460,
// dQ 637 / 549; 33 506 tokens in samples of 2 100 692 / 676, 872 / 834; 64 / 8 heads, samples of 5 000 tokens, 4 430 / 4 362,
// 5 660 / 5 458.
//   dK/dV by itself, K and V in straight / through LDS: 850 / 809 on those packed samples, 183 / 178 on 8 334 tokens in samples
// of 1 000, 1 300 / 1 265 on the 33 506 tokens, 30.6 / 30.0 (whole backward) on one sample of 221, at head_dim 64 71.5 / 71.0 on 4 758
// tokens, 29.4 / 29.2 (whole backward) on 900 tokens, 8 / 8 heads.  dK and dV out: at head_dim 128
// through LDS loses, 807 / 801, 177.5 / 176.3, 129.6 / 129.1 on four samples of 1 280, 42.8 / 41.6 on eight of 560 with 16 / 16
// heads, 37.3 / 37.0 (whole backward) on 500 tokens, and even on long rows, so they go straight; at 64 it is even but for small
// grids (whole backward of 900 tokens on 8 / 8 heads 29.2 / 28.9).
template <int D>
struct Rows {
    static constexpr int kRB = kRowBytesOf<D>, kChunks = D / 8, kPieces = D / 16;  // 16-byte chunks of a row; pieces of 1024 bytes
    char *a, *b;
    template <int P>
    __device__ __forceinline__ char* piece() const { return P < kPieces / 2 ? a + 1024 * P : b + 1024 * (P - kPieces / 2); }
    // byte offset from the first row of what lane l moves in a piece, rows row_bytes apart; rows past `last_row` become it
    static __device__ __forceinline__ uint32_t lane_off(int p, uint32_t row_bytes, int l, int last_row) {
        const int row = 64 / kChunks * p + l / kChunks;
        return static_cast<uint32_t>(min(row, last_row)) * row_bytes + (((l % kChunks) ^ row_swizzle<D>(row)) << 4);
    }
    __device__ __forceinline__ void copy_in(const void* base, uint32_t row_bytes, int l, int last_row) const {
        static_for<0, kPieces>([&](auto P) {
            constexpr int p = decltype(P)::value;
            dma16(base, lane_off(p, row_bytes, l, last_row), lds_addr(piece<p>()));
        });
    }
    // what lane l has moved in piece P
    template <int P>
    __device__ __forceinline__ uint4 chunk(int l) const { return *reinterpret_cast<const uint4*>(piece<P>() + 16 * l); }
    template <int P>
    __device__ __forceinline__ void put_chunk(u32x4 x, int l) const { *reinterpret_cast<u32x4*>(piece<P>() + 16 * l) = x; }
    // row l % 32 as MFMA operands
    __device__ __forceinline__ void operands(Frag8 (&f)[D / 16], int l, int nat) const {
        const char* at = l & 16 ? b - 16 * kRB : a;
        static_for<0, D / 16>([&](auto S) { f[decltype(S)::value].v = ld_rows<decltype(S)::value>(at, nat); });
    }
    // ... and back
    __device__ __forceinline__ void put_operands(const Frag8 (&f)[D / 16], int l, int nat) const {
        char* const at = l & 16 ? b - 16 * kRB : a;
        static_for<0, D / 16>([&](auto S) { *reinterpret_cast<uint4*>(at + (nat ^ (decltype(S)::value << 5))) = f[decltype(S)::value].u; });
    }
    // head dims 32 db .. of an accumulator whose column is row l % 32: a lane holds pieces of four head dims, 8 bytes in bf16.
    // Rows r and r + 16 share a swizzle, so a half-wave meets every 16-byte slot twice: 64 cycles of bank conflicts per wave and
    // output at d = 128.
    __device__ __forceinline__ void put(int db, const f32x16& x, float factor, int l) const {
        const int row = l & 31;
        char* const at = (row & 16 ? b - 16 * kRB : a) + row * kRB + 8 * (l >> 5);
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            *reinterpret_cast<uint2*>(at + (((4 * db + i4) ^ row_swizzle<D>(row)) << 4)) =
                make_uint2(pack2(x[4 * i4] * factor, x[4 * i4 + 1] * factor), pack2(x[4 * i4 + 2] * factor, x[4 * i4 + 3] * factor));
    }
    // the first n_rows rows to memory
    __device__ __forceinline__ void copy_out(void* base, uint32_t row_bytes, int l, int n_rows) const {
        uint4 x[kPieces];
        lds_exchange();
        static_for<0, kPieces>([&](auto P) { x[decltype(P)::value] = chunk<decltype(P)::value>(l); });
        lds_exchange();
        static_for<0, kPieces>([&](auto P) {
            constexpr int p = decltype(P)::value;
            if (64 / kChunks * p + l / kChunks < n_rows) *reinterpret_cast<uint4*>(static_cast<char*>(base) + lane_off(p, row_bytes, l, 31)) = x[p];
        });
    }
};

// Reader of a tile list walked in one direction: position k = 0, 1, ... maps to
// list[first + step * k] (step = +1 or -1), n positions in all.  Lane l keeps entry
// 64 b + l of the current batch b; the next batch is requested when a batch is entered,
// i.e. 64 positions before its first use.  get(k) must be called with non-decreasing k,
// from wave-uniform control flow.  The refill is a compiler-tracked load, waited for with
// vmcnt(0), which waits for every asynchronous copy in flight as well: the tile loops call get()
// where there is none.  Ahead of the loops the trimming of shared queries and the second group of a
// split dK/dV row call it while Q, dO, K or V rows are on their way, and wait for those too.
struct EntryStream {
    const int* list;
    int first, step, n, l;
    int cur, nxt, batch;
    __device__ __forceinline__ int fetch(int b) const {
        const int k = min(64 * b + l, n - 1);
        return list[first + step * k];
    }
    // the list of row `rl` of a grid, forwards (step 1) or backwards (step -1)
    template <int GRID>
    __device__ __forceinline__ void init(const DeviceMeta& m, const RowLaunch& rl, int step_, int l_) {
        list = m.list.entry[GRID];
        step = step_; n = rl.count; l = l_;
        first = step > 0 ? rl.begin : rl.begin + n - 1;
        batch = 0;
        nxt = 0;
        if (m.in_args) {
            cur = small_entries(static_cast<uint32_t>(rl.begin), step, n);
            return;
        }
        cur = n > 0 ? fetch(0) : 0;
        nxt = n > 64 ? fetch(1) : 0;
    }
    __device__ __forceinline__ int get(int k) {
        if ((k >> 6) != batch) {
            batch = k >> 6;
            cur = nxt;
            if (64 * (batch + 1) < n) nxt = fetch(batch + 1);
        }
        return __builtin_amdgcn_readlane(cur, k & 63);
    }
    __device__ __forceinline__ int peek(int k) const { return __builtin_amdgcn_readlane(cur, k & 63); }  // k in the current batch
};

// What a wave of a q-major kernel works on: 32 queries of one head.  Where a kv group has a multiple of four heads, the four
// waves of a workgroup take four heads of it on the same queries, otherwise one head on 128 queries.  A workgroup stages and
// waits for every tile that one of its waves reads: with short samples 128 neighbouring queries read 5.6 tiles where 32 read
// 4.3 (65 536 tokens of packed samples of 450), with samples of 5 000 tokens 34.1 and 33.1.  Measured, one head / four, forward
// and dQ in us, 32 q / 8 kv heads: those short samples 487 / 463 and 677 / 625, 8 334 tokens in samples of 1 000 103 / 101 and
// 136 / 131, 33 506 tokens in samples of 2 100 682 / 675 and 873 / 855; 64 / 8 heads, samples of 5 000 tokens, 4 365 / 4 331 and
// 5 612 / 5 556; head_dim 64, 4 758 tokens, 46 / 43 and 49 / 46.  Which tile comes first is known only once the descriptors of
// the queries are, so a grid that the chip holds at once, which lasts as long as one workgroup, keeps one head: a step of one
// sample of 221 tokens 46.8 / 48.9.  At head_dim 64 the chip holds 768 workgroups at once, but four heads are the faster way from
// 513 on there too: 640 / 704 / 768 workgroups, forward 14.2 / 13.7, 14.4 / 14.1, 14.6 / 14.5, backward 38.3 / 37.6, 39.3 / 38.8,
// 40.3 / 39.8.
constexpr int kTwoPerCu = 512;  // workgroups
struct QueryBlock {
    int kvh, h;     // kv head, q head
    int row;        // position in the launch order of the q-tile of 128
    int first;      // the wave's first query, in the q-tile
    bool together;  // the waves share their queries
};
__device__ __forceinline__ QueryBlock query_block(int Hq, int Hkv, int n_rows, int w) {
    // heads of one kv group are neighbours in launch order and share an XCD when Hkv == 8
    const int G = Hq / Hkv, rest = blockIdx.x / Hkv, j = rest % G;
    QueryBlock b;
    b.kvh = blockIdx.x % Hkv;
    b.row = rest / G;
    b.together = (G & 3) == 0 && static_cast<int64_t>(n_rows) * Hq > kTwoPerCu;
    // the last queries of a tile have the longest lists and go first
    b.first = 32 * (b.together ? 3 - (j & 3) : w);
    b.h = b.kvh * G + (b.together ? (j & ~3) + w : j);
    return b;
}

// Whether one of the 32 queries from q0 on (tk: this lane's) may read a key of the tile of list entry e.
__device__ __forceinline__ bool reads_tile(int e, int q0, const Tok4& tk) {
    const int k0 = (e >> 2) * 64;
    // k0 <= q0 is k0 <= q for all 32: tiles of keys start at multiples of 64
    return (e & 3) == PSATTN_TILE_FULL ||
           (k0 <= q0 && __builtin_amdgcn_ballot_w64(k0 + 63 >= tk.s && !(tk.hole_lo <= k0 && k0 + 64 <= tk.hole_hi)) != 0);
}

// ---- rotary position embedding (Section 3.1: position ids follow the paired format)
// Dimension i < 64 is paired with i + 64 and the pair is turned by the angle of (position, i).
// The table row of a position holds cos of the 64 angles, then sin.  All layouts in these kernels
// keep both members of a pair in the same lane, so rotating is lane-local.

// position id of token t: prompt and first response count on from the sample's start; a later
// response skips the hidden range [hole_lo, hole_hi), which puts it right behind the prompt
__device__ inline int rope_position(const Tok4& tk, int t) {
    return tk.s == kPadStart ? 0 : t - tk.s - (tk.hole_hi - tk.hole_lo);
}

// (x1, x2) -> turned by +angle (inverse = false) or -angle (inverse = true)
template <bool INVERSE>
__device__ __forceinline__ void rope_turn(float& x1, float& x2, float c, float s) {
    const float y1 = INVERSE ? fmaf(x2, s, x1 * c) : fmaf(-x2, s, x1 * c);
    const float y2 = INVERSE ? fmaf(-x1, s, x2 * c) : fmaf(x1, s, x2 * c);
    x1 = y1;
    x2 = y2;
}

// What rope_frag8 takes of the table row `row` of the token's position for dims i0 .. i0 + 7, i0 < 64: cosines, then sines.
__device__ __forceinline__ void rope_load8(float4* turn, const float* row, int i0) {
    turn[0] = *reinterpret_cast<const float4*>(row + i0);
    turn[1] = *reinterpret_cast<const float4*>(row + i0 + 4);
    turn[2] = *reinterpret_cast<const float4*>(row + 64 + i0);
    turn[3] = *reinterpret_cast<const float4*>(row + 64 + i0 + 4);
}

// Rotates 8 packed bf16 (dims i0 .. i0 + 7) and their partners (dims 64 + i0 ..) in place
__device__ __forceinline__ void rope_frag8(Frag8& lo, Frag8& hi, const float4* turn) {
    const float4 c0 = turn[0], c1 = turn[1], s0 = turn[2], s1 = turn[3];
    const float cs[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
    const float sn[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
    uint32_t lw[4] = {lo.u.x, lo.u.y, lo.u.z, lo.u.w}, hw[4] = {hi.u.x, hi.u.y, hi.u.z, hi.u.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float a0 = __uint_as_float(lw[j] << 16), a1 = __uint_as_float(lw[j] & 0xffff0000u);
        float b0 = __uint_as_float(hw[j] << 16), b1 = __uint_as_float(hw[j] & 0xffff0000u);
        rope_turn<false>(a0, b0, cs[2 * j], sn[2 * j]);
        rope_turn<false>(a1, b1, cs[2 * j + 1], sn[2 * j + 1]);
        f32x2 va = {a0, a1}, vb = {b0, b1};
        lo.p[j] = __builtin_convertvector(va, bf16x2);
        hi.p[j] = __builtin_convertvector(vb, bf16x2);
    }
}

// Finished sums of a wave (accumulator whose column is the lane's row) that are not all finite, as bits: group 4 db + i4
// is head dims 32 db + 8 i4 + 4 g .. + 3.
template <int N>
__device__ __forceinline__ uint32_t not_finite_groups(const f32x16 (&x)[N]) {
    uint32_t bits = 0;
#pragma unroll
    for (int n = 0; n < 4 * N; ++n) {
        uint32_t top = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) top = max(top, __float_as_uint(x[n >> 2][4 * (n & 3) + c]) & 0x7fffffffu);
        if (top >= 0x7f800000u) bits |= 1u << n;
    }
    return bits;
}
template <int N>
__device__ __forceinline__ void set_group(f32x16 (&x)[N], int n, const f32x4& v) {
#pragma unroll
    for (int m = 0; m < 4 * N; ++m)
#pragma unroll
        for (int c = 0; c < 4; ++c) x[m >> 2][4 * (m & 3) + c] = m == n ? v[c] : x[m >> 2][4 * (m & 3) + c];
}
// Walks the groups that not_finite_groups has named, of the rows [row0, row0 + 32) below T.  Rare: row and half are found
// anew from the lane's number, so that the kernel's loop keeps no registers for it.
struct AgainGroups {  // for (AgainGroups n(bits, row0, T); n.any(); n.next()): group n.group(), head dims n.dim() .. + 3 of row n.row
    uint32_t bits;
    int row, half;
    __device__ __forceinline__ AgainGroups(uint32_t b, int row0, int T) : bits(b) {
        const int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
        row = row0 + (l & 31);
        half = l >> 5;
        if (row >= T) bits = 0;
    }
    __device__ __forceinline__ bool any() const { return bits != 0; }
    __device__ __forceinline__ void next() { bits &= bits - 1; }
    __device__ __forceinline__ int group() const { return __builtin_ctz(bits); }
    __device__ __forceinline__ int dim() const { return 32 * (group() >> 2) + 8 * (group() & 3) + 4 * half; }
};
template <int N>
__device__ __forceinline__ void multiply(f32x16 (&x)[N], float factor) {
#pragma unroll
    for (int db = 0; db < N; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) x[db][i] *= factor;
}

}  // namespace mma
}  // namespace psattn
