// bf16 MFMA dK/dV kernel for gfx950; layout and staging helpers are in psattn_mfma_common.h.
//
// grid: one workgroup per (k-tile of 128 keys, kv-head); 4 waves x 32 keys, one wave per
// SIMD (or two workgroups of 64 keys for the same, on grids that are bound by their longest row: see psattn_dkdv_bf16_mfma).  The workgroup walks the G query heads of its group and, for each, the q-tiles
// (64 queries) that can read its keys (the k-major tile list of the block mask, paper
// Section 3.1), so the prompt's keys collect the contributions of prompt, chosen and
// rejected queries in one place, without atomics.
//
// Register plan.  A wave keeps dK and dV of its 32 keys (2 x 64 fp32 per lane) and its K
// and V fragments (2 x 32 registers per lane) for the whole kernel: 192 registers that only
// MFMA instructions ever touch.  They live in the accumulation registers a[0:191], which
// MFMA reads and writes directly and the vector ALU cannot address; the ordinary registers
// are left to the scores, the LDS operand ring and the softmax arithmetic.  The compiler
// cannot express this split (once a kernel needs more than 256 registers it sends either
// every MFMA result or none to the accumulation registers, and moves whole accumulators
// back and forth), so all MFMAs of this kernel are issued from inline assembly that names
// the accumulation registers itself; everything else is ordinary compiled code.  This file
// is built with the compiler's own use of accumulation registers for spilling switched off,
// so a[0:191] belong to the assembly alone.
//
// The compiler does not know that the assembly statements are MFMAs and inserts no wait
// states after them: settle() stands wherever another kind of instruction reads what a
// chain of MFMAs has produced.
#include "psattn_mfma_common.h"

namespace psattn {
namespace {
using namespace mma;

constexpr int kAccDV = 0;     // a[16 db + i]: dV^T block db (head dims 32 db ..), accumulator element i
constexpr int kAccDK = 64;    // likewise dK^T
constexpr int kRegK = 128;    // a[128 + 4 t ..]: K fragment of step t (head dims 16 t ..), B operand
constexpr int kRegV = 160;    // likewise V
constexpr int kAccRegs = 192;

// a[A0 : A0 + 15] += x y
template <int A0>
__device__ __forceinline__ void acc_mfma(bf16x8 x, bf16x8 y) {
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(A0), "n"(A0 + 15), "v"(x), "v"(y));
}

// acc (ordinary registers) = x * a[B0 : B0 + 3] (+ acc unless FIRST)
template <int B0, bool FIRST>
__device__ __forceinline__ void score_mfma(f32x16& acc, bf16x8 x) {
    if constexpr (FIRST)
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], 0" : "=&v"(acc) : "v"(x), "n"(B0), "n"(B0 + 3));
    else
        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, a[%2:%3], %0" : "+v"(acc) : "v"(x), "n"(B0), "n"(B0 + 3));
}

template <int A>
__device__ __forceinline__ void acc_set(uint32_t v) {
    asm volatile("v_accvgpr_write_b32 a[%0], %1" ::"n"(A), "v"(v));
}

template <int A>
__device__ __forceinline__ float acc_get() {
    float v;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(v) : "n"(A));
    return v;
}

// 24 wait states: more than the longest MFMA needs before its result may be read
__device__ __forceinline__ void settle() {
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
}

// ------------------------------------------------------------------ one q-tile
// With one wave per SIMD nothing hides latency but the wave's own instruction stream, so a
// q-tile is processed as 64 explicitly ordered slots, one MFMA each:
//   slots  0-15  S, dP of queries 0-31
//   slots 16-31  S, dP of queries 32-63      + softmax/dS arithmetic of queries 0-31
//   slots 32-47  dV, dK from queries 0-31    + softmax/dS arithmetic of queries 32-63
//   slots 48-63  dV, dK from queries 32-63
// The LDS operand of slot m is requested kAhead slots earlier into a register ring.

constexpr int kQTileBytes = 64 * kRowBytes;
constexpr int kAhead = 4;  // measured: 3 and 5 are both slower

// Which of a lane's elements of a q-tile are allowed, the queries that read its key being rows [lo, hi) of the tile: bit j for
// element 2 j, bit 16 + j for element 2 j + 1.
__device__ inline uint32_t pair_bits(int lo, int hi, int g) {
    const int a = elems_below(min(max(lo, 0), 64), g), b = elems_below(min(max(hi, 0), 64), g);
    const auto below = [](int n) { return ((1u << ((n + 1) >> 1)) - 1) | ((1u << (n >> 1)) - 1) << 16; };
    return below(b) & ~below(a);
}
// AND-mask for the packed bf16 pair J (elements 2 J, 2 J + 1), by two instructions: each half moves its bit to the sign and fills
// itself with it.  All sixteen masks ahead of the tile's first MFMA took 70 instructions, which nothing hid.
template <int J>
__device__ __forceinline__ uint32_t pair_mask(uint32_t bits) {
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    s16x2 x = __builtin_bit_cast(s16x2, bits);
    x = x << static_cast<short>(15 - J);
    return __builtin_bit_cast(uint32_t, x >> static_cast<short>(15));
}

__device__ inline uint32_t word(const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ inline float comp(const float4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// The LDS operands of the first kAhead slots (Q and dO rows of query block 0, head dims 0-31),
// requested as soon as the tile's data is visible so that the list bookkeeping between the barrier
// and the first MFMA overlaps their latency (configuration 5: 8.38 -> 8.30 ms).
__device__ __forceinline__ void tile_prefetch(Frag8 (&ring)[8], const char* sQ, const char* sG, const LaneOffsets& lo) {
    static_for<0, kAhead>([&](auto M) {
        constexpr int m = decltype(M)::value, t = m >> 1;
        ring[m & 7].v = ld_rows<t>((m & 1) ? sG : sQ, lo.nat);
    });
}

// FULL: every pair of the tile is allowed, no mask work at all (`bits`, from pair_bits, is not read).
// copy_piece(k), k = 0 .. PIECES - 1, issues one instruction of the next tile's asynchronous copy;
// the pieces are spread over the first slots.
template <bool FULL, int PIECES, typename CopyPiece>
__device__ __forceinline__ void dkdv_tile(const char* sQ, const char* sG, const float* sL, const float* sD,
                                          const LaneOffsets& lo, uint32_t bits, float c, int g,
                                          Frag8 (&ring)[8], CopyPiece&& copy_piece) {
    f32x16 s[2], dp[2];
    u32x4 pw[2][2], dw[2][2];  // packed P and dS of a block: [block][half] is one B operand
    float4 Lc, Ln;
    float p0 = 0.f, p1 = 0.f;
    uint32_t mask = 0;

    auto request = [&](auto M) {  // LDS operand of slot m -> ring[m % 8]
        constexpr int m = decltype(M)::value;
        if constexpr (m < 32) {
            constexpr int b = m >> 4, t = (m & 15) >> 1;
            const char* x = (m & 1) ? sG : sQ;
            ring[m & 7].v = ld_rows<t>(x + b * 32 * kRowBytes, lo.nat);
        } else if constexpr (m < 64) {
            constexpr int j = (m - 32) & 15, b = (m - 32) >> 4, half = j >> 3, db = (j & 7) >> 1;
            const char* x = (j & 1) ? sQ : sG;
            ring[m & 7].v = ld_cols<db, half>(x + 32 * b * kRowBytes, lo.tr1, lo.tr2);
        }
    };
    // dP accumulators of block b start from -delta of their queries (element i belongs to
    // query 32 b + acc_row(i, g)), so that dS = P o (dP - delta) is one multiplication
    auto start_dp = [&](auto B) {
        constexpr int b = decltype(B)::value;
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const float4 d = *reinterpret_cast<const float4*>(sD + 32 * b + 8 * i4 + 4 * g);
            dp[b][4 * i4] = d.x; dp[b][4 * i4 + 1] = d.y; dp[b][4 * i4 + 2] = d.z; dp[b][4 * i4 + 3] = d.w;
        }
    };
    auto lse4 = [&](int b, int i4) {  // LSE * log2 e of 4 consecutive queries
        return *reinterpret_cast<const float4*>(sL + 32 * b + 8 * i4 + 4 * g);
    };

    // slots 0 .. kAhead - 1 were requested by the caller right behind the barrier (tile_prefetch)
    start_dp(std::integral_constant<int, 0>{});
    Lc = lse4(0, 0);
    static_for<0, 64>([&](auto M) {
        constexpr int m = decltype(M)::value;
        request(std::integral_constant<int, m + kAhead>{});
        // Copy pieces go out every other slot: the four waves issue theirs at the same moment and
        // the CU's address unit takes one such instruction per ~16 cycles, so a piece per slot
        // from each wave would queue up and stall the waves.
        if constexpr (m < 2 * PIECES && (m & 1) == 0) copy_piece(std::integral_constant<int, m / 2>{});
        if constexpr (m == 10) start_dp(std::integral_constant<int, 1>{});
        // One wait per two slots: naming the next slot's operand here makes the compiler wait
        // for both now (the statement itself is empty), and the odd slot then needs none.
        if constexpr ((m & 1) == 0) asm volatile("" ::"v"(ring[(m + 1) & 7].v));
        if constexpr (m < 32) {
            constexpr int b = m >> 4, t = (m & 15) >> 1;
            if constexpr (m & 1) score_mfma<kRegV + 4 * t, false>(dp[b], ring[m & 7].v);  // dP - delta = dO V^T - delta
            else score_mfma<kRegK + 4 * t, t == 0>(s[b], ring[m & 7].v);                   // S = Q K^T
        } else {
            constexpr int j = (m - 32) & 15, b = (m - 32) >> 4, half = j >> 3, db = (j & 7) >> 1;
            if constexpr (j & 1) acc_mfma<kAccDK + 16 * db>(ring[m & 7].v, __builtin_bit_cast(bf16x8, dw[b][half]));
            else acc_mfma<kAccDV + 16 * db>(ring[m & 7].v, __builtin_bit_cast(bf16x8, pw[b][half]));
        }
        if constexpr (m >= 16 && m < 48) {
            // slot pair (2j, 2j + 1) of the phase turns accumulator elements 2j, 2j + 1 of
            // block b into packed P and packed dS: the exponentials in the even slot, the
            // rest in the odd one
            constexpr int n = m - 16, b = n >> 4, k = n & 15, j = k >> 1, i = 2 * j;
            // No wait states are needed here: the chain that produced S of block b (k = 0) or dP
            // (k = 1) ended three slots ago, and the two MFMAs issued since then each held the
            // matrix pipeline for as long as an MFMA takes to finish.
            if constexpr ((k & 3) == 0 && n + 4 < 32) Ln = lse4((n + 4) >> 4, ((n + 4) & 15) >> 2);
            if constexpr ((k & 1) == 0) {
                if constexpr (!FULL) mask = pair_mask<8 * b + j>(bits);
                p0 = __builtin_amdgcn_exp2f(fmaf(s[b][i], c, -comp(Lc, i & 3)));
                p1 = __builtin_amdgcn_exp2f(fmaf(s[b][i + 1], c, -comp(Lc, (i + 1) & 3)));
            } else {
                pw[b][j >> 2][j & 3] = FULL ? pack2(p0, p1) : pack2(p0, p1) & mask;
                const float d0 = p0 * dp[b][i], d1 = p1 * dp[b][i + 1];
                dw[b][j >> 2][j & 3] = FULL ? pack2(d0, d1) : pack2(d0, d1) & mask;
            }
            if constexpr ((k & 3) == 3) Lc = Ln;
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

// S = 1: the four waves hold 128 keys and walk the list together.
// S = 2: a workgroup holds 64 keys, two waves each, twice over: its two groups of waves take every other step of the walk
// (a step is one head on one q-tile) with tiles of their own, and their partial sums are added in LDS at the end.  Twice as
// many workgroups, each half as long; see launch_mfma_dkdv for when.
template <int S>
__global__ __launch_bounds__(256) void psattn_dkdv_bf16_mfma(AttnArgs a) {
    constexpr int kWaves = 4 / S, kRows = 64 / kWaves, kOps = kRows / 4, kPieces = 2 * kOps + 1;
    // tiles of Q (two buffers), of dO (two buffers) per group; then LSE * log2(e) and -delta
    __shared__ __attribute__((aligned(16))) char smem[S][4][kQTileBytes];
    __shared__ __attribute__((aligned(16))) float sStat[S][2][2][64];
    __shared__ __attribute__((aligned(16))) char sRows[S == 1 ? 4 * 64 * kRowBytes : 1];  // K and V rows of each wave
    // a[0:191] are in use: makes the kernel's register allocation cover them
    asm volatile("" ::: "a0", "a191");
    fetch_args(a);
    const int tid = threadIdx.x, wg = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, c32 = l & 31, g = l >> 5;
    const int group = S == 1 ? 0 : wg / kWaves, w = S == 1 ? wg : wg % kWaves;  // wave index in its group
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv, G = Hq / Hkv;
    const int kvh = blockIdx.x % Hkv, rest = blockIdx.x / Hkv;
    const RowLaunch rl = row_launch<kGridK>(a.meta, rest / S);  // one scalar load: row, list bounds, first entry
    const int row0 = rl.row * 128 + (rest % S) * (128 / S) + 32 * w;  // the wave's first key
    const int key = row0 + c32;
    const bool kvalid = key < T;
    const TokenLoad begun = token_begin(a.meta, key);
    const float c = a.scale * kLog2e;
    LaneOffsets lo = lane_offsets(l);
    const int l_nat = lo.nat;
    if constexpr (S > 1) {  // the group's tiles
        const int at = group * static_cast<int>(sizeof(smem[0]));
        lo.nat += at;
        lo.tr1 += at;
        lo.tr2 += at;
    }
    // K and V rows of the wave's keys pass through LDS: an unsplit row has room of its own, a split one takes its second buffers
    char* const own = S == 1 ? sRows + 4 * kRowBytes * 16 * w : nullptr;
    const Rows<128> k_rows = S == 1 ? Rows<128>{own, own + 16 * kRowBytes}
                                    : Rows<128>{smem[group][1] + kRows * w * kRowBytes, smem[group][1] + (kRows * w + 16) * kRowBytes};
    const Rows<128> v_rows = S == 1 ? Rows<128>{own + 32 * kRowBytes, own + 48 * kRowBytes}
                                    : Rows<128>{smem[group][3] + kRows * w * kRowBytes, smem[group][3] + (kRows * w + 16) * kRowBytes};
    const uint32_t k_row_bytes = static_cast<uint32_t>(Hkv) * kRowBytes;
    {
        const int last_row = min(max(T - 1 - row0, 0), 31);
        const size_t at0 = (static_cast<size_t>(min(row0, T - 1)) * Hkv + kvh) * kRowBytes;
        k_rows.copy_in(static_cast<const char*>(a.K) + at0, k_row_bytes, l, last_row);
        v_rows.copy_in(static_cast<const char*>(a.V) + at0, k_row_bytes, l, last_row);
    }
    const int n_ent = rl.count;
    const int n_steps = n_ent * G;
    const int n_it = (n_steps - group + S - 1) / S;      // the group's share: steps group, group + S, ...
    const int n_loop = (n_steps + S - 1) / S;            // every wave joins every barrier

    // Staging of one q-tile (64 rows x 256 B of Q and of dO, 64 LSE * log2 e, 64 delta):
    // asynchronous global -> LDS copies, issued one tile ahead into the buffer the
    // previous tile has just vacated; see tile_rows for the last tile of the buffer.  What stands between a tile's barrier and its
    // first MFMA is covered by nothing, so as little as can be is done there: lane offsets that stay, scalar addresses
    // that move on by a head, a tile loop whose buffers alternate without a test.  With the masks beside the MFMAs, backward of
    // eight samples of 1 040 tokens 271 -> 264 us, of one of 8 000 1 454 -> 1 425, of packed samples of 450, 63 000 tokens, 1 278 -> 1 248.
    const uint32_t row_bytes = static_cast<uint32_t>(Hq) * 256u;
    uint32_t cp_lane[kOps], cp_stat;
    int cp_last = 63;  // last row that they are made for
    auto lane_rows = [&](int last) {
        const int lx = opaque(l);
#pragma unroll
        for (int i = 0; i < kOps; ++i) {
            const int row = kRows * w + 4 * i + (lx >> 4);
            cp_lane[i] = static_cast<uint32_t>(min(row, last)) * row_bytes + (((lx & 15) ^ row_swizzle<128>(row)) << 4);
        }
        cp_stat = 4u * static_cast<uint32_t>(min(lx, last));
    };
    lane_rows(63);
    // The copy of one tile is 2 kOps + 1 instructions per lane: the first kOps are Q rows, then dO rows, the last one the
    // statistics.  copy_setup fixes the tile, copy_piece issues one piece.
    const char* cp_q = static_cast<const char*>(a.Q);    // first Q row of the tile being copied (this head)
    const char* cp_g = static_cast<const char*>(a.dO);   // first dO row
    const float* cp_s = a.lse2;                          // first statistic (waves 0, 1)
    auto copy_setup = [&](int ent, int h) {
        const int q0 = (ent >> 2) * 64;
        tile_rows(min(T - 1 - q0, 63), cp_last, lane_rows);
        const size_t tile_elems = (static_cast<size_t>(q0) * Hq + h) * 128;
        cp_q = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.Q) + tile_elems);
        cp_g = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.dO) + tile_elems);
        cp_s = (w ? a.delta : a.lse2) + static_cast<size_t>(h) * T + q0;
    };
    auto copy_piece = [&](auto P, auto BUF) {
        constexpr int p = decltype(P)::value, buf = decltype(BUF)::value;
        if constexpr (p < kOps) dma16(cp_q, cp_lane[p], lds_addr(smem[0][buf]) + group * sizeof(smem[0]) + (kRows * w + 4 * p) * kRowBytes);
        else if constexpr (p < 2 * kOps) dma16(cp_g, cp_lane[p - kOps], lds_addr(smem[0][2 + buf]) + group * sizeof(smem[0]) + (kRows * w + 4 * (p - kOps)) * kRowBytes);
        else if (w < 2) dma4(cp_s, cp_stat, lds_addr(sStat[0][0][buf]) + group * sizeof(sStat[0]) + (w ? sizeof(sStat[0][0]) : 0));  // wave 0: LSE * log2 e, wave 1: -delta
    };
    // Walk order: q-tiles from the last to the first, and for each q-tile the G heads
    // of the group.  Every k-tile of a sample ends at the same q-tile, so workgroups
    // of neighbouring k-tiles (which run at the same time on the same XCD) read the
    // same Q / dO tile at the same moment and share it through L2.
    EntryStream es;
    int pk = 0, ph = 0;  // walk position and head (within the group of heads) of the group's next step
    auto advance = [&](int steps) {
        ph += steps;
        while (ph >= G) { ph -= G; ++pk; }
    };
    int ent = 0, it = 0;
    bool started = false;  // the list
    if (n_steps > 0) {
        ent = rl.first_entry;
        if constexpr (S > 1) {
            advance(group);
            if (pk >= n_ent) pk = ph = 0;  // nothing to do for this group: it copies a tile that it does not use
            if (pk > 0) {
                es.init<kGridK>(a.meta, rl, -1, l);
                ent = es.get(pk);
            }
        }
        started = pk > 0;
        copy_setup(ent, kvh * G + ph);
        static_for<0, kPieces>([&](auto P) { copy_piece(P, std::integral_constant<int, 0>{}); });
        advance(S);
    }
    if (!started) es.init<kGridK>(a.meta, rl, -1, l);
    const Tok4 found = token_search(a.meta, key);
    Tok4 tk = found;  // chosen below; queries [key, tk.key_hi) read this key
    // dK, dV accumulators a[0:127] = 0; K, V fragments -> a[128:191]
    static_for<0, 128>([&](auto R) { acc_set<decltype(R)::value>(0u); });
    {
        if (n_steps > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kOps) : "memory");  // the first tile's copies are younger
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        Frag8 f[8];
        k_rows.operands(f, l, l_nat);
        static_for<0, 32>([&](auto R) { acc_set<kRegK + decltype(R)::value>(word(f[decltype(R)::value / 4].u, decltype(R)::value % 4)); });
        v_rows.operands(f, l, l_nat);
        static_for<0, 32>([&](auto R) { acc_set<kRegV + decltype(R)::value>(word(f[decltype(R)::value / 4].u, decltype(R)::value % 4)); });
    }
    // One tile; the buffer index is a compile-time constant, so every LDS address is a lane
    // constant plus an immediate offset.
    auto tile = [&](auto BUF) {
        constexpr int buf = decltype(BUF)::value;
        // this wave's copies of tile `it` have landed; after the barrier every wave's
        // have, and tile it - 1 (same buffer as it + 1) is no longer read
        dma_wait_barrier<0>();
        Frag8 ring[8];
        const char *sQ = smem[0][buf], *sG = smem[0][2 + buf];  // the group's tiles are behind them by what lo holds
        const float *sL = sStat[group][0][buf], *sD = sStat[group][1][buf];
        tile_prefetch(ring, sQ, sG, lo);
        __builtin_amdgcn_sched_barrier(0);
        const int q0 = (ent >> 2) * 64;
        const bool full = (ent & 3) == PSATTN_TILE_FULL;
        // After the last tile the copy is issued once more (same tile, other buffer): the slots
        // then need no branch around each piece; nobody reads that buffer.
        if (it + 1 < n_it) {
            if (ph < S) {  // another q-tile
                ent = es.get(pk);
                copy_setup(ent, kvh * G + ph);
            } else {       // same q-tile, S heads on: 128 S elements / S T statistics further on
                cp_q += 256 * S;
                cp_g += 256 * S;
                cp_s += S * T;
            }
            advance(S);
        }
        ++it;
        auto piece = [&](auto P) { copy_piece(P, std::integral_constant<int, buf ^ 1>{}); };
        uint32_t bits = 0;
        if (S > 1 && it > n_it) {  // the other group's last step
        } else if (full) {
            dkdv_tile<true, kPieces>(sQ, sG, sL, sD, lo, bits, c, g, ring, piece);
        } else if (__builtin_amdgcn_ballot_w64(max(key, q0) < min(tk.key_hi, q0 + 64)) == 0) {
            // PARTIAL tile none of whose queries reads any of this wave's 32 keys (two of the four
            // waves on the first q-tile of every causal diagonal, and the keys of another sample or
            // response): the wave only issues its share of the next tile's copy
            static_for<0, kPieces>([&](auto P) { piece(P); });
#pragma unroll
            for (int m = 0; m < kAhead; ++m) asm volatile("" ::"v"(ring[m].v));  // nothing is left on its way
        } else {
            bits = pair_bits(key - q0, tk.key_hi - q0, g);
            dkdv_tile<false, kPieces>(sQ, sG, sL, sD, lo, bits, c, g, ring, piece);
        }
    };
    // Every load above has retired before the loop starts, so the loop body holds no
    // wait on a compiler-tracked load (such a wait would also cover the copies in flight).
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    tk = token_choose(a.meta, begun, found);
    settle();  // the register writes above, before the first MFMA reads them
    while (it < n_loop) {
        tile(std::integral_constant<int, 0>{});
        if (it >= n_loop) break;
        tile(std::integral_constant<int, 1>{});
    }
    // no copy may still be writing to LDS when the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    settle();  // the last MFMAs, before dK / dV are read out
    if constexpr (S > 1) {
        // Group 0 hands its dK to group 1, which hands its dV to group 0; each adds the other's part to its own.
        __syncthreads();  // every wave's reads and copies are done: the tiles' space is free
        char* const mine = &smem[0][0][0] + wg * kQTileBytes + 16 * l;
        const char* const theirs = &smem[0][0][0] + (wg ^ kWaves) * kQTileBytes + 16 * l;
        auto give = [&](auto A0) {
            static_for<0, 16>([&](auto I) {
                constexpr int r = decltype(A0)::value + 4 * decltype(I)::value;
                *reinterpret_cast<float4*>(mine + 1024 * decltype(I)::value) = make_float4(acc_get<r>(), acc_get<r + 1>(), acc_get<r + 2>(), acc_get<r + 3>());
            });
        };
        auto take = [&](auto A0) {
            static_for<0, 16>([&](auto I) {
                constexpr int r = decltype(A0)::value + 4 * decltype(I)::value;
                const float4 x = *reinterpret_cast<const float4*>(theirs + 1024 * decltype(I)::value);
                acc_set<r>(__float_as_uint(acc_get<r>() + x.x));
                acc_set<r + 1>(__float_as_uint(acc_get<r + 1>() + x.y));
                acc_set<r + 2>(__float_as_uint(acc_get<r + 2>() + x.z));
                acc_set<r + 3>(__float_as_uint(acc_get<r + 3>() + x.w));
            });
        };
        using DV = std::integral_constant<int, kAccDV>;
        using DK = std::integral_constant<int, kAccDK>;
        if (group) give(DV{}); else give(DK{});
        __syncthreads();
        if (group) take(DK{}); else take(DV{});
    }
    auto get = [&](auto A0) {
        f32x16 x;
        static_for<0, 16>([&](auto I) { x[decltype(I)::value] = acc_get<decltype(A0)::value + decltype(I)::value>(); });
        return x;
    };
    const int lx = opaque(l);
    const size_t out0 = (static_cast<size_t>(row0) * Hkv + kvh) * 128, row_elems = static_cast<size_t>(Hkv) * 128;
    if (S == 1 || group == 0)
        static_for<0, 4>([&](auto DB) {
            constexpr int db = decltype(DB)::value;
            store_block(static_cast<uint16_t*>(a.dV) + out0, row_elems, T - row0, db, get(std::integral_constant<int, kAccDV + 16 * db>{}), 1.f, lx);
        });
    if (S > 1 && group == 0) return;
    if (a.rope) {
        // K arrived rotated: turn dK back by the key's angles (accumulator element 4 i4 + k of block
        // db is head dim 32 db + 8 i4 + 4 g + k; its partner sits in block db + 2)
        const float* trow = a.rope + (kvalid ? static_cast<size_t>(rope_position(tk, key)) * 128 : 0);
        static_for<0, 2>([&](auto DB) {
            constexpr int db = decltype(DB)::value;
            f32x16 x = get(std::integral_constant<int, kAccDK + 16 * db>{}), y = get(std::integral_constant<int, kAccDK + 16 * (db + 2)>{});
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4 c = *reinterpret_cast<const float4*>(trow + 32 * db + 8 * i4 + 4 * g);
                const float4 s = *reinterpret_cast<const float4*>(trow + 64 + 32 * db + 8 * i4 + 4 * g);
                const float cs[4] = {c.x, c.y, c.z, c.w}, sn[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float lo = x[4 * i4 + k], hi = y[4 * i4 + k];
                    rope_turn<true>(lo, hi, cs[k], sn[k]);
                    x[4 * i4 + k] = lo;
                    y[4 * i4 + k] = hi;
                }
            }
            store_block(static_cast<uint16_t*>(a.dK) + out0, row_elems, T - row0, db, x, a.scale, lx);
            store_block(static_cast<uint16_t*>(a.dK) + out0, row_elems, T - row0, db + 2, y, a.scale, lx);
        });
    } else {
        static_for<0, 4>([&](auto DB) {
            constexpr int db = decltype(DB)::value;
            store_block(static_cast<uint16_t*>(a.dK) + out0, row_elems, T - row0, db, get(std::integral_constant<int, kAccDK + 16 * db>{}), a.scale, lx);
        });
    }
}

}  // namespace

// Which of the two.  A workgroup is a serial chain of as many steps (heads of the group x q-tiles) as its row is long, one
// workgroup per CU, so a launch takes at least its longest chain however few workgroups there are; splitting halves the
// chain and costs 10 - 15 % more work (every tile is staged for 64 keys instead of 128) and the exchange at the end.  The
// line lies where the longest chain is 1.6 times a CU's share of all steps, at chains of 8 steps, and already at 1.3 shares
// where the chain is 8 steps longer than those, which pay for the exchange.  Measured, whole backward, unsplit / split, 32 q / 8 kv heads
// by that ratio: 1.00 (three samples of 2 600 tokens) 514 / 534 us, 1.04 258 / 271, 1.19 234 / 243, 1.22 154 / 155, 1.28 230 / 225, 1.48 (four of
// 1 280) 207 / 200, 1.52 417 / 361, 1.60 208 / 182; 64 / 8 heads 1.29 691 / 663; chains too short for it, 28 / 4 heads, 1.31 (130 samples of
// 50 tokens, 21 steps) 83 / 99, 1.47 78 / 92, 16 / 4 heads 1.39 (28 steps) 91 / 110.  228 random tables from 1.3 to 1.6, split over unsplit: all of
// them 0.99 (0.83 - 1.22), the 85 past the line 0.91 (0.83 - 1.04), chains under 24 steps 1.00 - 1.22.  dK/dV
// alone, kernels of before: 1.96 112 / 78, 3.8 105 / 64, 7.5 88 / 54, 24 (180 tokens) 26 / 19; 64 / 8 heads 1.48 246 / 220, 2.96
// 218 / 137, 4.0 322 / 186; 28 / 4 heads 4.8 279 / 159, 8.1 283 / 159; 16 / 16 heads 0.76 42 / 62.
constexpr int64_t kCus = 256;
constexpr bool split_rows(int64_t chain, int64_t steps) {
    return chain >= 8 && (10 * chain * kCus >= 16 * steps || 10 * (chain - 8) * kCus >= 13 * steps);
}

int launch_mfma_dkdv(const AttnArgs& a, void* stream) {
    const unsigned grid = static_cast<unsigned>(a.meta.n_rows[kGridK]) * a.Hkv;
    if (grid == 0) return 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t chain = static_cast<int64_t>(a.size[kGridK].longest) * (a.Hq / a.Hkv), steps = a.size[kGridK].n_entries * a.Hq;
    if (split_rows(chain, steps)) psattn_dkdv_bf16_mfma<2><<<2 * grid, 256, 0, s>>>(a);
    else psattn_dkdv_bf16_mfma<1><<<grid, 256, 0, s>>>(a);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
