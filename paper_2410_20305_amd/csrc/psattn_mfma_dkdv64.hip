// bf16 MFMA dK/dV kernel for gfx950, head_dim 64; layout and staging helpers are in psattn_mfma_common.h.
//
// grid: one workgroup per (k-tile of 128 keys, kv-head), or two of 64 keys; 4 waves x 32 keys.  The walk is that of the head_dim 128
// kernel (the G query heads of the group, and for each the q-tiles of 64 queries that can read the keys, so that the
// prompt's keys collect the contributions of prompt, chosen and rejected queries in one place, without atomics), but
// at half the head dimension dK, dV and the K / V fragments of a wave take 96 registers instead of 192: the whole
// kernel fits 256, the compiler can manage it, and two waves share a SIMD, so that one wave's softmax arithmetic
// meets the other's MFMAs.  What bounds it is both: per 64 x 32 scores a wave issues 64 MFMAs (2 048 cycles of the
// matrix pipeline; P and dS enter as three operands each, see make_operand) and about 515 vector instructions.  Measured
// on a step of 8 samples, 4 758 tokens, 32 q / 8 kv heads: forward + dQ + dK/dV 14.9 ms on one thread per row, 0.18 ms on
// these.
#include "psattn_mfma_common.h"

namespace psattn {
namespace {
using namespace mma;

constexpr int kRB = kRowBytesOf<64>;

// S = 1: the four waves hold 128 keys and walk the list together.  S = 2: a workgroup holds 64 keys, two waves each, twice
// over: its two groups of waves take every other step of the walk (a step is one head on one q-tile) with tiles of their
// own, and their partial sums are added in LDS at the end.  Twice as many workgroups, each half as long; see
// launch_mfma_dkdv64 for when.
template <int S>
__global__ __launch_bounds__(256, 2) void psattn_dkdv64_bf16_mfma(AttnArgs a) {
    constexpr int kWaves = 4 / S, kRows = 64 / kWaves, kOps = kRows / 8, kPieces = 2 * kOps + 1;
    // tiles of Q (two buffers), of dO (two buffers) per group; then LSE * log2(e) and -delta
    __shared__ __attribute__((aligned(16))) char smem[S][4][64 * kRB];
    __shared__ __attribute__((aligned(16))) float sStat[S][2][2][64];
    __shared__ __attribute__((aligned(16))) char sRows[S == 1 ? 4 * 64 * kRB : 1];  // K and V rows, later dK and dV rows, of each wave
    fetch_args(a);
    const int tid = threadIdx.x, wg = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, c32 = l & 31, g = l >> 5;
    const int group = S == 1 ? 0 : wg / kWaves, w = S == 1 ? wg : wg % kWaves;  // wave index in its group
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv, G = Hq / Hkv;
    const int kvh = blockIdx.x % Hkv, rest = blockIdx.x / Hkv;
    const RowLaunch rl = row_launch<kGridK>(a.meta, rest / S);  // one scalar load: row, list bounds, first entry
    const int row0 = rl.row * 128 + (rest % S) * (128 / S) + 32 * w;  // the wave's first key
    const int key = row0 + c32;
    const TokenLoad begun = token_begin(a.meta, key);
    // K and V rows of the wave's keys pass through LDS: an unsplit row has room of its own, a split one takes its second buffers
    char *const k_at = S == 1 ? sRows + 64 * kRB * w : smem[group][1] + kRows * w * kRB;
    char *const v_at = S == 1 ? k_at + 32 * kRB : smem[group][3] + kRows * w * kRB;
    const Rows<64> k_rows{k_at, k_at + 16 * kRB}, v_rows{v_at, v_at + 16 * kRB};
    const uint32_t k_row_bytes = static_cast<uint32_t>(Hkv) * kRB;
    {
        const int last_row = min(max(T - 1 - row0, 0), 31);
        const size_t at0 = (static_cast<size_t>(min(row0, T - 1)) * Hkv + kvh) * kRB;
        k_rows.copy_in(static_cast<const char*>(a.K) + at0, k_row_bytes, l, last_row);
        v_rows.copy_in(static_cast<const char*>(a.V) + at0, k_row_bytes, l, last_row);
    }
    Frag8 kf[4], vf[4];
    f32x16 dk[2], dv[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) { dk[db][i] = 0.f; dv[db][i] = 0.f; }

    const float c = a.scale * kLog2e;
    LaneOffsets lo = lane_offsets<64>(l);
    const int l_nat = lo.nat;
    if constexpr (S > 1) {  // the group's tiles
        const int at = group * static_cast<int>(sizeof(smem[0]));
        lo.nat += at;
        lo.tr1 += at;
        lo.tr2 += at;
    }
    const int n_ent = rl.count;
    const int n_steps = n_ent * G;
    const int n_it = (n_steps - group + S - 1) / S;  // the group's share: steps group, group + S, ...
    const int n_loop = (n_steps + S - 1) / S;        // every wave joins every barrier

    // Q and dO tiles and their statistics are copied global -> LDS asynchronously, one tile ahead, into the buffer the
    // previous tile has just vacated; rows past the end of the buffer re-read the last token and are masked.
    const uint32_t row_bytes = static_cast<uint32_t>(Hq) * kRB;
    struct Lane { uint32_t off[kOps]; };
    auto lane_rows = [&](int last_row) {
        Lane d;
#pragma unroll
        for (int i = 0; i < kOps; ++i) {
            const int row = kRows * w + 8 * i + (l >> 3);
            d.off[i] = static_cast<uint32_t>(min(row, last_row)) * row_bytes + (((l & 7) ^ row_swizzle<64>(row)) << 4);
        }
        return d;
    };
    const Lane dml = lane_rows(63);
    const char *cp_q = nullptr, *cp_g = nullptr;  // first Q and dO row of the tile being copied
    const float* cp_s = nullptr;                  // this lane's statistic (waves 0, 1 of a group)
    Lane cp_lane = dml;
    auto copy_setup = [&](int ent, int h) {
        const int q0 = (ent >> 2) * 64;
        int rmax = T - 1 - q0;
        const size_t tile_elems = (static_cast<size_t>(q0) * Hq + h) * 64;
        cp_q = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.Q) + tile_elems);
        cp_g = reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.dO) + tile_elems);
        cp_s = (w ? a.delta : a.lse2) + static_cast<size_t>(h) * T + q0 + min(l, rmax);
        cp_lane = dml;
        if (rmax < 63) {
            asm volatile("; clipped tile" : "+s"(rmax));  // keeps the clamped offsets' arithmetic in this branch
            cp_lane = lane_rows(rmax);
        }
    };
    auto copy_piece = [&](auto P, auto BUF) {
        constexpr int p = decltype(P)::value, buf = decltype(BUF)::value;
        const uint32_t at = group * static_cast<uint32_t>(sizeof(smem[0])) + kRows * w * kRB;
        if constexpr (p < kOps) dma16(cp_q, cp_lane.off[p], lds_addr(smem[0][buf]) + at + 1024 * p);
        else if constexpr (p < 2 * kOps) dma16(cp_g, cp_lane.off[p - kOps], lds_addr(smem[0][2 + buf]) + at + 1024 * (p - kOps));
        else if (w < 2) dma4(cp_s, lds_addr(sStat[0][0][buf]) + group * sizeof(sStat[0]) + (w ? sizeof(sStat[0][0]) : 0));  // wave 0: LSE * log2 e, wave 1: -delta
    };
    // q-tiles from the last to the first and the heads innermost: neighbouring k-tiles share Q / dO tiles through L2
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
    constexpr int kAhead = 2, kRing = 4;
    auto tile = [&](auto BUF) {
        constexpr int buf = decltype(BUF)::value;
        dma_wait_barrier<0>();
        const int q0 = (ent >> 2) * 64;
        const bool full = (ent & 3) == PSATTN_TILE_FULL;
        // after the last tile the same tile is copied once more (to the other buffer, which nobody reads)
        if (it + 1 < n_it) {
            if (ph < S) {  // another q-tile
                ent = es.get(pk);
                copy_setup(ent, kvh * G + ph);
            } else {       // same q-tile, S heads on
                cp_q += kRB * S;
                cp_g += kRB * S;
                cp_s += S * T;
            }
            advance(S);
        }
        ++it;
        if (S > 1 && it > n_it) return;  // the other group's last step: nothing is copied behind it
        const char *sQ = smem[0][buf], *sG = smem[0][2 + buf];  // the group's tiles are behind them by what lo holds
        const float *sL = sStat[group][0][buf], *sD = sStat[group][1][buf];
        uint32_t bits = 0xffffffffu;
        if (!full) {
            bits = elem_range_bits(key - q0, tk.key_hi - q0, g);
            if (__builtin_amdgcn_ballot_w64(bits != 0) == 0) {
                static_for<0, kPieces>([&](auto P) { copy_piece(P, std::integral_constant<int, buf ^ 1>{}); });
                return;
            }
        }
        // Per block b of 32 queries: slots 16 b + 0-7 S, dP (alternating), the P / dS arithmetic, slots 16 b + 8-15
        // dV, dK (alternating).  The LDS operand of a slot is requested kAhead slots earlier, across the arithmetic too.
        Frag8 ring[kRing];
        auto request = [&](auto M) {
            constexpr int m = decltype(M)::value;
            if constexpr (m < 32) {
                constexpr int b = m >> 4, j = m & 15;
                if constexpr (j < 8) {
                    constexpr int t = j >> 1;
                    ring[m % kRing].v = ld_rows<t>(((j & 1) ? sG : sQ) + 32 * b * kRB, lo.nat);
                } else {
                    constexpr int half = (j >> 2) & 1, db = (j >> 1) & 1;
                    ring[m % kRing].v = ld_cols<db, half, 64>(((j & 1) ? sQ : sG) + 32 * b * kRB, lo.tr1, lo.tr2);
                }
            }
        };
        static_for<0, kAhead>([&](auto M) { request(M); });
        static_for<0, 2>([&](auto B) {
            constexpr int b = decltype(B)::value;
            f32x16 s, dp;
            // dP starts from -delta, so that dS = P o (dP - delta) is one multiplication
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4 d = *reinterpret_cast<const float4*>(sD + 32 * b + 8 * i4 + 4 * g);
                dp[4 * i4] = d.x; dp[4 * i4 + 1] = d.y; dp[4 * i4 + 2] = d.z; dp[4 * i4 + 3] = d.w;
#pragma unroll
                for (int k = 0; k < 4; ++k) s[4 * i4 + k] = 0.f;
            }
            static_for<0, 8>([&](auto J) {
                constexpr int j = decltype(J)::value, m = 16 * b + j, t = j >> 1;
                request(std::integral_constant<int, m + kAhead>{});
                if constexpr (8 * b + j < kPieces) copy_piece(std::integral_constant<int, 8 * b + j>{}, std::integral_constant<int, buf ^ 1>{});
                if constexpr (j & 1) dp = mfma(ring[m % kRing].v, vf[t].v, dp);
                else s = mfma(ring[m % kRing].v, kf[t].v, s);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (!full) {
                asm volatile("; mask of a PARTIAL tile" ::: "memory");
                static_for<0, 16>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    s[i] = keep_or_neg_inf<16 * b + i>(s[i], bits);
                });
            }
            Operand<64> pb[2], dsb[2];
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4 L = *reinterpret_cast<const float4*>(sL + 32 * b + 8 * i4 + 4 * g);
                const float Ls[4] = {L.x, L.y, L.z, L.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i = 4 * i4 + k;
                    s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c, -Ls[k]));
                    dp[i] *= s[i];
                }
            }
            pb[0] = make_operand<64>(s, 0); pb[1] = make_operand<64>(s, 1);
            dsb[0] = make_operand<64>(dp, 0); dsb[1] = make_operand<64>(dp, 1);
            __builtin_amdgcn_sched_barrier(0);
            static_for<8, 16>([&](auto J) {
                constexpr int j = decltype(J)::value, m = 16 * b + j, half = (j >> 2) & 1, db = (j >> 1) & 1;
                request(std::integral_constant<int, m + kAhead>{});
                if constexpr (j & 1) dk[db] = mfma_parts<64>(ring[m % kRing].v, dsb[half], dk[db]);
                else dv[db] = mfma_parts<64>(ring[m % kRing].v, pb[half], dv[db]);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    // every compiler-tracked load above has retired before the loop starts, so the loop body holds no wait of the
    // compiler's that would also cover copies in flight
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    tk = token_choose(a.meta, begun, found);
    k_rows.operands(kf, l, l_nat);
    v_rows.operands(vf, l, l_nat);
    // in registers before a copy takes their place
#pragma unroll
    for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(kf[t].v), "+v"(vf[t].v)::"memory");
    while (it + 1 < n_loop) {
        tile(std::integral_constant<int, 0>{});
        tile(std::integral_constant<int, 1>{});
    }
    if (it < n_loop) tile(std::integral_constant<int, 0>{});
    // no copy may still be writing to LDS when the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (S > 1) {
        // Group 0 hands its dK to group 1, which hands its dV to group 0; each adds the other's part to its own.
        __syncthreads();  // every wave's reads and copies are done: the tiles' space is free
        char* const mine = &smem[0][0][0] + wg * 8192 + 16 * l;
        const char* const theirs = &smem[0][0][0] + (wg ^ kWaves) * 8192 + 16 * l;
        auto give = [&](const f32x16 (&x)[2]) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                *reinterpret_cast<float4*>(mine + 1024 * i) = make_float4(x[i >> 2][4 * (i & 3)], x[i >> 2][4 * (i & 3) + 1], x[i >> 2][4 * (i & 3) + 2], x[i >> 2][4 * (i & 3) + 3]);
        };
        auto take = [&](f32x16 (&x)[2]) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float4 y = *reinterpret_cast<const float4*>(theirs + 1024 * i);
                x[i >> 2][4 * (i & 3)] += y.x;
                x[i >> 2][4 * (i & 3) + 1] += y.y;
                x[i >> 2][4 * (i & 3) + 2] += y.z;
                x[i >> 2][4 * (i & 3) + 3] += y.w;
            }
        };
        if (group) give(dv); else give(dk);
        __syncthreads();
        if (group) take(dk); else take(dv);
    }
    // sums that are not finite are taken again (psattn_exact.h), before anything is stored: dK and dV may take K's and V's memory
    multiply(dk, a.scale);
    if (S == 1 || group == 0)
        for (AgainGroups n(not_finite_groups(dv), row0, T); n.any(); n.next())
            set_group(dv, n.group(), exact_dkdv<uint16_t, 64, false, -1>(a, kvh, n.row, n.dim()));
    if (S == 1 || group == 1)
        for (AgainGroups n(not_finite_groups(dk), row0, T); n.any(); n.next())
            set_group(dk, n.group(), exact_dkdv<uint16_t, 64, true, -1>(a, kvh, n.row, n.dim()));
    if constexpr (S > 1) __syncthreads();
    // (a split row: the second group's tiles, which nobody uses any more)
    const int lx = opaque(l);
    char* const out = S == 1 ? k_at : &smem[S - 1][0][0] + wg * 32 * kRB;
    const Rows<64> out_rows{out, out + 16 * kRB};
    const size_t out0 = (static_cast<size_t>(row0) * Hkv + kvh) * kRB;
    if (S == 1 || group == 0) {
#pragma unroll
        for (int db = 0; db < 2; ++db) out_rows.put(db, dv[db], 1.f, lx);
        out_rows.copy_out(static_cast<char*>(a.dV) + out0, k_row_bytes, lx, T - row0);
    }
    if (S == 1 || group == 1) {
#pragma unroll
        for (int db = 0; db < 2; ++db) out_rows.put(db, dk[db], 1.f, lx);
        out_rows.copy_out(static_cast<char*>(a.dK) + out0, k_row_bytes, lx, T - row0);
    }
}

}  // namespace

// Which of the two.  A workgroup is a serial chain of as many steps (heads of the group x q-tiles) as its row is long; with
// two workgroups per CU a launch is bound by its longest chain until that falls below half of a CU's share of all steps.
// Splitting halves the chain and costs a few per cent more work (every tile is staged for 64 keys instead of 128) and the
// exchange at the end; the line lies where the longest chain is a CU's share.  Measured, dK/dV alone, unsplit / split, 32 q / 8 kv
// heads: one sample of 2 000 tokens (chain 128, share 34) 266 / 137 us; four of 1 280 (80, 54) 173 / 114; 4 758 tokens (52, 31)
// 116 / 70; eight of 860 (64, 61) 155 / 121; outside the line 24 of 300 (32, 33) 79 / 64, fourteen of 600 (48, 58) 123 / 104;
// 16 / 16 heads, two of 1 600 (26, 22) 68 / 49, outside eight of 500 (10, 13) 32 / 32, 24 of 256 (4, 9) 29 / 33, 24 of 300 (8, 17)
// 41 / 44; 8 / 8 heads, one sample of 40 tokens (chain 1) 8.3 / 8.5, of 180 (3) 12.9 / 10.8.  Rows in groups of four heads would gain
// below the line as well; it keeps the order of sums of the tables there.
constexpr int64_t kCus = 256;

int launch_mfma_dkdv64(const AttnArgs& a, void* stream) {
    const unsigned grid = static_cast<unsigned>(a.meta.n_rows[kGridK]) * a.Hkv;
    if (grid == 0) return 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t chain = static_cast<int64_t>(a.size[kGridK].longest) * (a.Hq / a.Hkv), steps = a.size[kGridK].n_entries * a.Hq;
    if (chain > 0 && chain * kCus >= steps) psattn_dkdv64_bf16_mfma<2><<<2 * grid, 256, 0, s>>>(a);
    else psattn_dkdv64_bf16_mfma<1><<<grid, 256, 0, s>>>(a);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
