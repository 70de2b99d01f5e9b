// bf16 MFMA dK/dV kernel for gfx950, head_dim 64; layout and staging helpers are in psattn_mfma_common.h.
//
// grid: one workgroup per (k-tile of 128 keys, kv-head); 4 waves x 32 keys.  The walk is that of the head_dim 128
// kernel (the G query heads of the group, and for each the q-tiles of 64 queries that can read the keys, so that the
// prompt's keys collect the contributions of prompt, chosen and rejected queries in one place, without atomics), but
// at half the head dimension dK, dV and the K / V fragments of a wave take 96 registers instead of 192: the whole
// kernel fits 256, the compiler can manage it, and two waves share a SIMD, so that one wave's softmax arithmetic
// meets the other's MFMAs.  What bounds it is that arithmetic: per 64 x 32 scores a wave issues 32 MFMAs (1 024
// cycles of the matrix pipeline) and about 300 vector instructions.  Measured on a step of 8 samples, 4 758 tokens,
// 32 q / 8 kv heads: forward + dQ + dK/dV 14.9 ms on the one-thread-per-row kernels, 0.15 ms on these.
#include "psattn_mfma_common.h"

namespace psattn {
namespace {
using namespace mma;

constexpr int kRB = kRowBytesOf<64>;

__global__ __launch_bounds__(256, 2) void psattn_dkdv64_bf16_mfma(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) char sQ[2][64 * kRB];  // double buffered
    __shared__ __attribute__((aligned(16))) char sG[2][64 * kRB];  // dO
    __shared__ __attribute__((aligned(16))) float sL[2][64];       // LSE * log2(e)
    __shared__ __attribute__((aligned(16))) float sD[2][64];       // -delta
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, c32 = l & 31, g = l >> 5;
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv, G = Hq / Hkv;
    const DeviceCsr& csr = a.meta.bwd;
    const RowLaunch rl = csr.launch[blockIdx.x / Hkv];  // one scalar load: row, list bounds, first entry
    const int kvh = blockIdx.x % Hkv, kt = rl.row;
    const int key = kt * 128 + 32 * w + c32;
    const bool kvalid = key < T;
    const int key_hi = kvalid ? a.meta.tok[key].key_hi : 0;  // queries [key, key_hi) read this key
    const size_t koff = (static_cast<size_t>(key) * Hkv + kvh) * 64;

    Frag8 kf[4], vf[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        kf[t].u = kvalid ? *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.K) + koff + 16 * t + 8 * g) : make_uint4(0, 0, 0, 0);
        vf[t].u = kvalid ? *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.V) + koff + 16 * t + 8 * g) : make_uint4(0, 0, 0, 0);
    }
    f32x16 dk[2], dv[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) { dk[db][i] = 0.f; dv[db][i] = 0.f; }

    const float c = a.scale * kLog2e;
    const LaneOffsets lo = lane_offsets<64>(l);
    const int e0 = rl.begin, n_ent = rl.count;
    const int n_it = n_ent * G;

    // Q and dO tiles and their statistics are copied global -> LDS asynchronously, one tile ahead, into the buffer the
    // previous tile has just vacated; rows past the end of the buffer re-read the last token and are masked.
    const uint32_t row_bytes = static_cast<uint32_t>(Hq) * kRB;
    const DmaLaneOf<64> dml = dma_lane<64>(row_bytes, w, l);
    PairCopyOf<64> pc;
    const float* cp_s = nullptr;  // this lane's statistic (waves 0, 1)
    auto copy_setup = [&](int ent, int h) {
        const int q0 = (ent >> 2) * 64, rmax = T - 1 - q0;
        const size_t tile_elems = (static_cast<size_t>(q0) * Hq + h) * 64;
        pair_copy_setup(pc, reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.Q) + tile_elems),
                        reinterpret_cast<const char*>(static_cast<const uint16_t*>(a.dO) + tile_elems), row_bytes, rmax, dml, w, l);
        cp_s = (w ? a.delta : a.lse2) + static_cast<size_t>(h) * T + q0 + min(l, rmax);
    };
    auto copy_piece = [&](auto P, auto BUF) {
        constexpr int p = decltype(P)::value, buf = decltype(BUF)::value;
        if constexpr (p < 4) pair_copy_piece<p>(pc, sQ[buf], sG[buf], w);
        else if (w < 2) dma4(cp_s, lds_addr(w ? sD[buf] : sL[buf]));  // wave 0: LSE * log2 e, wave 1: -delta
    };
    // q-tiles from the last to the first and the heads innermost: neighbouring k-tiles share Q / dO tiles through L2
    EntryStream es;
    es.init(csr.entry, e0 + n_ent - 1, -1, n_ent, l);
    int pk = 0, ph = 0;  // walk position and head (within the group) of the next tile
    int ent = 0, it = 0;
    if (n_it > 0) {
        ent = rl.first_entry;
        copy_setup(ent, kvh * G);
        static_for<0, 5>([&](auto P) { copy_piece(P, std::integral_constant<int, 0>{}); });
        if (++ph == G) { ph = 0; ++pk; }
    }
    constexpr int kAhead = 2, kRing = 4;
    auto tile = [&](auto BUF) {
        constexpr int buf = decltype(BUF)::value;
        dma_wait_barrier<0>();
        const int q0 = (ent >> 2) * 64;
        const bool full = (ent & 3) == PSATTN_TILE_FULL;
        // after the last tile the same tile is copied once more (to the other buffer, which nobody reads)
        if (it + 1 < n_it) {
            if (ph == 0) {
                ent = es.get(pk);
                copy_setup(ent, kvh * G);
            } else {  // same q-tile, next head of the group
                pc.a += kRB;
                pc.b += kRB;
                cp_s += T;
            }
            if (++ph == G) { ph = 0; ++pk; }
        }
        ++it;
        uint32_t bits = 0xffffffffu;
        if (!full) {
            bits = elem_range_bits(key - q0, key_hi - q0, g);
            if (__builtin_amdgcn_ballot_w64(bits != 0) == 0) {
                static_for<0, 5>([&](auto P) { copy_piece(P, std::integral_constant<int, buf ^ 1>{}); });
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
                    ring[m % kRing].v = ld_rows<t>(((j & 1) ? sG[buf] : sQ[buf]) + 32 * b * kRB, lo.nat);
                } else {
                    constexpr int half = (j >> 2) & 1, db = (j >> 1) & 1;
                    ring[m % kRing].v = ld_cols<db, half, 64>(((j & 1) ? sQ[buf] : sG[buf]) + 32 * b * kRB, lo.tr1, lo.tr2);
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
                const float4 d = *reinterpret_cast<const float4*>(sD[buf] + 32 * b + 8 * i4 + 4 * g);
                dp[4 * i4] = d.x; dp[4 * i4 + 1] = d.y; dp[4 * i4 + 2] = d.z; dp[4 * i4 + 3] = d.w;
#pragma unroll
                for (int k = 0; k < 4; ++k) s[4 * i4 + k] = 0.f;
            }
            static_for<0, 8>([&](auto J) {
                constexpr int j = decltype(J)::value, m = 16 * b + j, t = j >> 1;
                request(std::integral_constant<int, m + kAhead>{});
                if constexpr (b == 0 && j < 5) copy_piece(J, std::integral_constant<int, buf ^ 1>{});
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
            bf16x8 pb[2], dsb[2];
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4 L = *reinterpret_cast<const float4*>(sL[buf] + 32 * b + 8 * i4 + 4 * g);
                const float Ls[4] = {L.x, L.y, L.z, L.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i = 4 * i4 + k;
                    s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], c, -Ls[k]));
                    dp[i] *= s[i];
                }
            }
            pb[0] = pack8(s, 0); pb[1] = pack8(s, 1);
            dsb[0] = pack8(dp, 0); dsb[1] = pack8(dp, 1);
            __builtin_amdgcn_sched_barrier(0);
            static_for<8, 16>([&](auto J) {
                constexpr int j = decltype(J)::value, m = 16 * b + j, half = (j >> 2) & 1, db = (j >> 1) & 1;
                request(std::integral_constant<int, m + kAhead>{});
                if constexpr (j & 1) dk[db] = mfma(ring[m % kRing].v, dsb[half], dk[db]);
                else dv[db] = mfma(ring[m % kRing].v, pb[half], dv[db]);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    // every compiler-tracked load above has retired before the loop starts, so the loop body holds no wait of the
    // compiler's that would also cover copies in flight
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    while (it + 1 < n_it) {
        tile(std::integral_constant<int, 0>{});
        tile(std::integral_constant<int, 1>{});
    }
    if (it < n_it) tile(std::integral_constant<int, 0>{});
    // no copy may still be writing to LDS when the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int row0 = kt * 128 + 32 * w;
    const size_t out0 = (static_cast<size_t>(row0) * Hkv + kvh) * 64, row_elems = static_cast<size_t>(Hkv) * 64;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
        store_block(static_cast<uint16_t*>(a.dV) + out0, row_elems, T - row0, db, dv[db], 1.f, l);
        store_block(static_cast<uint16_t*>(a.dK) + out0, row_elems, T - row0, db, dk[db], a.scale, l);
    }
}

}  // namespace

int launch_mfma_dkdv64(const AttnArgs& a, void* stream) {
    const unsigned grid = static_cast<unsigned>(a.meta.bwd.n_rows) * a.Hkv;
    if (grid == 0) return 0;
    psattn_dkdv64_bf16_mfma<<<grid, 256, 0, static_cast<hipStream_t>(stream)>>>(a);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
