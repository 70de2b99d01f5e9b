// bf16 MFMA forward kernel for gfx950; layout and staging helpers are in psattn_mfma_common.h.  Built three times:
// psattn_mfma_fwd.hip and psattn_mfma_fwd3.hip (head_dim 128, two and three workgroups to a CU) and psattn_mfma_fwd64.hip (64).
#pragma once
#include "psattn_mfma_common.h"

namespace psattn {
namespace {
using namespace mma;

// max(a, b, c)
__device__ __forceinline__ float fmax3(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }

// ------------------------------------------------------------------ forward
// grid: as many workgroups as (q-tile of 128 queries, q-head); 4 waves x 32 queries of one head or of four (query_block).
// D = head_dim.  D = 128: 64 KB of LDS and under 256 registers, two workgroups per CU.  D = 64: half of both.
// kLateV (D = 128): 48 KB and 168 registers, three workgroups per CU.  V has one buffer and travels while the scores of its own
// tile are computed, behind a second barrier per tile; the third wave of a SIMD covers that barrier, the softmax arithmetic and
// the rows' way in and out better than two do.  To fit, the operand ring holds three slots instead of four (one slot of look-ahead
// instead of two: 4 % slower), lane offsets are taken again in every tile instead of kept, and a clipped last tile stands for
// the last 64 rows of the buffer (with a mask from its own first key on) instead of keeping clamped offsets.  Raising the waves'
// priority for the second product changes nothing (+-0.5 %).  mfma_fwd_three says where it is the faster one.
template <int D, bool kLateV>
__global__ __launch_bounds__(256, D == 64 || kLateV ? 3 : 2) void psattn_fwd_bf16_mfma(AttnArgs a) {
    constexpr int kRB = kRowBytesOf<D>, kSteps = D / 16, kBlocks = D / 32;  // MFMA steps of a score, 32-wide blocks of an output row
    __shared__ __attribute__((aligned(16))) char sKb[2][64 * kRB];  // double buffered
    __shared__ __attribute__((aligned(16))) char sVb[kLateV ? 1 : 2][64 * kRB];
    fetch_args(a);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, c32 = l & 31, g = l >> 5;
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv;
    const QueryBlock qb = query_block(Hq, Hkv, a.meta.n_rows[kGridQ], w);
    const RowLaunch rl = row_launch<kGridQ>(a.meta, qb.row);  // one scalar load: row, list bounds
    const int kvh = qb.kvh, h = qb.h, row0 = rl.row * 128 + qb.first;
    const int q_row = row0 + c32;
    const bool valid = q_row < T;
    const TokenLoad begun = token_begin(a.meta, q_row);

    const uint16_t* Q = static_cast<const uint16_t*>(a.Q);
    const uint16_t* K = static_cast<const uint16_t*>(a.K) + kvh * D;
    const uint16_t* V = static_cast<const uint16_t*>(a.V) + kvh * D;

    // Q passes through the places of buffer 1 (late V: of the one V buffer) that the wave's own K / V copies take later
    const LaneOffsets lo = lane_offsets<D>(l);
    const uint32_t q_row_bytes = static_cast<uint32_t>(Hq) * kRB;
    const Rows<D> rows1{sKb[1] + 16 * w * kRB, sVb[kLateV ? 0 : 1] + 16 * w * kRB};
    // rotary embedding: the table row of this lane's query, both members of a pair in the same lane
    float4 turn[D == 128 ? 16 : 1];
    Tok4 found = {kPadStart, 0, 0, 0};
    if constexpr (D == 128) if (a.rope) {
        found = token_search(a.meta, q_row);
        const float* row = a.rope + static_cast<size_t>(rope_position(token_choose(a.meta, begun, found), q_row)) * 128;
#pragma unroll
        for (int t = 0; t < 4; ++t) rope_load8(turn + 4 * t, row, 16 * t + 8 * g);
    }
    Frag8 qf[kSteps];
    // (the asynchronous copies move 16-byte groups, on which every tensor has to start; a Q that does not was read as it lies
    // before its rows came by such copies, and still is, straight into the registers)
    const bool straight = D == 128 && (reinterpret_cast<uintptr_t>(a.Q) & 15) != 0;
    if (straight) {
#pragma unroll
        for (int t = 0; t < kSteps; ++t)
            qf[t].u = valid ? *reinterpret_cast<const uint4*>(Q + (static_cast<size_t>(q_row) * Hq + h) * D + 16 * t + 8 * g) : make_uint4(0, 0, 0, 0);
    } else {
        rows1.copy_in(reinterpret_cast<const char*>(Q) + (static_cast<size_t>(min(row0, T - 1)) * Hq + h) * kRB, q_row_bytes, l, min(max(T - 1 - row0, 0), 31));
    }
    f32x16 o[kBlocks];
#pragma unroll
    for (int db = 0; db < kBlocks; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    float m = -INFINITY, lsum = 0.f;
    const float c = a.scale * kLog2e;
    constexpr int kAhead = 2, kRing = kLateV ? 3 : 4;  // measured: 1 and 3 are both slower

    // K / V tiles are copied global -> LDS asynchronously, one tile ahead, into the
    // buffer the previous tile has just vacated; one barrier per tile.
    const uint32_t row_bytes = static_cast<uint32_t>(Hkv) * kRB;
    const char* Kb = reinterpret_cast<const char*>(K);
    const char* Vb = reinterpret_cast<const char*>(V);
    PairCopyOf<D> pc{Kb, Vb, dma_lane<D>(row_bytes, w, l)};
    int cp_last = 63;  // last row that the lanes' offsets are made for
    // late V: K and V are set up and copied one after the other; a clipped tile takes the last 64 rows; the lane's offset in the first piece
    auto late_start = [&](int ent) { return min((ent >> 2) * 64, T - 64); };
    const uint32_t late_lane = pc.lane.off[0];
    auto late_piece = [&](const char* from, char* to, auto P) {
        constexpr int p = decltype(P)::value;
        dma16(from + static_cast<size_t>(4 * p) * row_bytes, opaque(late_lane) ^ (p << 4), lds_addr(to) + 16 * w * kRB + 1024 * p);
    };
    auto copy_setup = [&](int ent) {
        const int k0 = kLateV ? late_start(ent) : (ent >> 2) * 64;
        const size_t at = static_cast<size_t>(k0) * row_bytes;
        pc.a = Kb + at;
        if constexpr (kLateV) return;
        pc.b = Vb + at;
        tile_rows(min(T - 1 - k0, 63), cp_last, [&](int last) { pc.lane = dma_lane<D>(row_bytes, w, opaque(l), last); });
    };
    EntryStream es;
    int ent = rl.first_entry, it = 0, n_ent = rl.count;
    auto first_copy = [&] {
        if (it < n_ent) {
            copy_setup(ent);
            if constexpr (kLateV) static_for<0, kBlocks>([&](auto P) { late_piece(pc.a, sKb[0], P); });
            else static_for<0, 2 * kBlocks>([&](auto P) { pair_copy_piece<decltype(P)::value>(pc, sKb[0], sVb[0], w); });
        }
    };
    if (!qb.together) first_copy();
    if (!(D == 128 && a.rope)) found = token_search(a.meta, q_row);
    es.init<kGridQ>(a.meta, rl, 1, l);
    Tok4 tk = found;
    if (qb.together) {
        tk = token_choose(a.meta, begun, found);
        // waves that share their queries leave out the tiles at both ends of the list that are there for the q-tile's others (at
        // the back, below, of lists that one batch of the reader holds)
        while (it < n_ent && !reads_tile(ent, row0, tk))
            if (++it < n_ent) ent = es.get(it);
        first_copy();
    }
    if (qb.together && n_ent <= 64)
        while (it + 1 < n_ent && !reads_tile(es.peek(n_ent - 1), row0, tk)) --n_ent;
    const int n_tiles = n_ent - it;
    // One tile.  The buffer index is a compile-time constant (the loop below is unrolled
    // by two), so every LDS address is a lane constant plus an immediate offset.
    auto tile = [&](auto BUF) {
        constexpr int buf = decltype(BUF)::value;
        // this wave's copies of tile `it` have landed; after the barrier every wave's
        // have, and every wave has left the other buffer
        dma_wait_barrier<0>();
        const int k0 = (ent >> 2) * 64, k_first = kLateV ? late_start(ent) : k0;
        bool full = (ent & 3) == PSATTN_TILE_FULL;
        if constexpr (kLateV) pc.b = Vb + static_cast<size_t>(k_first) * row_bytes;
        auto piece = [&](auto P) {  // V of this tile, then K of the next
            constexpr int p = decltype(P)::value;
            if constexpr (!kLateV) pair_copy_piece<p>(pc, sKb[buf ^ 1], sVb[(buf ^ 1) % (sizeof(sVb) / sizeof(sVb[0]))], w);
            else if constexpr (p < kBlocks) late_piece(pc.b, sVb[0], P);
            else late_piece(pc.a, sKb[buf ^ 1], std::integral_constant<int, p - kBlocks>{});
        };
        // The next tile's copy is issued piece by piece, on every other slot of the S phase.  After
        // the last tile the same tile is copied once more (to the other buffer, which nobody
        // reads), so the slots need no branch.
        if (it + 1 < n_ent) {
            ent = es.get(it + 1);
            copy_setup(ent);
        }
        ++it;
        // PARTIAL tile: this lane's allowed elements as a bit mask (the query reads keys
        // [tk.s, q_row] except [hole_lo, hole_hi)).  A wave none of whose 32 queries reads any
        // key of the tile only issues its share of the copy and leaves the SIMD to the other
        // workgroup's wave (two of the four waves on the second tile of every causal diagonal).
        uint32_t bits = 0xffffffffu;
        if (!full) {
            bits = elem_range_bits(max(tk.s, k0) - k_first, q_row + 1 - k_first, g) & ~elem_range_bits(tk.hole_lo - k_first, tk.hole_hi - k_first, g);
            if (__builtin_amdgcn_ballot_w64(bits != 0) == 0) {
                static_for<0, 2 * kBlocks>([&](auto P) { piece(P); });
                if constexpr (kLateV) dma_wait_barrier<kBlocks>();  // the other waves' second barrier
                return;
            }
            full = __builtin_amdgcn_ballot_w64(bits != 0xffffffffu) == 0;  // for these 32 queries
        }
        const char* sK = sKb[buf];
        const char* sV = sVb[kLateV ? 0 : buf];
        // 2 kS MFMA slots per tile: 0 .. kS - 1 S^T = K Q^T (rows = keys, column = this lane's
        // query), kS .. 2 kS - 1 O^T += V^T P^T.  The LDS operand of slot m is requested kAhead
        // slots earlier into a register ring.
        constexpr int kS = 2 * kSteps;
        Frag8 ring[kRing];
        const int nat = kLateV ? opaque(lo.nat) : lo.nat;  // what it is XORed with is not kept across tiles
        auto request = [&](auto M) {
            constexpr int m = decltype(M)::value;
            if constexpr (m < kS) {
                constexpr int t = m >> 1, kb = m & 1;
                ring[m % kRing].v = ld_rows<t>(sK + kb * 32 * kRB, nat);
            } else if constexpr (m < 2 * kS) {
                constexpr int j = m - kS, kb = j / (2 * kBlocks), half = (j / kBlocks) & 1, db = j % kBlocks;
                ring[m % kRing].v = ld_cols<db, half, D>(sV + 32 * kb * kRB, lo.tr1, lo.tr2);
            }
        };
        f32x16 s[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
        static_for<0, kAhead>([&](auto M) { request(M); });
        static_for<0, kS>([&](auto M) {
            constexpr int m = decltype(M)::value, t = m >> 1, kb = m & 1;
            if constexpr (!kLateV || m + kAhead < kS) request(std::integral_constant<int, m + kAhead>{});
            if constexpr ((m & 1) == 0) piece(std::integral_constant<int, m / 2>{});  // every other slot: see PairCopyOf
            s[kb] = mfma(ring[m % kRing].v, qf[t].v, s[kb]);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!full) {
            asm volatile("; mask of a PARTIAL tile" ::: "memory");
            static_for<0, 32>([&](auto E) {
                constexpr int e = decltype(E)::value;
                s[e >> 4][e & 15] = keep_or_neg_inf<e>(s[e >> 4][e & 15], bits);
            });
        }
        // The maxima are ordinary compiled code (head_dim 128 is built with -fno-honor-nans, so that
        // fmaxf(fmaxf(a, b), c) becomes one v_max3_f32 without NaN-quieting instructions): the compiler
        // sees a vector-ALU reader of MFMA results and places the wait states such a reader needs.  (An
        // inline-assembly maximum is not seen as one, and then read scores of the previous tile now and then.)
        // four independent chains each for the maximum and (below) the sum
        float mxp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) mxp[r] = fmax3(s[0][r], s[1][r], s[0][r + 4]);
#pragma unroll
        for (int r = 0; r < 4; ++r) mxp[r] = fmax3(mxp[r], s[1][r + 4], s[0][r + 8]);
#pragma unroll
        for (int r = 0; r < 4; ++r) mxp[r] = fmax3(mxp[r], s[1][r + 8], s[0][r + 12]);
#pragma unroll
        for (int r = 0; r < 4; ++r) mxp[r] = fmax3(mxp[r], s[1][r + 12], mxp[r]);
        float mx = fmax3(mxp[0], mxp[1], fmax3(mxp[2], mxp[3], mxp[3]));
        const Halves mh = halves(mx);
        mx = fmax3(mh.lo, mh.hi, mh.hi);
        // Exact running maximum; O and l are rescaled only in tiles where some row's maximum
        // moves (wave ballot).  Letting the reference lag behind the maximum was measured
        // both ways: a fixed lag of 2^8 saves 5 % of this kernel but the largest probability of
        // a row is then no longer exactly 1 and its bf16 rounding shows in O on short rows
        // (0.012 against a bar of 1e-2); a lag bounded by the row's sum so far keeps the
        // accuracy but saves nothing measurable.
        const float m_new = fmaxf(m, mx * c);
        if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
            asm volatile("; rescale" ::: "memory");
            const float m_to = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m - m_to);  // m = -inf: 0 (nothing accumulated yet)
            lsum *= alpha;
#pragma unroll
            for (int db = 0; db < kBlocks; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
            m = m_new;
        }
        const float m_use = m == -INFINITY ? 0.f : m;
        float ps[4] = {0.f, 0.f, 0.f, 0.f};
        Operand<D> pb[2][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s[kb][i] = __builtin_amdgcn_exp2f(fmaf(s[kb][i], c, -m_use));
                ps[i & 3] += s[kb][i];
            }
            pb[kb][0] = make_operand<D>(s[kb], 0);
            pb[kb][1] = make_operand<D>(s[kb], 1);
        }
        const float psum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
        lsum += psum;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kLateV) {
            dma_wait_barrier<kBlocks>();  // every wave's V of this tile has landed, the next K may be on its way
            static_for<0, kAhead>([&](auto M) { request(std::integral_constant<int, kS + decltype(M)::value>{}); });
        }
        static_for<kS, 2 * kS>([&](auto M) {
            constexpr int m_ = decltype(M)::value, j = m_ - kS, kb = j / (2 * kBlocks), half = (j / kBlocks) & 1, db = j % kBlocks;
            request(std::integral_constant<int, m_ + kAhead>{});
            o[db] = mfma_parts<D>(ring[m_ % kRing].v, pb[kb][half], o[db]);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Q fragments are in registers before the loop starts, so the loop body holds no wait
    // on a compiler-tracked load (such a wait would also cover the copies in flight)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    tk = token_choose(a.meta, begun, found);
    if (!straight) rows1.operands(qf, l, lo.nat);
    if constexpr (D == 128) if (a.rope) {
        // the rotated row is also saved for the backward, which streams Q tiles straight into LDS and cannot rotate them on the way
#pragma unroll
        for (int t = 0; t < 4; ++t) rope_frag8(qf[t], qf[t + 4], turn + 4 * t);
        if (a.Qr) {
            rows1.put_operands(qf, l, lo.nat);
            rows1.copy_out(static_cast<char*>(a.Qr) + (static_cast<size_t>(row0) * Hq + h) * kRB, q_row_bytes, l, T - row0);
        }
    }
    // ... and the place in LDS is done with before the second tile's copies take it
#pragma unroll
    for (int t = 0; t < kSteps; ++t) asm volatile("" : "+v"(qf[t].v)::"memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    if constexpr (kLateV) {  // with the last tile by itself three registers are spilled
        while (it < n_ent) {
            tile(std::integral_constant<int, 0>{});
            if (it >= n_ent) break;
            tile(std::integral_constant<int, 1>{});
        }
    } else {  // one sample of 900 tokens 21.9 us, of 500 15.1; in the other form 22.5 and 15.4
        while (it + 1 < n_ent) {
            tile(std::integral_constant<int, 0>{});
            tile(std::integral_constant<int, 1>{});
        }
        if (it < n_ent) tile(std::integral_constant<int, 0>{});
    }
    // no copy may still be writing to LDS when the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const Halves lh = halves(lsum);
    const float l_tot = lh.lo + lh.hi;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    multiply(o, inv);
    if constexpr (D == 64) {
        // sums that are not finite, and rows without a sum, are taken again (psattn_exact.h)
        uint32_t again = not_finite_groups(o);
        if (!(l_tot > 0.f) && tk.s != kPadStart) again = 0xff;
        for (AgainGroups n(again, row0, T); n.any(); n.next()) set_group(o, n.group(), exact_o<uint16_t, D>(a, h, n.row, n.dim()));
    }
    // Four heads on the same queries leave through LDS, one head straight.  Measured, straight / through LDS, in us: four heads, 32 / 8,
    // moderate samples of 1 000, 16 384 tokens 165.5 / 161.8, 8 334 tokens 93.5 / 92.8, four samples of 940 43.5 / 43.1, head_dim 64,
    // ten of 256 13.4 / 13.1; one head, one sample of 180 tokens 7.6 / 7.8, of 221 8.8 / 9.1, 500 tokens 10.5 / 10.7, 16 / 16 heads, eight
    // samples of 560 22.6 / 23.1, 28 / 4 heads, two of 1 600 46.6 / 47.1, head_dim 64, 16 / 16 heads, 24 samples of 256 16.0 / 16.4.
    const int lx = opaque(l);
    if (qb.together) {  // the buffer that the last tile was not in; late V: both of K, whose last reader is ahead of the last barrier
        const Rows<D> rows{sKb[n_tiles & 1] + 16 * w * kRB, kLateV ? sKb[~n_tiles & 1] + 16 * w * kRB : sVb[(n_tiles & 1) % (sizeof(sVb) / sizeof(sVb[0]))] + 16 * w * kRB};
#pragma unroll
        for (int db = 0; db < kBlocks; ++db) rows.put(db, o[db], 1.f, lx);
        rows.copy_out(static_cast<char*>(a.Oout) + (static_cast<size_t>(row0) * Hq + h) * kRB, q_row_bytes, lx, T - row0);
    } else {
        uint16_t* orow = static_cast<uint16_t*>(a.Oout) + (static_cast<size_t>(row0) * Hq + h) * D;
#pragma unroll
        for (int db = 0; db < kBlocks; ++db) store_block(orow, static_cast<size_t>(Hq) * D, T - row0, db, o[db], 1.f, lx);
    }
    if (lx < 32 && row0 + lx < T)
        a.LSEout[static_cast<size_t>(h) * T + row0 + lx] = l_tot > 0.f ? m * kLn2 + __logf(l_tot) : -INFINITY;
}

}  // namespace
}  // namespace psattn
