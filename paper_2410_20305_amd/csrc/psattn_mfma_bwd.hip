// bf16 MFMA backward (dQ; dK/dV) kernels for gfx950; layout and staging helpers are in psattn_mfma_common.h.
#include "psattn_mfma_common.h"

namespace psattn {
namespace {
using namespace mma;

// ------------------------------------------------------------------ dQ (q-major)
// D = head_dim.  D = 128: 64 KB of LDS and under 256 registers, two workgroups per CU.  D = 64: half of both.
template <int D>
__global__ __launch_bounds__(256, D == 128 ? 2 : 3) void psattn_dq_bf16_mfma(AttnArgs a) {
    constexpr int kRB = kRowBytesOf<D>, kSteps = D / 16, kBlocks = D / 32;  // MFMA steps of a score, 32-wide blocks of a dQ row
    __shared__ __attribute__((aligned(16))) char sKb[2][64 * kRB];  // double buffered
    __shared__ __attribute__((aligned(16))) char sVb[2][64 * kRB];
    fetch_args(a);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, c32 = l & 31, g = l >> 5;
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv;
    const QueryBlock qb = query_block(Hq, Hkv, a.meta.n_rows[kGridQ], w);
    const RowLaunch rl = row_launch<kGridQ>(a.meta, qb.row);  // one scalar load: row, list bounds
    const int kvh = qb.kvh, h = qb.h, row0 = rl.row * 128 + qb.first;
    const int q_row = row0 + c32;
    const bool valid = q_row < T;
    const TokenLoad begun = token_begin(a.meta, q_row);

    const uint16_t* K = static_cast<const uint16_t*>(a.K) + kvh * D;
    const uint16_t* V = static_cast<const uint16_t*>(a.V) + kvh * D;
    // dO and Q pass through the places that the wave's own K / V copies take later
    const LaneOffsets lo = lane_offsets<D>(l);
    const uint32_t q_row_bytes = static_cast<uint32_t>(Hq) * kRB;
    const int last_row = min(max(T - 1 - row0, 0), 31);
    const size_t at0 = (static_cast<size_t>(min(row0, T - 1)) * Hq + h) * kRB;
    const Rows<D> rows0{sKb[0] + 16 * w * kRB, sVb[0] + 16 * w * kRB}, rows1{sKb[1] + 16 * w * kRB, sVb[1] + 16 * w * kRB};
    u32x4 orow[kSteps];
#pragma unroll
    for (int t = 0; t < kSteps; ++t) orow[t] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.O) + at0 + Rows<D>::lane_off(t, q_row_bytes, l, last_row));
    rows0.copy_in(static_cast<const char*>(a.dO) + at0, q_row_bytes, l, last_row);
    rows1.copy_in(static_cast<const char*>(a.Q) + at0, q_row_bytes, l, last_row);
    const float lse_row = valid ? a.LSE[static_cast<size_t>(h) * T + q_row] : -INFINITY;
    const Tok4 found = token_search(a.meta, q_row);
    EntryStream es;
    es.init<kGridQ>(a.meta, rl, 1, l);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const Tok4 tk = token_choose(a.meta, begun, found);
    // Rows without keys (padding) have LSE = -inf.  Their scores are masked to -inf below;
    // with +inf here exp2(score - lse2) is 0 for them instead of exp2(-inf + inf).  (A row with keys has LSE = -inf only
    // where its scores are not numbers; head_dim 64 passes that on to whatever reads the row.)
    const bool no_keys = D == 64 ? tk.s == kPadStart : lse_row == -INFINITY;
    const float lse2 = no_keys ? INFINITY : lse_row * kLog2e;
    Frag8 qf[kSteps], gf[kSteps];
    rows0.operands(gf, l, lo.nat);
    rows1.operands(qf, l, lo.nat);
    // they are in registers before the first K / V tile takes the place of dO, and O that of Q
#pragma unroll
    for (int t = 0; t < kSteps; ++t) asm volatile("" : "+v"(qf[t].v), "+v"(gf[t].v)::"memory");
    Frag8 of[kSteps];
    static_for<0, kSteps>([&](auto P) { rows1.template put_chunk<decltype(P)::value>(orow[decltype(P)::value], l); });
    lds_exchange();
    rows1.operands(of, l, lo.nat);
    // K / V tiles are copied global -> LDS asynchronously, one tile ahead, into the
    // buffer the previous tile has just vacated; one barrier per tile.
    const uint32_t row_bytes = static_cast<uint32_t>(Hkv) * kRB;
    PairCopyOf<D> pc{reinterpret_cast<const char*>(K), reinterpret_cast<const char*>(V), dma_lane<D>(row_bytes, w, l)};
    int cp_last = 63;  // last row that the lanes' offsets are made for
    auto copy_setup = [&](int ent) {
        const int k0 = (ent >> 2) * 64;
        const size_t at = static_cast<size_t>(k0) * row_bytes;
        tile_rows(min(T - 1 - k0, 63), cp_last, [&](int last) { pc.lane = dma_lane<D>(row_bytes, w, opaque(l), last); });
        pc.a = reinterpret_cast<const char*>(K) + at;
        pc.b = reinterpret_cast<const char*>(V) + at;
    };
    int ent = rl.first_entry, it = 0, n_ent = rl.count;
    // waves that share their queries leave out the tiles at both ends of the list that are there for the q-tile's others (at
    // the back, below, of lists that one batch of the reader holds)
    if (qb.together)
        while (it < n_ent && !reads_tile(ent, row0, tk))
            if (++it < n_ent) ent = es.get(it);
    if (it < n_ent) {
        copy_setup(ent);
        static_for<0, 2 * kBlocks>([&](auto P) { pair_copy_piece<decltype(P)::value>(pc, sKb[0], sVb[0], w); });
    }
    // delta = rowsum(dO o O): this lane holds half of both rows; the result also goes to the workspace for the dK/dV pass that
    // follows.  Each half is one chain of sums, head dims ascending, while the first tile is on its way.
    float dl = 0.f;
#pragma unroll
    for (int t = 0; t < kSteps; ++t) {
        const uint32_t ow[4] = {of[t].u.x, of[t].u.y, of[t].u.z, of[t].u.w};
        const uint32_t gw[4] = {gf[t].u.x, gf[t].u.y, gf[t].u.z, gf[t].u.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            dl = fmaf(__uint_as_float(ow[j] << 16), __uint_as_float(gw[j] << 16), dl);
            dl = fmaf(__uint_as_float(ow[j] & 0xffff0000u), __uint_as_float(gw[j] & 0xffff0000u), dl);
        }
    }
    const Halves dh = halves(dl);
    dl = dh.lo + dh.hi;
    asm volatile("" : "+v"(dl)::"memory");  // ... and O is done with before the second tile's copies take its place
    if (valid && g == 0) {
        a.delta[static_cast<size_t>(h) * T + q_row] = -dl;  // the dK/dV kernel starts its dP accumulators from -delta
        a.lse2[static_cast<size_t>(h) * T + q_row] = lse2;
    }
    const float c = a.scale * kLog2e;

    f32x16 dq[kBlocks];
#pragma unroll
    for (int db = 0; db < kBlocks; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;

    // head_dim 128: dP starts from -delta, which stands in sixteen registers that the first MFMA of a block adds to, so that
    // dS = P o (dP - delta) is one multiplication (at 64, within 168 registers, they would be spilled)
    f32x16 minus_delta;
#pragma unroll
    for (int i = 0; i < 16; ++i) minus_delta[i] = -dl;
    if (qb.together && n_ent <= 64)
        while (it + 1 < n_ent && !reads_tile(es.peek(n_ent - 1), row0, tk)) --n_ent;
    const int n_tiles = n_ent - it;
    constexpr int kAhead = 2, kRing = 4;  // measured: 1 and 3 are both slower
    // One tile = 2 kB MFMA slots, per block kb of 32 keys:
    //   slots kB kb + 0 .. kS - 1   S^T = K Q^T and dP^T = V dO^T (alternating)
    //   (dS arithmetic of the block)
    //   slots kB kb + kS .. kB - 1  dQ^T += K^T dS^T
    // The LDS operand of slot m is requested kAhead slots earlier into a register ring,
    // across the arithmetic too.  Two workgroups share a CU: the other wave of the SIMD
    // fills the gaps.  The buffer index is a compile-time constant (the loop below is
    // unrolled by two), so every LDS address is a lane constant plus an immediate offset.
    // Only PARTIAL tiles (full == false) run the mask arithmetic.
    constexpr int kS = 2 * kSteps, kB = kS + 2 * kBlocks;
    auto tile = [&](auto BUF, int k0, bool full) {
        constexpr int buf = decltype(BUF)::value;
        // PARTIAL tile: this lane's allowed elements as a bit mask (the query reads keys
        // [tk.s, q_row] except [hole_lo, hole_hi)).  A wave none of whose 32 queries reads any
        // key of the tile only issues its share of the copy and leaves the SIMD to the other
        // workgroup's wave.
        uint32_t bits = 0xffffffffu;
        // skip32[kb]: none of the wave's 32 queries reads any of the 32 keys of block kb (PARTIAL tiles
        // only): the block's kB MFMAs and its arithmetic are left out
        bool skip32[2] = {false, false};
        if (!full) {
            bits = elem_range_bits(tk.s - k0, q_row + 1 - k0, g) & ~elem_range_bits(tk.hole_lo - k0, tk.hole_hi - k0, g);
            skip32[0] = __builtin_amdgcn_ballot_w64((bits & 0xffffu) != 0) == 0;
            skip32[1] = __builtin_amdgcn_ballot_w64((bits >> 16) != 0) == 0;
            if (skip32[0]) {  // the next tile's copy rides on the first block's slots: issue it here instead
                static_for<0, 2 * kBlocks>([&](auto P) { pair_copy_piece<decltype(P)::value>(pc, sKb[buf ^ 1], sVb[buf ^ 1], w); });
                if (skip32[1]) return;
            }
            full = __builtin_amdgcn_ballot_w64(bits != 0xffffffffu) == 0;  // for these 32 queries
        }
        const char* sK = sKb[buf];
        const char* sV = sVb[buf];
        Frag8 ring[kRing];
        auto request = [&](auto M) {
            constexpr int m = decltype(M)::value;
            if constexpr (m < 2 * kB) {
                constexpr int kb = m / kB, j = m % kB;
                if constexpr (j < kS) {
                    constexpr int t = j >> 1;
                    ring[m % kRing].v = ld_rows<t>(((j & 1) ? sV : sK) + kb * 32 * kRB, lo.nat);
                } else {
                    constexpr int half = (j - kS) / kBlocks, db = (j - kS) % kBlocks;
                    ring[m % kRing].v = ld_cols<db, half, D>(sK + 32 * kb * kRB, lo.tr1, lo.tr2);
                }
            }
        };
        static_for<0, 2>([&](auto KB) {
            constexpr int kb = decltype(KB)::value;
            if (skip32[kb]) return;
            // the first operands of a block are requested by the block before it, unless there is none
            if (kb == 0 || skip32[0]) static_for<0, kAhead>([&](auto M) { request(std::integral_constant<int, kB * kb + decltype(M)::value>{}); });
            f32x16 s, dp;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = 0.f;
            if constexpr (D == 128) dp = minus_delta;
            else {
#pragma unroll
                for (int i = 0; i < 16; ++i) dp[i] = 0.f;
            }
            static_for<0, kS>([&](auto J) {
                constexpr int j = decltype(J)::value, m = kB * kb + j, t = j >> 1;
                request(std::integral_constant<int, m + kAhead>{});
                if constexpr (m < kS && (m & 1) == 0) pair_copy_piece<m / 2>(pc, sKb[buf ^ 1], sVb[buf ^ 1], w);  // every other slot: see PairCopyOf
                if constexpr (j & 1) dp = mfma(ring[m % kRing].v, gf[t].v, dp);
                else s = mfma(ring[m % kRing].v, qf[t].v, s);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (!full) {
                asm volatile("; mask of a PARTIAL tile" ::: "memory");
                // masked scores become -inf, so p = 0 below
                static_for<0, 16>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    s[i] = keep_or_neg_inf<16 * kb + i>(s[i], bits);
                });
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[i], c, -lse2));
                s[i] = p * (D == 128 ? dp[i] : dp[i] - dl);  // dS^T
            }
            Operand<D> dsb[2];
            dsb[0] = make_operand<D>(s, 0);
            dsb[1] = make_operand<D>(s, 1);
            __builtin_amdgcn_sched_barrier(0);
            static_for<kS, kB>([&](auto J) {
                constexpr int j = decltype(J)::value, m = kB * kb + j, half = (j - kS) / kBlocks, db = (j - kS) % kBlocks;
                request(std::integral_constant<int, m + kAhead>{});
                dq[db] = mfma_parts<D>(ring[m % kRing].v, dsb[half], dq[db]);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    auto step = [&](auto BUF) {
        constexpr int buf = decltype(BUF)::value;
        // this wave's copies of tile `it` have landed; after the barrier every wave's
        // have, and every wave has left the other buffer
        dma_wait_barrier<0>();
        const int k0 = (ent >> 2) * 64;
        const bool full = (ent & 3) == PSATTN_TILE_FULL;
        // The next tile's copy is issued piece by piece, on every other slot of the first sixteen.
        // After the last tile the same tile is copied once more (to the other buffer, which
        // nobody reads), so the slots need no branch.
        if (it + 1 < n_ent) {
            ent = es.get(it + 1);
            copy_setup(ent);
        }
        ++it;
        tile(BUF, k0, full);
    };
    // every compiler-tracked load and store above has retired before the loop starts, so
    // the loop body holds no wait of the compiler's that would also cover copies in flight
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    while (it + 1 < n_ent) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
    if (it < n_ent) step(std::integral_constant<int, 0>{});
    // no copy may still be writing to LDS when the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (D == 128) if (a.rope) {
        // Q arrived rotated: what was accumulated is the gradient w.r.t. the rotated query; turning
        // it back by the same angles gives the gradient w.r.t. the unrotated one.  Accumulator
        // element i of block db is head dim 32 db + 8 (i / 4) + 4 g + i % 4; its partner sits in
        // block db + 2 at the same i.
        const float* trow = a.rope + static_cast<size_t>(rope_position(tk, q_row)) * 128;
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4 c = *reinterpret_cast<const float4*>(trow + 32 * db + 8 * i4 + 4 * g);
                const float4 s = *reinterpret_cast<const float4*>(trow + 64 + 32 * db + 8 * i4 + 4 * g);
                const float cs[4] = {c.x, c.y, c.z, c.w}, sn[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float lo = dq[db][4 * i4 + k], hi = dq[db + 2][4 * i4 + k];
                    rope_turn<true>(lo, hi, cs[k], sn[k]);
                    dq[db][4 * i4 + k] = lo;
                    dq[db + 2][4 * i4 + k] = hi;
                }
            }
    }
    if constexpr (D == 64) {  // sums that are not finite are taken again (psattn_exact.h)
        multiply(dq, a.scale);
        for (AgainGroups n(not_finite_groups(dq), row0, T); n.any(); n.next())
            set_group(dq, n.group(), exact_dq<uint16_t, D>(a, h, n.row, n.dim(), -a.delta[static_cast<size_t>(h) * T + n.row]));
    }
    // the buffer that the last tile was not in
    const int lx = opaque(l);
    const Rows<D> rows{sKb[n_tiles & 1] + 16 * w * kRB, sVb[n_tiles & 1] + 16 * w * kRB};
#pragma unroll
    for (int db = 0; db < kBlocks; ++db) rows.put(db, dq[db], D == 64 ? 1.f : a.scale, lx);
    rows.copy_out(static_cast<char*>(a.dQ) + (static_cast<size_t>(row0) * Hq + h) * kRB, q_row_bytes, lx, T - row0);
}

}  // namespace

int launch_mfma_dq(const AttnArgs& a, void* stream) {
    const unsigned grid = static_cast<unsigned>(a.meta.n_rows[kGridQ]) * a.Hq;
    if (grid == 0) return 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (a.d == 128) psattn_dq_bf16_mfma<128><<<grid, 256, 0, s>>>(a);
    else psattn_dq_bf16_mfma<64><<<grid, 256, 0, s>>>(a);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
