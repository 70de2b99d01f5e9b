// fp32 matrix-core kernels for any tile grid, any scale, float or bfloat16 storage, head_dim 64 or 128.  They serve
// the fp32 configuration (where the 1e-5 tolerance rules out bf16 products) and every shape the bf16 kernels are not
// built for.  All products are v_mfma_f32_16x16x4_f32 (fp32 operands, fp32 accumulation), exponentials are expf / logf;
// scores are never stored.
//
// What bounds them: at the sizes this path is used for (up to a few thousand tokens on a few heads) the chip is far
// from full and a kernel lasts as long as its longest chain of loads, so the work is cut as finely as the matrix
// instruction allows: a workgroup owns 16 queries of one head (forward, dQ) or 16 keys of one kv-head (dK/dV) and its
// eight waves share the 16-wide blocks of the other axis round-robin; their partial results are combined through LDS
// in a fixed order (no atomics).  Operands go from global memory (L1 / L2) straight into registers as 16-byte loads
// in both orientations; nothing is staged.  A step of one 168-token fp32 sample on one head of 64: forward 222 us,
// delta + dQ 143 us, dK/dV 524 us with one thread per row; 7.7 us and, dQ and dK/dV in one launch, 11.4 us with these.
//
// Operand layout of the 16x16x4 product (r = lane % 16, g = lane / 16): A element (row r, k g), B element (k g,
// column r), C register i = (row 4 g + i, column r).
//   scores   S^T = K Q^T: a lane loads 16 bytes of its key's (query's) row at head dims 16 t + 4 g; component c of
//            load t is step (t, c), which contracts head dims {16 t + 4 g + c}.
//   outputs  O^T += V^T P^T: C register i of the scores is the B operand of step i, which contracts keys {4 g + i};
//            the A operand is 16 bytes of key 4 g + i at head dims 64 h + 4 r: component c gives output block (h, c),
//            whose row r is head dim 64 h + 4 r + c, so that a lane ends up with four neighbouring head dims.
//
// Sums that are not finite are taken again on the allowed pairs alone (psattn_exact.h).
//
// Which 16-wide blocks hold an allowed pair follows from the per-token descriptors of Algorithm 3 alone (a query block
// reads keys from its earliest sample start to its last query, without the blocks that are hidden from all its rows;
// a key block is read by queries up to its largest key_hi), so the tile lists are not needed here.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "psattn_exact.h"

namespace psattn {
namespace {

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kB = 16;  // rows of a block

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <typename F>
__device__ inline int over_rows(int x, F f) {  // f over the 16 rows of the block (the same in all lanes)
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) x = f(x, __shfl_xor(x, m));
    return __builtin_amdgcn_readfirstlane(x);
}
__device__ inline float sum_groups(float x) {  // over the four lanes that share a row
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// Key blocks that the 16 queries of a block can read: [first, last], except those inside [hole_lo, hole_hi).
struct KeyRange {
    int first, last, hole_lo, hole_hi;
    __device__ inline bool skip(int kb) const { return kB * kb >= hole_lo && kB * kb + kB <= hole_hi; }
};
__device__ inline KeyRange key_range(const Tok4& tk, int q0, int T) {
    const bool real = tk.s != kPadStart;
    KeyRange k;
    const int s = over_rows(tk.s, [](int x, int y) { return min(x, y); });
    k.hole_lo = over_rows(real ? tk.hole_lo : INT32_MIN, [](int x, int y) { return max(x, y); });
    k.hole_hi = over_rows(real ? tk.hole_hi : INT32_MAX, [](int x, int y) { return min(x, y); });
    k.first = s / kB;
    k.last = s == kPadStart ? -1 : (min(T, q0 + kB) - 1) / kB;
    return k;
}

// rows `row` of a [T, H, D] tensor, clamped to the last token (what a clamped row yields is masked)
template <typename E, int D>
__device__ inline const E* row_of(const void* base, int row, int T, int H, int h) {
    return static_cast<const E*>(base) + (static_cast<size_t>(min(row, T - 1)) * H + h) * D;
}

// score operand: this lane's 16 bytes of every 16 head dims of its row
template <typename E, int D>
__device__ inline void load_rows(f32x4 (&x)[D / 16], const E* row, int g) {
#pragma unroll
    for (int t = 0; t < D / 16; ++t) x[t] = ld4(row + 16 * t + 4 * g);
}
template <int D>
__device__ inline f32x4 dot_rows(const f32x4 (&x)[D / 16], const f32x4 (&y)[D / 16]) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, s2 = s;  // two chains: a dependent product waits for the one before it
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        s = mfma4(x[t][0], y[t][0], s);
        s2 = mfma4(x[t][1], y[t][1], s2);
        s = mfma4(x[t][2], y[t][2], s);
        s2 = mfma4(x[t][3], y[t][3], s2);
    }
    return s + s2;
}
// output operand: 16 bytes of each of the block's rows 4 g + i
template <typename E, int D>
__device__ inline void load_cols(f32x4 (&x)[4][D / 64], const void* base, int r0, int T, int H, int h, int r, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const E* row = row_of<E, D>(base, r0 + 4 * g + i, T, H, h);
#pragma unroll
        for (int hh = 0; hh < D / 64; ++hh) x[i][hh] = ld4(row + 64 * hh + 4 * r);
    }
}
template <int D>
__device__ inline void add_outer(f32x4 (&acc)[D / 16], const f32x4 (&x)[4][D / 64], const f32x4& p) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < D / 16; ++b) acc[b] = mfma4(x[i][b >> 2][b & 3], p[i], acc[b]);
}

// partial results of the waves, [wave][row][head dim], rows padded against bank conflicts
template <int D>
struct Partials {
    float v[kWaves][kB][D + 4];
};
template <int D>
__device__ inline void put_partial(Partials<D>& sm, const f32x4 (&acc)[D / 16], int w, int r, int g) {
#pragma unroll
    for (int hh = 0; hh < D / 64; ++hh)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 v = {acc[4 * hh][i], acc[4 * hh + 1][i], acc[4 * hh + 2][i], acc[4 * hh + 3][i]};
            *reinterpret_cast<f32x4*>(&sm.v[w][r][64 * hh + 16 * g + 4 * i]) = v;
        }
}
// the workgroup's 512 threads as (row, four head dims); D = 64 needs half of them
template <int D>
__device__ inline bool my_quad(int tid, int& row, int& d) {
    row = tid / (D / 4);
    d = 4 * (tid % (D / 4));
    return row < kB;
}
template <int D>
__device__ inline f32x4 sum_partials(const Partials<D>& sm, int row, int d) {
    f32x4 v = *reinterpret_cast<const f32x4*>(&sm.v[0][row][d]);
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += *reinterpret_cast<const f32x4*>(&sm.v[w][row][d]);
    return v;
}

// ---------------------------------------------------------------- forward
template <typename E, int D>
__global__ __launch_bounds__(kThreads) void generic_fwd(AttnArgs a, int first) {
    fetch_args(a);
    __shared__ Partials<D> sm;
    __shared__ float s_m[kWaves][kB], s_l[kWaves][kB];
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv, n_blocks = (T - 1) / kB + 1;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), r = tid & 15, g = (tid >> 4) & 3;
    const int block = first + static_cast<int>(blockIdx.x);
    const int h = block % Hq, kvh = h / (Hq / Hkv), q0 = kB * (n_blocks - 1 - block / Hq);
    const int q = q0 + r;
    const TokenLoad begun = token_begin(a.meta, q);
    f32x4 qf[D / 16], acc[D / 16];
    load_rows<E, D>(qf, row_of<E, D>(a.Q, q, T, Hq, h), g);
    const Tok4 tk = token_choose(a.meta, begun, token_search(a.meta, q));
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const KeyRange kr = key_range(tk, q0, T);
    float m = -INFINITY, l = 0.f;
    for (int kb = kr.first + w; kb <= kr.last; kb += kWaves) {
        if (kr.skip(kb)) continue;
        const int k0 = kB * kb;
        f32x4 kf[D / 16], vc[4][D / 64];
        load_rows<E, D>(kf, row_of<E, D>(a.K, k0 + r, T, Hkv, kvh), g);
        load_cols<E, D>(vc, a.V, k0, T, Hkv, kvh, r, g);
        f32x4 s = dot_rows<D>(kf, qf);
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = allowed(tk, q, k0 + 4 * g + i) ? s[i] * a.scale : -INFINITY;
            mx = fmaxf(mx, s[i]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mn = fmaxf(m, mx), ref = mn == -INFINITY ? 0.f : mn;
        const float alpha = expf(m - ref);  // m = -inf: 0
        l *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) { s[i] = expf(s[i] - ref); l += s[i]; }
#pragma unroll
        for (int b = 0; b < D / 16; ++b) acc[b] *= alpha;
        add_outer<D>(acc, vc, s);
        m = mn;
    }
    l = sum_groups(l);
    put_partial<D>(sm, acc, w, r, g);
    if (g == 0) { s_m[w][r] = m; s_l[w][r] = l; }
    __syncthreads();
    int row, d;
    const bool mine = my_quad<D>(tid, row, d) && q0 + row < T;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    if (mine) {
        float mt = s_m[0][row], lt = 0.f;
#pragma unroll
        for (int i = 1; i < kWaves; ++i) mt = fmaxf(mt, s_m[i][row]);
        const float ref = mt == -INFINITY ? 0.f : mt;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            const float f = expf(s_m[i][row] - ref);
            lt = fmaf(s_l[i][row], f, lt);
            o += *reinterpret_cast<const f32x4*>(&sm.v[i][row][d]) * f;
        }
        o *= lt > 0.f ? 1.f / lt : 0.f;
        if (!is_finite(o) || !(lt > 0.f)) o = exact_o<E, D>(a, h, q0 + row, d);  // (no sum: padding, or scores of -inf alone)
        if (d == 0) a.LSEout[static_cast<size_t>(h) * T + q0 + row] = lt > 0.f ? mt + logf(lt) : -INFINITY;
    }
    __syncthreads();  // nobody reads Q any more: O may take its memory
    if (mine) st4(static_cast<E*>(a.Oout) + (static_cast<size_t>(q0 + row) * Hq + h) * D + d, o);
}

// ---------------------------------------------------------------- delta = rowsum(dO o O), dQ
template <typename E, int D>
__device__ inline void dq_block(const AttnArgs& a, Partials<D>& sm, int block) {
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv, n_blocks = (T - 1) / kB + 1;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), r = tid & 15, g = (tid >> 4) & 3;
    const int h = block % Hq, kvh = h / (Hq / Hkv), q0 = kB * (n_blocks - 1 - block / Hq);
    const int q = q0 + r;
    const TokenLoad begun = token_begin(a.meta, q);
    f32x4 qf[D / 16], gf[D / 16], acc[D / 16];
    load_rows<E, D>(qf, row_of<E, D>(a.Q, q, T, Hq, h), g);
    load_rows<E, D>(gf, row_of<E, D>(a.dO, q, T, Hq, h), g);
    const Tok4 tk = token_choose(a.meta, begun, token_search(a.meta, q));
    const float lse = a.LSE[static_cast<size_t>(h) * T + min(q, T - 1)];
    float delta = 0.f;
    {
        const E* orow = row_of<E, D>(a.O, q, T, Hq, h);
#pragma unroll
        for (int t = 0; t < D / 16; ++t) {
            const f32x4 o = ld4(orow + 16 * t + 4 * g);
#pragma unroll
            for (int c = 0; c < 4; ++c) delta = fmaf(o[c], gf[t][c], delta);
            acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    delta = sum_groups(delta);
    if (w == 0 && g == 0 && q < T) a.delta[static_cast<size_t>(h) * T + q] = delta;
    const KeyRange kr = key_range(tk, q0, T);
    for (int kb = kr.first + w; kb <= kr.last; kb += kWaves) {
        if (kr.skip(kb)) continue;
        const int k0 = kB * kb;
        f32x4 kf[D / 16], vf[D / 16], kc[4][D / 64];
        load_rows<E, D>(kf, row_of<E, D>(a.K, k0 + r, T, Hkv, kvh), g);
        load_rows<E, D>(vf, row_of<E, D>(a.V, k0 + r, T, Hkv, kvh), g);
        load_cols<E, D>(kc, a.K, k0, T, Hkv, kvh, r, g);
        const f32x4 s = dot_rows<D>(kf, qf), dp = dot_rows<D>(vf, gf);
        f32x4 ds;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            ds[i] = allowed(tk, q, k0 + 4 * g + i) ? expf(s[i] * a.scale - lse) * (dp[i] - delta) : 0.f;
        add_outer<D>(acc, kc, ds);
    }
    put_partial<D>(sm, acc, w, r, g);
    __syncthreads();
    int row, d;
    if (!my_quad<D>(tid, row, d) || q0 + row >= T) return;
    f32x4 dq = sum_partials<D>(sm, row, d) * scale_of(a);
    if (!is_finite(dq)) dq = exact_dq<E, D>(a, h, q0 + row, d, a.delta[static_cast<size_t>(h) * T + q0 + row]);
    st4(static_cast<E*>(a.dQ) + (static_cast<size_t>(q0 + row) * Hq + h) * D + d, dq);
}

// ---------------------------------------------------------------- dK, dV
// the waves share the (query block, head of the group) pairs, heads innermost; OWN_DELTA: delta = rowsum(dO o O) is
// computed here, from O, instead of being read from what the dQ pass left
template <typename E, int D, bool OWN_DELTA>
__device__ inline void dkdv_block(const AttnArgs& a, Partials<D>& sm, int block) {
    const int T = a.meta.T, Hq = a.Hq, Hkv = a.Hkv, G = Hq / Hkv;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), r = tid & 15, g = (tid >> 4) & 3;
    const int kvh = block % Hkv, k0 = kB * (block / Hkv), key = k0 + r;
    const int key_hi = token_choose(a.meta, token_begin(a.meta, key), token_search(a.meta, key)).key_hi;  // queries [key, key_hi) read this key
    f32x4 kf[D / 16], vf[D / 16], dk[D / 16], dv[D / 16];
    load_rows<E, D>(kf, row_of<E, D>(a.K, key, T, Hkv, kvh), g);
    load_rows<E, D>(vf, row_of<E, D>(a.V, key, T, Hkv, kvh), g);
#pragma unroll
    for (int b = 0; b < D / 16; ++b) dk[b] = dv[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int q_end = over_rows(key_hi, [](int x, int y) { return max(x, y); });
    const int n_it = q_end > k0 ? ((q_end - k0 + kB - 1) / kB) * G : 0;
    for (int it = w; it < n_it; it += kWaves) {
        const int q0 = k0 + kB * (it / G), h = kvh * G + it % G;
        f32x4 qf[D / 16], gf[D / 16], qc[4][D / 64], gc[4][D / 64];
        float lse[4], delta[4];
        load_rows<E, D>(gf, row_of<E, D>(a.dO, q0 + r, T, Hq, h), g);
        if constexpr (OWN_DELTA) {
            const E* orow = row_of<E, D>(a.O, q0 + r, T, Hq, h);
            float dl = 0.f;
#pragma unroll
            for (int t = 0; t < D / 16; ++t) {
                const f32x4 o = ld4(orow + 16 * t + 4 * g);
#pragma unroll
                for (int c = 0; c < 4; ++c) dl = fmaf(o[c], gf[t][c], dl);  // the dQ pass's order of sums
            }
            dl = sum_groups(dl);
#pragma unroll
            for (int i = 0; i < 4; ++i) delta[i] = __shfl(dl, 4 * g + i);
            if constexpr (D == 128) __builtin_amdgcn_sched_barrier(0);  // O is used up before the other operands need its registers
        }
        load_rows<E, D>(qf, row_of<E, D>(a.Q, q0 + r, T, Hq, h), g);
        load_cols<E, D>(qc, a.Q, q0, T, Hq, h, r, g);
        load_cols<E, D>(gc, a.dO, q0, T, Hq, h, r, g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const size_t at = static_cast<size_t>(h) * T + min(q0 + 4 * g + i, T - 1);
            lse[i] = a.LSE[at];
            if constexpr (!OWN_DELTA) delta[i] = a.delta[at];
        }
        const f32x4 s = dot_rows<D>(qf, kf), dp = dot_rows<D>(gf, vf);
        f32x4 p, ds;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = q0 + 4 * g + i;
            const bool ok = key <= q && q < key_hi;
            p[i] = ok ? expf(s[i] * a.scale - lse[i]) : 0.f;
            ds[i] = ok ? p[i] * (dp[i] - delta[i]) : 0.f;
        }
        add_outer<D>(dv, gc, p);
        add_outer<D>(dk, qc, ds);
    }
    int row, d;
    const bool mine = my_quad<D>(tid, row, d) && k0 + row < T;
    const size_t at = (static_cast<size_t>(k0 + row) * Hkv + kvh) * D + d;
    f32x4 xk = {0.f, 0.f, 0.f, 0.f}, xv = xk;
    put_partial<D>(sm, dk, w, r, g);
    __syncthreads();
    if (mine) xk = sum_partials<D>(sm, row, d) * scale_of(a);
    __syncthreads();
    put_partial<D>(sm, dv, w, r, g);
    __syncthreads();
    if (mine) {
        xv = sum_partials<D>(sm, row, d);
        if (!is_finite(xk)) xk = exact_dkdv<E, D, true, OWN_DELTA ? 0 : 1>(a, kvh, k0 + row, d);
        if (!is_finite(xv)) xv = exact_dkdv<E, D, false, OWN_DELTA ? 0 : 1>(a, kvh, k0 + row, d);
    }
    __syncthreads();  // nobody reads K and V any more: dK and dV may take their memory
    if (mine) {
        st4(static_cast<E*>(a.dK) + at, xk);
        st4(static_cast<E*>(a.dV) + at, xv);
    }
}

template <typename E, int D>
__global__ __launch_bounds__(kThreads) void generic_dq(AttnArgs a, int first) {
    fetch_args(a);
    __shared__ Partials<D> sm;
    dq_block<E, D>(a, sm, first + static_cast<int>(blockIdx.x));
}
template <typename E, int D>
__global__ __launch_bounds__(kThreads) void generic_dkdv(AttnArgs a, int first) {
    fetch_args(a);
    __shared__ Partials<D> sm;
    dkdv_block<E, D, false>(a, sm, first + static_cast<int>(blockIdx.x));
}
// both at once: neither needs anything of the other
template <typename E, int D>
__global__ __launch_bounds__(kThreads) void generic_bwd(AttnArgs a, int first) {
    fetch_args(a);
    __shared__ Partials<D> sm;
    const int block = first + static_cast<int>(blockIdx.x), n_dkdv = ((a.meta.T - 1) / kB + 1) * a.Hkv;
    if (block < n_dkdv) dkdv_block<E, D, true>(a, sm, block);
    else dq_block<E, D>(a, sm, block - n_dkdv);
}

}  // namespace

// A grid of 512 threads may hold just under 2^23 workgroups (2^32 threads); more go in several launches.
constexpr int64_t kMostGroups = int64_t{1} << 22;

#define PSATTN_DISPATCH(KERNEL, HEADS)                                                                      \
    do {                                                                                                    \
        hipStream_t s = static_cast<hipStream_t>(stream);                                                   \
        const int64_t groups = (static_cast<int64_t>(a.meta.T) + kB - 1) / kB * (HEADS);                    \
        if (groups > INT32_MAX) return static_cast<int>(hipErrorInvalidConfiguration);                      \
        for (int64_t at = 0; at < groups; at += kMostGroups) {                                              \
            const int first = static_cast<int>(at);                                                         \
            const unsigned grid = static_cast<unsigned>(std::min(groups - at, kMostGroups));                \
            if (dt == PSATTN_F32 && a.d == 64) KERNEL<float, 64><<<grid, kThreads, 0, s>>>(a, first);       \
            else if (dt == PSATTN_F32) KERNEL<float, 128><<<grid, kThreads, 0, s>>>(a, first);              \
            else if (a.d == 64) KERNEL<uint16_t, 64><<<grid, kThreads, 0, s>>>(a, first);                   \
            else KERNEL<uint16_t, 128><<<grid, kThreads, 0, s>>>(a, first);                                 \
            if (const hipError_t err = hipGetLastError(); err != hipSuccess) return static_cast<int>(err);  \
        }                                                                                                   \
        return 0;                                                                                           \
    } while (0)

int launch_generic_fwd(int dt, const AttnArgs& a, void* stream) { PSATTN_DISPATCH(generic_fwd, a.Hq); }
int launch_generic_dq(int dt, const AttnArgs& a, void* stream) { PSATTN_DISPATCH(generic_dq, a.Hq); }
int launch_generic_dkdv(int dt, const AttnArgs& a, void* stream) { PSATTN_DISPATCH(generic_dkdv, a.Hkv); }
int launch_generic_bwd(int dt, const AttnArgs& a, void* stream) { PSATTN_DISPATCH(generic_bwd, a.Hq + a.Hkv); }

// One launch lets the dK/dV workgroups start with the dQ ones instead of behind them, for a recomputed delta per pair of
// blocks.  It pays while both together do not fill the chip many times over and dK/dV is not the longer of the two by far
// (its chains grow with the heads of a group).  Measured, whole fp32 step, one launch / two, head_dim 64 then 128, over 1 to
// 16 query heads and 40 to 4 000 tokens (84 tables): up to 174 workgroups 25 / 27 to 60 / 77 us and 27 / 32 to 92 / 98, but
// groups of four heads at 128 from 145 workgroups on 151 / 144, 308 / 286 (315), 154 / 146 (290); 1 250 to 2 500 workgroups,
// samples of 1 000 tokens, 196 / 229 and 377 / 421 (4 / 1 heads), 331 / 341 and 635 / 660 (8 / 2), samples of 2 000, 574 / 529
// and 1 133 / 1 035 (8 / 2); 4 000 and more 336 / 310, 1 143 / 1 057.  The losses inside the line, eleven of 76 tables, are 1 to
// 9 %, the gains up to 31 %; what separates them is not a size that the host knows.
bool generic_bwd_in_one(const AttnArgs& a) {
    const int64_t groups = (static_cast<int64_t>(a.meta.T) + kB - 1) / kB * (a.Hq + a.Hkv);
    return groups <= 2560 && a.Hq <= 4 * a.Hkv;
}

}  // namespace psattn
