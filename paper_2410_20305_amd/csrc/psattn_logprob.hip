// Per-response log-probabilities and the DPO loss over prefix-shared sequences
// (paper Section 2.1, Eq. 1: the loss needs log pi(y | x) of every completion).
//
// In the prefix-shared sequence [prompt | response 1 | ... | response k] the logits row of a
// token predicts the next token of that token's own branch: inside a response the following
// token, and the LAST prompt token predicts the first token of every response.  Prompt rows
// other than the last, the last row of every response and padding predict nothing and are
// never read, which is where the prefix sharing saves work here too (the prompt is most of
// the tokens).
//
// All three passes stream logits rows of `vocab` elements and are bound by HBM bandwidth: one workgroup per row, 16-byte
// accesses from the row's first aligned element on (rows of an odd vocabulary start anywhere), online max / sum in fp32,
// one exponential per element.  65 536 rows of 32 000 bf16, 9 965 of them with a target: log-sum-exp 169 -> 98 us
// (6.5 TB/s), gradient 906 -> 884 us (5.5 TB/s, almost all of it writes; a plain fill reaches 5.6 - 5.8); 8 334 rows of
// 50 257 fp32, 3 206 with a target: 242 -> 100 us and 588 -> 476 us.
// Every sum is taken in a fixed order (no atomics): results are deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <type_traits>
#include <vector>

#include "psattn.h"

struct psattn_lp_plan {
    int32_t T = 0, n_samples = 0, n_resp = 0, n_rows = 0;
    int64_t n_items = 0;
    int device = -1;
    void* d_blob = nullptr;
    // device views into d_blob
    const int32_t* rows = nullptr;         // [n_rows]   logits rows that predict something, ascending
    const int32_t* row_desc = nullptr;     // [T]        -1: predicts nothing; j >= 0: row inside response j (predicts token row + 1);
                                           //            -2 - i: last prompt row of sample i (predicts the first token of each response)
    const int32_t* resp_first = nullptr;   // [n_resp]   first token of the response
    const int32_t* resp_len = nullptr;     // [n_resp]
    const int32_t* resp_prev = nullptr;    // [n_resp]   last prompt row of its sample, -1 if the prompt is empty
    const int32_t* samp_ptr = nullptr;     // [n_samples + 1] responses of sample i
};

namespace {

constexpr int kThreads = 256;

// Threads per row of the gradient, which writes far more than it reads: of long rows fewer open at a time suit the memory,
// short ones leave most of many threads without work.  Whole head, 256 / 512 / 1024 threads, 46 000 rows, of which 39 900
// have a target: 5 000 bf16 (10 000 bytes) 230 / 225 / 261 us, 8 000 349 / 323 / 349, 9 600 405 / 375 / 405, 11 000 501 / - /
// 461, 16 000 723 / - / 640; 33 600 rows with 9 600 targets: 5 000 100 / 95 / 92, 8 000 133 / 126 / 156, 11 000 222 / - / 189.
// On 65 536 rows of 32 000 the gradient alone 957 / 941 / 923 (non-temporal stores 965 / - / 884).
constexpr size_t kMidRowBytes = 8192, kWideRowBytes = 20480;  // 512 threads, 1024 threads
constexpr int kUnroll = 4;  // 16-byte loads in flight per lane of the log-sum-exp
// Non-temporal accesses where the data is larger than the 256 MB last-level cache, so that the pass that follows could
// not find it there anyway (reading 4 GB alone: 6.3 -> 7.1 TB/s).  Log-probabilities alone (a frozen policy's), rows read by
// ordinary / by non-temporal loads, us: 322 MB of rows with a target 66 / 58, 638 MB 118 / 104, 2.1 GB 352 / 315, 3.9 GB 667 / 598.
// Ordinary loads pay only where a gradient follows that takes the rows from the last one back and finds up to 256 MB of them: whole
// head, that way / this way, 322 MB 274 / 299, 638 MB of 4.2 GB 957 / 989, 822 MB 665 / 686, but 1.0 GB 533 / 528, 2.1 GB 1 058 / 1 020,
// 3.9 GB 2 046 / 1 994; with the last 224 MB alone by ordinary loads the log-probabilities still take 71 / 119 / 329 / 611.
constexpr size_t kCacheBytes = size_t{256} << 20;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

__device__ inline float ld1(const float* p) { return *p; }
__device__ inline float ld1(const uint16_t* p) { return __uint_as_float(static_cast<uint32_t>(*p) << 16); }
__device__ inline uint32_t pack_bf16(float a, float b) {  // round to nearest even
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ inline void st1(float* p, float v) { *p = v; }
__device__ inline void st1(uint16_t* p, float v) { *p = static_cast<uint16_t>(pack_bf16(v, 0.f)); }

template <typename E> struct Vec;
template <> struct Vec<uint16_t> { static constexpr int N = 8; };  // 16 bytes
template <> struct Vec<float> { static constexpr int N = 4; };

template <bool NT, typename E>
__device__ inline u32x4 load_raw(const E* p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    else return *reinterpret_cast<const u32x4*>(p);
}
__device__ inline void unpack(const u32x4& u, float (&x)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[2 * j] = __uint_as_float(u[j] << 16);
        x[2 * j + 1] = __uint_as_float(u[j] & 0xffff0000u);
    }
}
__device__ inline void unpack(const u32x4& u, float (&x)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = __uint_as_float(u[j]);
}
template <bool NT, typename E>
__device__ inline void store_vec(E* p, const float* x) {
    u32x4 u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if constexpr (sizeof(E) == 2) u[j] = pack_bf16(x[2 * j], x[2 * j + 1]);
        else u[j] = __float_as_uint(x[j]);
    }
    if constexpr (NT) __builtin_nontemporal_store(u, reinterpret_cast<u32x4*>(p));
    else *reinterpret_cast<u32x4*>(p) = u;
}

// A row seen as `head` single elements up to the first 16-byte boundary, n_vec aligned groups of N, and the rest.
struct RowSplit {
    int head, n_vec, tail;  // tail: index of the first element behind the groups
};
// WHOLE: every row starts on a boundary and is a whole number of groups (the host has looked)
template <bool WHOLE, typename E>
__device__ inline RowSplit split_row(const E* x, int vocab) {
    constexpr int N = Vec<E>::N;
    if constexpr (WHOLE) return RowSplit{0, vocab / N, vocab};
    const int mis = static_cast<int>(reinterpret_cast<uintptr_t>(x) / sizeof(E)) & (N - 1);
    RowSplit r;
    r.head = min(vocab, (N - mis) & (N - 1));
    r.n_vec = (vocab - r.head) / N;
    r.tail = r.head + r.n_vec * N;
    return r;
}

// (m, s) pairs of an online log-sum-exp: value = m + log s
__device__ inline void lse_merge(float& m, float& s, float m2, float s2) {
    const float mn = fmaxf(m, m2);
    if (mn == -INFINITY) { m = mn; s = 0.f; return; }
    s = s * __expf(m - mn) + s2 * __expf(m2 - mn);
    m = mn;
}

// block-wide reduction in a fixed order; result valid in thread 0
__device__ inline void block_lse(float& m, float& s, float* sm, float* ss) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float m2 = __shfl_down(m, off), s2 = __shfl_down(s, off);
        lse_merge(m, s, m2, s2);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sm[w] = m; ss[w] = s; }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < kThreads / 64; ++i) lse_merge(m, s, sm[i], ss[i]);
}

__device__ inline float block_sum(float v, float* sm) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sm[w] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < kThreads / 64; ++i) v += sm[i];
    return v;
}

// ---- pass 1: log-sum-exp of every row that predicts something
template <typename E, bool NT, bool WHOLE>
__global__ __launch_bounds__(kThreads) void psattn_lp_row_lse(const int32_t* rows, int vocab, const E* logits, float* row_lse) {
    __shared__ float sm[kThreads / 64], ss[kThreads / 64];
    const int row = rows[blockIdx.x];
    const E* x = logits + static_cast<size_t>(row) * vocab;
    constexpr int N = Vec<E>::N;
    const RowSplit r = split_row<WHOLE>(x, vocab);
    const E* xv = x + r.head;
    float m = -INFINITY, s = 0.f;
    auto groups = [&](auto COUNT, int c) {  // groups c, c + kThreads, ...
        constexpr int n = decltype(COUNT)::value;
        u32x4 raw[n];
#pragma unroll
        for (int u = 0; u < n; ++u) raw[u] = load_raw<NT>(xv + static_cast<size_t>(c + u * kThreads) * N);
        float mx = m;
#pragma unroll
        for (int u = 0; u < n; ++u) {
            float v[N];
            unpack(raw[u], v);
#pragma unroll
            for (int j = 0; j < N; ++j) mx = fmaxf(mx, v[j]);
        }
        const float ref = mx == -INFINITY ? 0.f : mx;
        s *= __expf(m - ref);
#pragma unroll
        for (int u = 0; u < n; ++u) {
            float v[N], acc = 0.f;
            unpack(raw[u], v);
#pragma unroll
            for (int j = 0; j < N; ++j) acc += __expf(v[j] - ref);
            s += acc;
        }
        m = mx;
    };
    int c = threadIdx.x;
    for (; c + (kUnroll - 1) * kThreads < r.n_vec; c += kThreads * kUnroll) groups(std::integral_constant<int, kUnroll>{}, c);
    for (; c < r.n_vec; c += kThreads) groups(std::integral_constant<int, 1>{}, c);
    auto one = [&](int i) {
        const float v = ld1(x + i), mx = fmaxf(m, v), ref = mx == -INFINITY ? 0.f : mx;
        s = s * __expf(m - ref) + __expf(v - ref);
        m = mx;
    };
    if constexpr (!WHOLE) {
        if (static_cast<int>(threadIdx.x) < r.head) one(threadIdx.x);
        for (int i = r.tail + threadIdx.x; i < vocab; i += kThreads) one(i);
    }
    block_lse(m, s, sm, ss);
    if (threadIdx.x == 0) row_lse[row] = m + __logf(s);
}

// ---- pass 2: log pi(response | prompt) = sum over its tokens of logit[row, token] - lse[row]
template <typename E>
__global__ __launch_bounds__(kThreads) void psattn_lp_resp_sum(const int32_t* resp_first, const int32_t* resp_len,
                                                               const int32_t* resp_prev, int vocab, const E* logits,
                                                               const int32_t* token_ids, const float* row_lse, float* resp_logp) {
    __shared__ float sm[kThreads / 64];
    const int j = blockIdx.x, first = resp_first[j], n = resp_len[j], prev = resp_prev[j];
    float acc = 0.f;
    for (int u = threadIdx.x; u < n; u += kThreads) {
        const int row = u == 0 ? prev : first + u - 1;
        if (row < 0) continue;  // empty prompt: nothing predicts the first token
        const int tok = token_ids[first + u];
        if (tok < 0 || tok >= vocab) continue;  // not a token of this vocabulary: contributes nothing
        acc += ld1(logits + static_cast<size_t>(row) * vocab + tok) - row_lse[row];
    }
    acc = block_sum(acc, sm);
    if (threadIdx.x == 0) resp_logp[j] = acc;
}

// ---- backward: d logits = sum over the row's items of d_logp[j] (onehot(target) - softmax(row))
template <typename E, bool NT, bool WHOLE, int kBwdThreads>
__global__ __launch_bounds__(kBwdThreads) void psattn_lp_bwd(const int32_t* row_desc, const int32_t* resp_first,
                                                          const int32_t* resp_len, const int32_t* samp_ptr, int vocab,
                                                          const E* logits, const int32_t* token_ids, const float* row_lse,
                                                          const float* d_logp, E* dlogits, int first) {
    const int row = first + static_cast<int>(blockIdx.x), desc = row_desc[row];
    const E* x = logits + static_cast<size_t>(row) * vocab;
    E* g = dlogits + static_cast<size_t>(row) * vocab;
    constexpr int N = Vec<E>::N;
    RowSplit sp = split_row<WHOLE>(g, vocab);
    if (desc == -1) {  // predicts nothing: the row of the gradient is zero, the logits are not read
        float z[N];
#pragma unroll
        for (int j = 0; j < N; ++j) z[j] = 0.f;
        for (int c = threadIdx.x; c < sp.n_vec; c += kBwdThreads) store_vec<NT>(g + sp.head + static_cast<size_t>(c) * N, z);
        if constexpr (!WHOLE) {
            if (static_cast<int>(threadIdx.x) < sp.head) st1(g + threadIdx.x, 0.f);
            for (int i = sp.tail + threadIdx.x; i < vocab; i += kBwdThreads) st1(g + i, 0.f);
        }
        return;
    }
    // total weight of the row's items
    int r0, r1;
    if (desc >= 0) { r0 = desc; r1 = desc + 1; }
    else { const int i = -2 - desc; r0 = samp_ptr[i]; r1 = samp_ptr[i + 1]; }
    // target token of item j of this row, -1 if the item does not exist (empty response) or its token
    // is not of this vocabulary
    auto target = [&](int j) {
        if (desc < 0 && resp_len[j] == 0) return -1;
        const int t = desc >= 0 ? token_ids[row + 1] : token_ids[resp_first[j]];
        return t >= 0 && t < vocab ? t : -1;
    };
    const int only = desc >= 0 ? target(r0) : -1;  // rows inside a response have one item
    float coef = 0.f;
    if (desc >= 0) {
        if (only >= 0) coef = d_logp[r0];
    } else {
        for (int j = r0; j < r1; ++j)
            if (target(j) >= 0) coef += d_logp[j];
    }
    const float lse = row_lse[row];
    if (!WHOLE && (reinterpret_cast<uintptr_t>(x) ^ reinterpret_cast<uintptr_t>(g)) & 15) sp = {0, 0, 0};  // the two rows share no 16-byte boundaries
    const E* xv = x + sp.head;
    E* gv = g + sp.head;
    auto grad = [&](float v) { return -coef * __expf(v - lse); };
    for (int c = threadIdx.x; c < sp.n_vec; c += kBwdThreads) {
        float v[N];
        unpack(load_raw<false>(xv + static_cast<size_t>(c) * N), v);
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = grad(v[k]);
        store_vec<NT>(gv + static_cast<size_t>(c) * N, v);
    }
    if constexpr (!WHOLE) {
        if (static_cast<int>(threadIdx.x) < sp.head) st1(g + threadIdx.x, grad(ld1(x + threadIdx.x)));
        for (int i = sp.tail + threadIdx.x; i < vocab; i += kBwdThreads) st1(g + i, grad(ld1(x + i)));
    }
    // the target columns: each is recomputed whole by the thread that has just stored it, so it is rounded once and two
    // responses that start with the same token add up
    const auto mine = [&](int tgt) {
        const int owner = tgt < sp.head ? tgt : tgt < sp.tail ? (tgt - sp.head) / N : tgt - sp.tail;
        return owner % kBwdThreads == static_cast<int>(threadIdx.x);
    };
    if (desc >= 0) {  // without reading the tables again, which would keep every wave of a short row waiting
        if (only >= 0 && mine(only)) st1(g + only, grad(ld1(x + only)) + coef);
        return;
    }
    for (int j = r0; j < r1; ++j) {
        const int tgt = target(j);
        if (tgt < 0 || !mine(tgt)) continue;
        float v = grad(ld1(x + tgt));
        for (int k = r0; k < r1; ++k)
            if (target(k) == tgt) v += d_logp[k];
        st1(g + tgt, v);
    }
}

// ---- DPO loss of (chosen, rejected) pairs and its derivative w.r.t. the policy log-probabilities
__global__ void psattn_dpo_loss_kernel(int n_pairs, float beta, const float* lp, const float* lr, float* loss, float* d_lp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pairs) return;
    const float z = beta * ((lp[2 * i] - lr[2 * i]) - (lp[2 * i + 1] - lr[2 * i + 1]));
    // -log sigmoid(z) = max(-z, 0) + log1p(exp(-|z|))
    loss[i] = fmaxf(-z, 0.f) + log1pf(expf(-fabsf(z)));
    const float dz = -1.f / (1.f + expf(z));
    if (d_lp) { d_lp[2 * i] = beta * dz; d_lp[2 * i + 1] = -beta * dz; }
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// All rows start on a 16-byte boundary and are whole numbers of 16 bytes.  Rows of a few KB spend a noticeable part of their
// time on finding that out one by one: 46 000 rows of 512 bf16 66.5 us, by the general path 71.1.
bool whole_rows(int32_t dt, int32_t vocab, const void* x) {
    return reinterpret_cast<uintptr_t>(x) % 16 == 0 && vocab % (dt == PSATTN_BF16 ? 8 : 4) == 0;
}

// n workgroups in grids of at most 2^31 threads (2^32 and more wrap around without an error)
template <typename F>
void in_grids(int32_t n, int threads, F launch) {
    const int64_t most = (int64_t{1} << 31) / threads;
    for (int64_t at = 0; at < n; at += most) launch(static_cast<int32_t>(at), static_cast<uint32_t>(std::min<int64_t>(n - at, most)));
}

}  // namespace

extern "C" {

int psattn_logprob_plan(int32_t n_samples, const int32_t* offset, const int32_t* prefix_len, const int32_t* resp_ptr,
                        const int32_t* resp_len, int32_t total_tokens, void* hip_stream, psattn_lp_plan** out) {
    if (!out) return PSATTN_EINVAL;
    *out = nullptr;
    if (n_samples < 0 || total_tokens < 0) return PSATTN_EINVAL;
    if (n_samples > 0 && (!offset || !prefix_len || !resp_ptr)) return PSATTN_EINVAL;
    try {
        const int32_t n_resp = n_samples > 0 ? resp_ptr[n_samples] : 0;
        if (n_samples > 0 && (resp_ptr[0] != 0 || n_resp < 0 || (n_resp > 0 && !resp_len))) return PSATTN_EINVAL;
        std::vector<int32_t> row_desc(static_cast<size_t>(total_tokens), -1), rows, first(n_resp), len(n_resp), prev(n_resp);
        int64_t prev_end = 0, n_items = 0;
        for (int32_t i = 0; i < n_samples; ++i) {
            const int64_t o = offset[i], p = prefix_len[i];
            if (o < 0 || p < 0 || resp_ptr[i + 1] < resp_ptr[i]) return PSATTN_EINVAL;
            if (o < prev_end) return PSATTN_EOVERLAP;
            int64_t t = o + p;
            bool any = false;
            for (int32_t j = resp_ptr[i]; j < resp_ptr[i + 1]; ++j) {
                const int64_t n = resp_len[j];
                if (n < 0) return PSATTN_EINVAL;
                if (t + n > total_tokens) return PSATTN_ERANGE;
                first[j] = static_cast<int32_t>(t);
                len[j] = static_cast<int32_t>(n);
                prev[j] = p > 0 ? static_cast<int32_t>(o + p - 1) : -1;
                for (int64_t u = 0; u + 1 < n; ++u) row_desc[t + u] = j;  // predicts token t + u + 1
                n_items += n - (p > 0 || n == 0 ? 0 : 1);
                any = any || n > 0;
                t += n;
            }
            if (t == o) return PSATTN_EINVAL;
            if (t > total_tokens) return PSATTN_ERANGE;
            if (p > 0 && any) row_desc[o + p - 1] = -2 - i;
            prev_end = t;
        }
        for (int32_t t = 0; t < total_tokens; ++t)
            if (row_desc[t] != -1) rows.push_back(t);
        psattn_lp_plan* pl = new psattn_lp_plan();
        pl->T = total_tokens; pl->n_samples = n_samples; pl->n_resp = n_resp;
        pl->n_rows = static_cast<int32_t>(rows.size()); pl->n_items = n_items;
        // one blob: rows | row_desc | first | len | prev | samp_ptr
        size_t off = 0;
        auto take = [&](size_t n) { const size_t o = off; off = align_up(off + n * sizeof(int32_t), 256); return o; };
        const size_t o_rows = take(rows.size()), o_desc = take(row_desc.size()), o_first = take(n_resp), o_len = take(n_resp),
                     o_prev = take(n_resp), o_ptr = take(static_cast<size_t>(n_samples) + 1);
        std::vector<char> host(off ? off : 256, 0);
        auto put = [&](size_t o, const int32_t* src, size_t n) { if (n) std::memcpy(host.data() + o, src, n * sizeof(int32_t)); };
        put(o_rows, rows.data(), rows.size());
        put(o_desc, row_desc.data(), row_desc.size());
        put(o_first, first.data(), n_resp);
        put(o_len, len.data(), n_resp);
        put(o_prev, prev.data(), n_resp);
        if (n_samples > 0) put(o_ptr, resp_ptr, static_cast<size_t>(n_samples) + 1);
        hipStream_t s = static_cast<hipStream_t>(hip_stream);
        if (hipGetDevice(&pl->device) != hipSuccess || hipMalloc(&pl->d_blob, host.size()) != hipSuccess) {
            (void)hipGetLastError();
            delete pl;
            return PSATTN_ENOMEM;
        }
        // the host vector dies with this call, so the copy has to be complete on return
        if (hipMemcpyAsync(pl->d_blob, host.data(), host.size(), hipMemcpyHostToDevice, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipFree(pl->d_blob);
            delete pl;
            return PSATTN_EHIP;
        }
        const char* d = static_cast<const char*>(pl->d_blob);
        pl->rows = reinterpret_cast<const int32_t*>(d + o_rows);
        pl->row_desc = reinterpret_cast<const int32_t*>(d + o_desc);
        pl->resp_first = reinterpret_cast<const int32_t*>(d + o_first);
        pl->resp_len = reinterpret_cast<const int32_t*>(d + o_len);
        pl->resp_prev = reinterpret_cast<const int32_t*>(d + o_prev);
        pl->samp_ptr = reinterpret_cast<const int32_t*>(d + o_ptr);
        *out = pl;
    } catch (const std::bad_alloc&) {
        return PSATTN_ENOMEM;
    }
    return PSATTN_OK;
}

int psattn_logprob_plan_free(psattn_lp_plan* plan) {
    if (!plan) return PSATTN_OK;
    int rc = PSATTN_OK;
    if (plan->d_blob && hipFree(plan->d_blob) != hipSuccess) rc = PSATTN_EHIP;
    delete plan;
    return rc;
}

int psattn_logprob_plan_info(const psattn_lp_plan* plan, int32_t* n_responses, int32_t* n_rows, int64_t* n_items) {
    if (!plan) return PSATTN_EINVAL;
    if (n_responses) *n_responses = plan->n_resp;
    if (n_rows) *n_rows = plan->n_rows;
    if (n_items) *n_items = plan->n_items;
    return PSATTN_OK;
}

int psattn_logprob_fwd(const psattn_lp_plan* plan, int32_t dt, int32_t vocab, const void* logits, const int32_t* token_ids,
                       float* row_lse, float* resp_logp, void* hip_stream) {
    if (!plan || vocab <= 0 || (dt != PSATTN_F32 && dt != PSATTN_BF16)) return PSATTN_EINVAL;
    if (plan->n_resp == 0) return PSATTN_OK;
    if (!logits || !token_ids || !row_lse || !resp_logp) return PSATTN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (plan->n_rows > 0) {
        const bool nt = static_cast<size_t>(plan->n_rows) * vocab * (dt == PSATTN_BF16 ? 2 : 4) > kCacheBytes;
        auto lse = [&](auto kernel, auto* x) {
            in_grids(plan->n_rows, kThreads, [&](int32_t at, uint32_t n) { kernel<<<n, kThreads, 0, s>>>(plan->rows + at, vocab, x, row_lse); });
        };
        const bool whole = whole_rows(dt, vocab, logits);
        auto typed = [&](auto* x) {
            using E = std::remove_const_t<std::remove_pointer_t<decltype(x)>>;
            if (nt) lse(whole ? psattn_lp_row_lse<E, true, true> : psattn_lp_row_lse<E, true, false>, x);
            else lse(whole ? psattn_lp_row_lse<E, false, true> : psattn_lp_row_lse<E, false, false>, x);
        };
        if (dt == PSATTN_BF16) typed(static_cast<const uint16_t*>(logits));
        else typed(static_cast<const float*>(logits));
    }
    auto sum = [&](auto* x) {
        in_grids(plan->n_resp, kThreads, [&](int32_t at, uint32_t n) {
            psattn_lp_resp_sum<<<n, kThreads, 0, s>>>(plan->resp_first + at, plan->resp_len + at, plan->resp_prev + at, vocab, x, token_ids, row_lse, resp_logp + at);
        });
    };
    if (dt == PSATTN_BF16) sum(static_cast<const uint16_t*>(logits));
    else sum(static_cast<const float*>(logits));
    return hipGetLastError() == hipSuccess ? PSATTN_OK : PSATTN_EHIP;
}

int psattn_logprob_bwd(const psattn_lp_plan* plan, int32_t dt, int32_t vocab, const void* logits, const int32_t* token_ids,
                       const float* row_lse, const float* d_resp_logp, void* dlogits, void* hip_stream) {
    if (!plan || vocab <= 0 || (dt != PSATTN_F32 && dt != PSATTN_BF16)) return PSATTN_EINVAL;
    if (plan->T == 0) return PSATTN_OK;
    if (!logits || !token_ids || !row_lse || !dlogits || (plan->n_resp > 0 && !d_resp_logp)) return PSATTN_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const size_t row_bytes = static_cast<size_t>(vocab) * (dt == PSATTN_BF16 ? 2 : 4);
    const bool nt = plan->T * row_bytes > kCacheBytes;
    const bool whole = whole_rows(dt, vocab, logits) && whole_rows(dt, vocab, dlogits);
    auto bwd = [&](auto nontemporal, auto whole_, auto threads, auto* x, auto* g) {
        constexpr int n = decltype(threads)::value;
        in_grids(plan->T, n, [&](int32_t at, uint32_t rows) {
            psattn_lp_bwd<std::remove_pointer_t<decltype(g)>, decltype(nontemporal)::value, decltype(whole_)::value, n><<<rows, n, 0, s>>>(
                plan->row_desc, plan->resp_first, plan->resp_len, plan->samp_ptr, vocab, x, token_ids, row_lse, d_resp_logp, g, at);
        });
    };
    auto typed = [&](auto* x, auto* g) {
        auto sized = [&](auto nontemporal, auto whole_) {
            if (row_bytes >= kWideRowBytes) bwd(nontemporal, whole_, std::integral_constant<int, 1024>{}, x, g);
            else if (row_bytes >= kMidRowBytes) bwd(nontemporal, whole_, std::integral_constant<int, 512>{}, x, g);
            else bwd(nontemporal, whole_, std::integral_constant<int, 256>{}, x, g);
        };
        if (nt && whole) sized(std::true_type{}, std::true_type{});
        else if (nt) sized(std::true_type{}, std::false_type{});
        else if (whole) sized(std::false_type{}, std::true_type{});
        else sized(std::false_type{}, std::false_type{});
    };
    if (dt == PSATTN_BF16) typed(static_cast<const uint16_t*>(logits), static_cast<uint16_t*>(dlogits));
    else typed(static_cast<const float*>(logits), static_cast<float*>(dlogits));
    return hipGetLastError() == hipSuccess ? PSATTN_OK : PSATTN_EHIP;
}

int psattn_dpo_loss(int32_t n_pairs, float beta, const float* logp_policy, const float* logp_ref, float* loss, float* d_logp,
                    void* hip_stream) {
    if (n_pairs < 0) return PSATTN_EINVAL;
    if (n_pairs == 0) return PSATTN_OK;
    if (!logp_policy || !logp_ref || !loss) return PSATTN_EINVAL;
    psattn_dpo_loss_kernel<<<(n_pairs + 255) / 256, 256, 0, static_cast<hipStream_t>(hip_stream)>>>(n_pairs, beta, logp_policy, logp_ref, loss, d_logp);
    return hipGetLastError() == hipSuccess ? PSATTN_OK : PSATTN_EHIP;
}

}  // extern "C"
