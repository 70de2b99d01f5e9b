// C-ABI entry points that touch the device: metadata upload, argument checks and
// kernel dispatch for psattn_fwd / psattn_bwd.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "psattn_internal.h"

using namespace psattn;

namespace {

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Device copy of a block mask: tok | lists.  Staged on the host: lists | seg_start | seg_tok | block_first; the
// descriptors of the tokens are expanded on the device, so that what crosses PCIe does not grow with T.
struct BlobLayout {
    size_t f_ent, f_lch, b_ent, b_lch, lists;         // inside the lists
    size_t tok;                                       // device: bytes of the token descriptors, the lists follow
    size_t seg_start, seg_tok, block_first, staged;   // host
};

BlobLayout layout_of(const psattn_meta& m) {
    BlobLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    L.f_ent = take(sizeof(int32_t) * m.fwd.entry.size());
    L.f_lch = take(sizeof(RowLaunch) * m.fwd.order.size());
    L.b_ent = take(sizeof(int32_t) * m.bwd.entry.size());
    L.b_lch = take(sizeof(RowLaunch) * m.bwd.order.size());
    L.lists = off;
    L.seg_start = take(sizeof(int32_t) * m.seg_start.size());
    L.seg_tok = take(sizeof(Tok4) * m.seg_tok.size());
    L.block_first = take(sizeof(int32_t) * (upload_blocks(m.T) + 1));
    L.staged = off;
    L.tok = align_up(sizeof(Tok4) * static_cast<size_t>(m.T), 256);
    return L;
}

// walk_backwards: the kernel of this grid starts with the last entry of a row
void fill_csr(int32_t* entry, RowLaunch* rl, const TileCsr& g, bool walk_backwards) {
    if (!g.entry.empty()) std::memcpy(entry, g.entry.data(), g.entry.size() * sizeof(int32_t));
    for (size_t i = 0; i < g.order.size(); ++i) {
        const int32_t r = g.order[i], b = g.row_ptr[r], n = g.row_ptr[r + 1] - b;
        rl[i] = RowLaunch{r, b, n, n > 0 ? g.entry[walk_backwards ? b + n - 1 : b] : 0};
    }
}

// ---- pooled metadata blobs
// A mini-batch needs one pinned staging buffer and one device buffer.
// Allocating and freeing them every training step would synchronise the device each
// time, so released pairs stay in a small per-process pool and are handed out again.
// A pair carries an event that marks the point after which the device no longer needs
// it (recorded when its meta object is released); it is reused once that event has
// completed.
struct Blob {
    void* d = nullptr;
    void* h = nullptr;
    void* hd = nullptr;   // h as the device addresses it
    size_t cap = 0;       // bytes of each of the two
    int device = -1;
    hipEvent_t idle = nullptr;  // completes when the previous user is done with d and h
};
constexpr size_t kPoolMax = 8;  // idle pairs kept; beyond that the smallest is freed
std::mutex g_pool_mu;
std::vector<Blob> g_pool;

void destroy_blob(Blob& b) {
    if (b.idle) { (void)hipEventSynchronize(b.idle); (void)hipEventDestroy(b.idle); }
    if (b.d) (void)hipFree(b.d);
    if (b.h) (void)hipHostFree(b.h);
    b = Blob{};
}

// Returns a pair of at least `bytes` on `device`; blocks only if every pooled candidate is
// still in use by the device and the pool is full.
int acquire_blob(size_t bytes, int device, Blob* out) {
    bool wait = false;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        int best = -1, busy = -1;  // best: smallest idle pair that fits
        for (size_t i = 0; i < g_pool.size(); ++i) {
            const Blob& b = g_pool[i];
            if (b.device != device || b.cap < bytes) continue;
            if (hipEventQuery(b.idle) == hipSuccess) {
                if (best < 0 || b.cap < g_pool[best].cap) best = static_cast<int>(i);
            } else {
                (void)hipGetLastError();  // hipErrorNotReady is not an error here
                if (busy < 0) busy = static_cast<int>(i);
            }
        }
        if (best < 0 && busy >= 0 && g_pool.size() >= kPoolMax) {
            best = busy;
            wait = true;
        }
        if (best >= 0) {
            *out = g_pool[best];
            g_pool.erase(g_pool.begin() + best);
        }
    }
    if (out->d) {
        if (wait && hipEventSynchronize(out->idle) != hipSuccess) { destroy_blob(*out); return PSATTN_EHIP; }
        return PSATTN_OK;
    }
    Blob b;
    b.device = device;
    b.cap = align_up(bytes + bytes / 4, 1 << 16);  // head-room: the next mini-batch differs a little
    if (hipEventCreateWithFlags(&b.idle, hipEventDisableTiming) != hipSuccess) { b.idle = nullptr; (void)hipGetLastError(); return PSATTN_EHIP; }
    if (hipHostMalloc(&b.h, b.cap, hipHostMallocDefault) != hipSuccess) { b.h = nullptr; (void)hipGetLastError(); destroy_blob(b); return PSATTN_ENOMEM; }
    if (hipHostGetDevicePointer(&b.hd, b.h, 0) != hipSuccess) { (void)hipGetLastError(); destroy_blob(b); return PSATTN_EHIP; }
    if (hipMalloc(&b.d, b.cap) != hipSuccess) { b.d = nullptr; (void)hipGetLastError(); destroy_blob(b); return PSATTN_ENOMEM; }
    *out = b;
    return PSATTN_OK;
}

// `stream`: the pair may be reused once the work enqueued there so far has finished.
void release_blob(Blob b, hipStream_t stream) {
    if (!b.d) return;
    if (hipEventRecord(b.idle, stream) != hipSuccess) { (void)hipGetLastError(); destroy_blob(b); return; }
    Blob drop;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        g_pool.push_back(b);
        if (g_pool.size() > kPoolMax) {
            size_t s = 0;
            for (size_t i = 1; i < g_pool.size(); ++i)
                if (g_pool[i].cap < g_pool[s].cap) s = i;
            drop = g_pool[s];
            g_pool.erase(g_pool.begin() + s);
        }
    }
    if (drop.d) destroy_blob(drop);
}

// A mask that fits travels with the kernels' arguments (psattn_mask.h).
bool put_in_args(psattn_meta& m) {
    const size_t n = m.seg_tok.size();
    if (m.T == 0 || m.T > kSmallTokens || n > kSmallRuns) return false;
    SmallMask s{};
    for (size_t i = 0; i < kSmallRuns; ++i) {
        uint64_t x = kSmallNone;
        if (i < n) {
            const Tok4& t = m.seg_tok[i];
            const int32_t f[5] = {m.seg_start[i], t.s == kPadStart ? static_cast<int32_t>(kSmallNone) : t.s, t.hole_lo, t.hole_hi, t.key_hi};
            x = 0;
            for (int k = 0; k < 5; ++k) x |= static_cast<uint64_t>(static_cast<uint32_t>(f[k])) << (kSmallField * k);
        }
        s.run[i] = x;
    }
    const TileCsr* grid[2] = {&m.fwd, &m.bwd};
    for (int g = 0; g < 2; ++g) {
        const TileCsr& c = *grid[g];
        if (c.order.size() > kSmallRows) return false;
        for (size_t i = 0; i < c.order.size(); ++i) {
            const int32_t r = c.order[i];
            uint32_t tiles = 0;
            for (int32_t k = c.row_ptr[r]; k < c.row_ptr[r + 1]; ++k) {
                const int32_t tile = c.entry[k] >> 2;
                if (tile >= kSmallTiles) return false;
                tiles |= ((c.entry[k] & 3) == PSATTN_TILE_FULL ? 0x10001u : 1u) << tile;
            }
            s.tiles[g][i] = tiles;
            s.row[g] |= static_cast<uint32_t>(r) << (4 * i);
        }
    }
    m.dev.small = s;
    m.dev.in_args = 1;
    return true;
}

int upload(psattn_meta* m, hipStream_t stream) {
    if (hipGetDevice(&m->device) != hipSuccess) return PSATTN_EHIP;
    m->dev.T = m->T;
    const TileCsr* grid[2] = {&m->fwd, &m->bwd};
    for (int g = 0; g < 2; ++g) {
        const int32_t n = static_cast<int32_t>(grid[g]->order.size());
        m->dev.n_rows[g] = n;
        m->size[g].n_entries = static_cast<int64_t>(grid[g]->entry.size());
        for (int32_t r = 0; r < n; ++r) m->size[g].longest = std::max(m->size[g].longest, grid[g]->row_ptr[r + 1] - grid[g]->row_ptr[r]);
    }
    if (put_in_args(*m)) {
        m->on_device = true;
        return PSATTN_OK;
    }
    const BlobLayout L = layout_of(*m);
    const size_t on_device = L.tok + L.lists;
    Blob b;
    const int rc = acquire_blob(std::max(L.staged, on_device), m->device, &b);
    if (rc != PSATTN_OK) return rc;
    m->h_stage = b.h;
    m->h_stage_dev = b.hd;
    m->d_blob = b.d;
    m->blob_cap = b.cap;
    m->blob_idle = b.idle;
    char* h = static_cast<char*>(m->h_stage);
    fill_csr(reinterpret_cast<int32_t*>(h + L.f_ent), reinterpret_cast<RowLaunch*>(h + L.f_lch), m->fwd, false);
    fill_csr(reinterpret_cast<int32_t*>(h + L.b_ent), reinterpret_cast<RowLaunch*>(h + L.b_lch), m->bwd, true);
    const int32_t n_seg = static_cast<int32_t>(m->seg_tok.size()), n_blocks = upload_blocks(m->T);
    std::memcpy(h + L.seg_start, m->seg_start.data(), m->seg_start.size() * sizeof(int32_t));
    if (n_seg > 0) std::memcpy(h + L.seg_tok, m->seg_tok.data(), m->seg_tok.size() * sizeof(Tok4));
    int32_t* first = reinterpret_cast<int32_t*>(h + L.block_first);
    for (int32_t k = 0, i = 0; k <= n_blocks; ++k) {
        const int64_t t = std::min<int64_t>(static_cast<int64_t>(k) * kUploadTokens, m->T - 1);
        while (i + 1 < n_seg && m->seg_start[i + 1] <= t) ++i;
        first[k] = i;
    }
    char* d = static_cast<char*>(m->d_blob);
    const char* hd = static_cast<const char*>(m->h_stage_dev);
    UploadArgs u{};
    u.seg_start = reinterpret_cast<const int32_t*>(hd + L.seg_start);
    u.seg_tok = reinterpret_cast<const Tok4*>(hd + L.seg_tok);
    u.block_first = reinterpret_cast<const int32_t*>(hd + L.block_first);
    u.n_seg = n_seg;
    u.T = m->T;
    u.tok = reinterpret_cast<Tok4*>(d);
    u.src = reinterpret_cast<const uint4*>(hd);
    u.dst = reinterpret_cast<uint4*>(d + L.tok);
    if (L.lists / 16 > static_cast<size_t>(INT32_MAX)) return PSATTN_EUNSUPPORTED;
    u.n_units = static_cast<int32_t>(L.lists / 16);
    if (launch_upload(u, stream) != 0) return PSATTN_EHIP;
    m->blob_bytes = on_device;
    const char* lists = d + L.tok;
    m->dev.list.tok = reinterpret_cast<const Tok4*>(d);
    m->dev.list.entry[0] = reinterpret_cast<const int32_t*>(lists + L.f_ent);
    m->dev.list.entry[1] = reinterpret_cast<const int32_t*>(lists + L.b_ent);
    m->dev.list.launch[0] = reinterpret_cast<const RowLaunch*>(lists + L.f_lch);
    m->dev.list.launch[1] = reinterpret_cast<const RowLaunch*>(lists + L.b_lch);
    m->on_device = true;
    return PSATTN_OK;
}

int release_meta(psattn_meta* meta, hipStream_t stream) {
    if (!meta) return PSATTN_OK;
    if (meta->d_blob) {
        Blob b;
        b.d = meta->d_blob; b.h = meta->h_stage; b.hd = meta->h_stage_dev; b.cap = meta->blob_cap; b.device = meta->device;
        b.idle = static_cast<hipEvent_t>(meta->blob_idle);
        // the event and the stream belong to the blob's device
        int cur = -1;
        const bool hop = hipGetDevice(&cur) == hipSuccess && cur != b.device;
        if (hop) (void)hipSetDevice(b.device);
        release_blob(b, stream);
        if (hop) (void)hipSetDevice(cur);
    }
    delete meta;
    return PSATTN_OK;
}

int check_common(const psattn_meta* meta, int32_t dt, int32_t Hq, int32_t Hkv, int32_t d) {
    if (!meta) return PSATTN_EINVAL;
    if (dt != PSATTN_F32 && dt != PSATTN_BF16) return PSATTN_EINVAL;
    if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0) return PSATTN_EINVAL;
    if (d != 64 && d != 128) return PSATTN_EINVAL;
    if (!meta->on_device) return PSATTN_ENODEVICE;
    // tile * heads products must fit the 1-D grid
    if (static_cast<int64_t>(meta->fwd.n_q_tiles) * Hq > INT32_MAX) return PSATTN_EUNSUPPORTED;
    return PSATTN_OK;
}

// The MFMA kernels fold the scale into a base-2 exponent and take row maxima before
// scaling, which needs scale > 0; anything else runs on the generic kernels.
bool mfma_fwd_ok(const psattn_meta* m, int32_t dt, int32_t d, float scale) {
    return dt == PSATTN_BF16 && (d == 128 || d == 64) && scale > 0.f && m->fwd.tile_q == kFwdTileQ &&
           m->fwd.tile_k == kFwdTileK;
}
bool mfma_bwd_ok(const psattn_meta* m, int32_t dt, int32_t d, float scale) {
    return mfma_fwd_ok(m, dt, d, scale) && m->bwd.tile_q == kBwdTileQ && m->bwd.tile_k == kBwdTileK;
}

// The matrix-core kernels move 16 bytes at a time, asynchronous copies among them.
template <typename... P>
bool aligned16(const P*... p) { return ((reinterpret_cast<uintptr_t>(p) | ...) & 15) == 0; }

// ---- optional per-pass event timing
bool g_profile = false;
struct EventPair { hipEvent_t a, b; int pass; };
std::vector<EventPair> g_events;
constexpr size_t kMaxPendingEvents = 1 << 16;

struct PassTimer {
    hipStream_t stream;
    EventPair ev{};
    bool active = false;
    PassTimer(int pass, void* s) : stream(static_cast<hipStream_t>(s)) {
        if (!g_profile) return;
        if (hipEventCreate(&ev.a) != hipSuccess) return;
        if (hipEventCreate(&ev.b) != hipSuccess) { (void)hipEventDestroy(ev.a); return; }
        ev.pass = pass;
        active = hipEventRecord(ev.a, stream) == hipSuccess;
    }
    ~PassTimer() {
        if (!active) return;
        (void)hipEventRecord(ev.b, stream);
        if (g_events.size() < kMaxPendingEvents) {
            g_events.push_back(ev);
        } else {  // nobody reads them: do not grow without bound
            (void)hipEventDestroy(ev.a);
            (void)hipEventDestroy(ev.b);
        }
    }
};

// kernel launched last per pass (psattn_kernel_name)
const char* g_last_kernel[4] = {nullptr, nullptr, nullptr, nullptr};

}  // namespace

namespace psattn {

size_t bwd_scratch_bytes(const psattn_meta* meta, int32_t n_q_heads) {
    return 2 * align_up(sizeof(float) * static_cast<size_t>(meta->T) * n_q_heads, 256) + 256;
}

int bwd_checked(const psattn_meta* meta, int32_t dt, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                float scale, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                const float* LSE, void* dQ, void* dK, void* dV, void* scratch_base, size_t scratch_bytes,
                void* hip_stream, const float* rope_table) {
    const int rc = check_common(meta, dt, n_q_heads, n_kv_heads, head_dim);
    if (rc != PSATTN_OK) return rc;
    if (meta->T == 0) return PSATTN_OK;
    if (!Q || !K || !V || !O || !dO || !LSE || !dQ || !dK || !dV || !scratch_base) return PSATTN_EINVAL;
    if (scratch_bytes < bwd_scratch_bytes(meta, n_q_heads)) return PSATTN_EINVAL;
    AttnArgs a{};
    a.meta = meta->dev;
    std::copy_n(meta->size, 2, a.size);
    a.Hq = n_q_heads; a.Hkv = n_kv_heads; a.d = head_dim; a.scale = scale;
    a.Q = Q; a.K = K; a.V = V; a.O = O; a.dO = dO; a.LSE = LSE;
    a.dQ = dQ; a.dK = dK; a.dV = dV;
    a.rope = rope_table;
    a.delta = reinterpret_cast<float*>(align_up(reinterpret_cast<uintptr_t>(scratch_base), 256));
    a.lse2 = a.delta + align_up(sizeof(float) * static_cast<size_t>(meta->T) * n_q_heads, 256) / sizeof(float);
    int err = 0;
    const bool mfma = mfma_bwd_ok(meta, dt, head_dim, scale) && (head_dim == 128 || aligned16(Q, K, V, O, dO, dQ, dK, dV));
    if (rope_table && !(mfma && head_dim == 128)) return PSATTN_EUNSUPPORTED;  // rotary embedding lives in these matrix-core kernels only
    // One launch reads Q, K, V, O and dO while the gradients are being written, two read O in the first and of K and V only
    // the workgroup's own rows in the second: a gradient that takes the memory of O, K or V needs them.
    const size_t e = dt == PSATTN_F32 ? 4 : 2, q_bytes = e * meta->T * n_q_heads * head_dim, kv_bytes = e * meta->T * n_kv_heads * head_dim;
    const auto apart = [&](const void* out, size_t n) {
        const auto from = [&](const void* in, size_t m) {
            const uintptr_t x = reinterpret_cast<uintptr_t>(out), y = reinterpret_cast<uintptr_t>(in);
            return x + n <= y || y + m <= x;
        };
        return from(Q, q_bytes) && from(O, q_bytes) && from(dO, q_bytes) && from(K, kv_bytes) && from(V, kv_bytes);
    };
    if (!mfma && generic_bwd_in_one(a) && apart(dQ, q_bytes) && apart(dK, kv_bytes) && apart(dV, kv_bytes)) {
        PassTimer t(3, hip_stream);
        g_last_kernel[1] = g_last_kernel[2] = g_last_kernel[3] = "generic_bwd";
        return launch_generic_bwd(dt, a, hip_stream) == 0 ? PSATTN_OK : PSATTN_EHIP;
    }
    {  // the dQ kernels compute delta themselves and leave it in the scratch for the dK/dV pass
        PassTimer t(2, hip_stream);
        err = mfma ? launch_mfma_dq(a, hip_stream) : launch_generic_dq(dt, a, hip_stream);
        g_last_kernel[1] = g_last_kernel[2] = mfma ? "psattn_dq_bf16_mfma" : "generic_dq";
    }
    if (err) return PSATTN_EHIP;
    {
        PassTimer t(3, hip_stream);
        err = !mfma ? launch_generic_dkdv(dt, a, hip_stream)
                    : head_dim == 64 ? launch_mfma_dkdv64(a, hip_stream) : launch_mfma_dkdv(a, hip_stream);
        g_last_kernel[3] = !mfma ? "generic_dkdv" : head_dim == 64 ? "psattn_dkdv64_bf16_mfma" : "psattn_dkdv_bf16_mfma";
    }
    return err == 0 ? PSATTN_OK : PSATTN_EHIP;
}

int fwd_checked(const psattn_meta* meta, int32_t dt, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                float scale, const void* Q, const void* K, const void* V, void* O, float* LSE,
                const float* rope_table, void* Qr, void* hip_stream) {
    int rc = check_common(meta, dt, n_q_heads, n_kv_heads, head_dim);
    if (rc != PSATTN_OK) return rc;
    if (meta->T == 0) return PSATTN_OK;
    if (!Q || !K || !V || !O || !LSE) return PSATTN_EINVAL;
    AttnArgs a{};
    a.meta = meta->dev;
    std::copy_n(meta->size, 2, a.size);
    a.Hq = n_q_heads; a.Hkv = n_kv_heads; a.d = head_dim; a.scale = scale;
    a.Q = Q; a.K = K; a.V = V; a.Oout = O; a.LSEout = LSE;
    a.rope = rope_table; a.Qr = Qr;
    const bool mfma = mfma_fwd_ok(meta, dt, head_dim, scale) && (head_dim == 128 || aligned16(Q, K, V, O));
    if (rope_table && !(mfma && head_dim == 128)) return PSATTN_EUNSUPPORTED;  // rotary embedding lives in these matrix-core kernels only
    int err;
    {
        PassTimer t(0, hip_stream);
        err = !mfma ? launch_generic_fwd(dt, a, hip_stream) : head_dim == 64 ? launch_mfma_fwd64(a, hip_stream) : mfma_fwd_three(a) ? launch_mfma_fwd3(a, hip_stream) : launch_mfma_fwd(a, hip_stream);
        g_last_kernel[0] = mfma ? "psattn_fwd_bf16_mfma" : "generic_fwd";
    }
    return err == 0 ? PSATTN_OK : PSATTN_EHIP;
}

}  // namespace psattn

extern "C" {

int psattn_profile_enable(int32_t on) {
    g_profile = on != 0;
    return PSATTN_OK;
}

int psattn_profile_read(double* sum_ms, int64_t* count) {
    if (!sum_ms || !count) return PSATTN_EINVAL;
    for (int i = 0; i < 4; ++i) { sum_ms[i] = 0.0; count[i] = 0; }
    int rc = PSATTN_OK;
    for (EventPair& e : g_events) {
        float ms = 0.f;
        if (hipEventSynchronize(e.b) != hipSuccess || hipEventElapsedTime(&ms, e.a, e.b) != hipSuccess) rc = PSATTN_EHIP;
        else { sum_ms[e.pass] += ms; count[e.pass]++; }
        (void)hipEventDestroy(e.a);
        (void)hipEventDestroy(e.b);
    }
    g_events.clear();
    return rc;
}

int psattn_build_meta(int32_t n_samples, const int32_t* offset, const int32_t* prefix_len,
                      const int32_t* chosen_len, const int32_t* rejected_len, int32_t total_tokens,
                      int32_t tile_q, int32_t tile_k, int32_t bwd_tile_q, int32_t bwd_tile_k,
                      void* hip_stream, psattn_meta** out) {
    psattn_meta* m = nullptr;
    int rc = build_host(n_samples, offset, prefix_len, chosen_len, rejected_len, total_tokens, tile_q,
                        tile_k, bwd_tile_q, bwd_tile_k, &m);
    if (rc != PSATTN_OK) return rc;
    rc = upload(m, static_cast<hipStream_t>(hip_stream));
    if (rc != PSATTN_OK) {
        release_meta(m, static_cast<hipStream_t>(hip_stream));
        *out = nullptr;
        return rc;
    }
    *out = m;
    return PSATTN_OK;
}

int psattn_build_meta_multi(int32_t n_samples, const int32_t* offset, const int32_t* prefix_len,
                            const int32_t* resp_ptr, const int32_t* resp_len, int32_t total_tokens,
                            int32_t tile_q, int32_t tile_k, int32_t bwd_tile_q, int32_t bwd_tile_k,
                            void* hip_stream, psattn_meta** out) {
    psattn_meta* m = nullptr;
    int rc = build_host_multi(n_samples, offset, prefix_len, resp_ptr, resp_len, total_tokens, tile_q, tile_k,
                              bwd_tile_q, bwd_tile_k, &m);
    if (rc != PSATTN_OK) return rc;
    rc = upload(m, static_cast<hipStream_t>(hip_stream));
    if (rc != PSATTN_OK) {
        release_meta(m, static_cast<hipStream_t>(hip_stream));
        *out = nullptr;
        return rc;
    }
    *out = m;
    return PSATTN_OK;
}

int psattn_free_meta(psattn_meta* meta) { return release_meta(meta, nullptr); }

int psattn_free_meta_async(psattn_meta* meta, void* hip_stream) {
    return release_meta(meta, static_cast<hipStream_t>(hip_stream));
}

int psattn_trim_pool(void) {
    std::vector<Blob> all;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        all.swap(g_pool);
    }
    int cur = -1;
    (void)hipGetDevice(&cur);
    for (Blob& b : all) {
        if (cur >= 0 && b.device != cur) (void)hipSetDevice(b.device);
        destroy_blob(b);
        if (cur >= 0 && b.device != cur) (void)hipSetDevice(cur);
    }
    return PSATTN_OK;
}

int psattn_uses_mfma(const psattn_meta* meta, int32_t dt, int32_t head_dim, float scale, int32_t backward) {
    if (!meta) return PSATTN_EINVAL;
    return (backward ? mfma_bwd_ok(meta, dt, head_dim, scale) : mfma_fwd_ok(meta, dt, head_dim, scale)) ? 1 : 0;
}

int psattn_fwd(const psattn_meta* meta, int32_t dt, int32_t n_q_heads, int32_t n_kv_heads,
               int32_t head_dim, float scale, const void* Q, const void* K, const void* V, void* O,
               float* LSE, void* hip_stream) {
    return fwd_checked(meta, dt, n_q_heads, n_kv_heads, head_dim, scale, Q, K, V, O, LSE, nullptr, nullptr, hip_stream);
}

size_t psattn_bwd_workspace_bytes(const psattn_meta* meta, int32_t n_q_heads, int32_t n_kv_heads,
                                  int32_t head_dim) {
    (void)n_kv_heads; (void)head_dim;
    if (!meta || n_q_heads <= 0) return 0;
    return bwd_scratch_bytes(meta, n_q_heads);
}

int psattn_bwd(const psattn_meta* meta, int32_t dt, int32_t n_q_heads, int32_t n_kv_heads,
               int32_t head_dim, float scale, const void* Q, const void* K, const void* V,
               const void* O, const void* dO, const float* LSE, void* dQ, void* dK, void* dV,
               void* workspace, size_t workspace_bytes, void* hip_stream) {
    return bwd_checked(meta, dt, n_q_heads, n_kv_heads, head_dim, scale, Q, K, V, O, dO, LSE, dQ, dK, dV, workspace,
                       workspace_bytes, hip_stream);
}

const char* psattn_kernel_name(int32_t dt, int32_t pass) {
    if (pass < 0 || pass > 3) return "";
    if (g_last_kernel[pass]) return g_last_kernel[pass];
    const bool bf = dt == PSATTN_BF16;
    switch (pass) {
        case 0: return bf ? "psattn_fwd_bf16_mfma" : "generic_fwd";
        case 1:
        case 2: return bf ? "psattn_dq_bf16_mfma" : "generic_dq";
        default: return bf ? "psattn_dkdv_bf16_mfma" : "generic_dkdv";
    }
}

}  // extern "C"
