// A whole self-attention layer on prefix-shared sequences: Q/K/V projections, rotary
// embedding with paired-format position ids, prefix-shared attention, output projection,
// forward and backward.  This is the "attention layer" micro-benchmark of the paper's
// Section 4.2: the projections are linear in the number of tokens, so sharing the prompt
// saves them as well as the quadratic attention part.
//
// The four projections and their gradients are plain dense GEMMs and go to rocBLAS
// (bf16 in, fp32 accumulate); everything between them is libpsattn's own kernels, called
// through its C ABI.  Separate shared library: libpsattn.so itself stays free of the BLAS
// dependency.  Weights follow the [out_features, in_features] row-major convention,
// y = x W^T.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <cstdint>
#include <new>

#include "psattn.h"
#include "psattn_layer.h"

struct psattn_layer {
    int32_t hidden = 0, Hq = 0, Hkv = 0, d = 0;
    rocblas_handle blas = nullptr;
};

namespace {

constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// activations and gradients kept between forward and backward, carved out of the caller's workspace
struct Slots {
    char *Q, *K, *V, *Qr, *Kr, *O, *dO, *dQ, *dK, *dV, *attn_ws;
    float* LSE;
    size_t attn_ws_bytes, total;
};

Slots carve(const psattn_layer* L, const psattn_meta* meta, int32_t T, void* base) {
    Slots s{};
    const size_t q = static_cast<size_t>(T) * L->Hq * L->d * 2, k = static_cast<size_t>(T) * L->Hkv * L->d * 2;
    char* p = reinterpret_cast<char*>(align_up(reinterpret_cast<uintptr_t>(base), 256));
    char* p0 = p;
    auto take = [&](size_t n) { char* r = p; p += align_up(n, 256); return r; };
    s.Q = take(q); s.K = take(k); s.V = take(k); s.Qr = take(q); s.Kr = take(k); s.O = take(q);
    s.dO = take(q); s.dQ = take(q); s.dK = take(k); s.dV = take(k);
    s.LSE = reinterpret_cast<float*>(take(static_cast<size_t>(T) * L->Hq * 4));
    s.attn_ws_bytes = psattn_bwd_workspace_bytes(meta, L->Hq, L->Hkv, L->d);
    s.attn_ws = take(s.attn_ws_bytes);
    s.total = static_cast<size_t>(p - p0) + 256;
    return s;
}

// row-major C[M x N] = op(A) op(B) (+ C if accumulate); bf16 operands and result, fp32 accumulation.
// A row-major matrix read as column-major is its transpose, so C^T = op(B)^T op(A)^T is the same
// call with the operands swapped and each operation flag kept.
int gemm_rm(rocblas_handle h, bool ta, bool tb, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda,
            const void* B, int64_t ldb, void* C, int64_t ldc, bool accumulate) {
    if (M == 0 || N == 0) return PSATTN_OK;
    if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return PSATTN_EUNSUPPORTED;
    const float alpha = 1.f, beta = accumulate ? 1.f : 0.f;
    const rocblas_status st = rocblas_gemm_ex(
        h, tb ? rocblas_operation_transpose : rocblas_operation_none, ta ? rocblas_operation_transpose : rocblas_operation_none,
        static_cast<rocblas_int>(N), static_cast<rocblas_int>(M), static_cast<rocblas_int>(K), &alpha, B,
        rocblas_datatype_bf16_r, static_cast<rocblas_int>(ldb), A, rocblas_datatype_bf16_r, static_cast<rocblas_int>(lda), &beta, C,
        rocblas_datatype_bf16_r, static_cast<rocblas_int>(ldc), C, rocblas_datatype_bf16_r, static_cast<rocblas_int>(ldc),
        rocblas_datatype_f32_r, rocblas_gemm_algo_standard, 0, 0);
    return st == rocblas_status_success ? PSATTN_OK : PSATTN_EHIP;
}

// The same for two products of one shape; a_step, b_step, c_step: elements from one's matrices to the other's.
int gemm_rm_pair(rocblas_handle h, bool ta, bool tb, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, int64_t a_step,
                 const void* B, int64_t ldb, int64_t b_step, void* C, int64_t ldc, int64_t c_step) {
    if (M == 0 || N == 0) return PSATTN_OK;
    if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return PSATTN_EUNSUPPORTED;
    const float alpha = 1.f, beta = 0.f;
    const rocblas_status st = rocblas_gemm_strided_batched_ex(
        h, tb ? rocblas_operation_transpose : rocblas_operation_none, ta ? rocblas_operation_transpose : rocblas_operation_none,
        static_cast<rocblas_int>(N), static_cast<rocblas_int>(M), static_cast<rocblas_int>(K), &alpha, B, rocblas_datatype_bf16_r,
        static_cast<rocblas_int>(ldb), b_step, A, rocblas_datatype_bf16_r, static_cast<rocblas_int>(lda), a_step, &beta, C,
        rocblas_datatype_bf16_r, static_cast<rocblas_int>(ldc), c_step, C, rocblas_datatype_bf16_r, static_cast<rocblas_int>(ldc),
        c_step, 2, rocblas_datatype_f32_r, rocblas_gemm_algo_standard, 0, 0);
    return st == rocblas_status_success ? PSATTN_OK : PSATTN_EHIP;
}

// dWk and dWv, n_out x hidden elements each, as one batch of two in `room` bytes: where one product by itself fills at most half
// of the 256 CUs (in tiles of 256 x 256) and the room holds both results.  Backward, one by one / as a pair, us, by hidden x n_out: 512 x
// 512 163 / 150, 1 024 x 1 024 291 / 272, 2 048 x 2 048 517 / 506, 4 096 x 1 024 1 041 / 1 024 (2 560 tokens 557 / 544, 10 240 2 127 / 2 081),
// 6 144 x 1 024 1 918 / 1 880, 4 096 x 2 048 1 202 / 1 188, 8 192 x 1 024 3 324 / 3 320; beyond the line, where the copies of the results
// cost more than the batch gives, 3 072 x 3 072 936 / 946 (10 240 tokens 1 784 / 1 913), 4 096 x 3 072 1 129 / 1 138, 4 096 x 4 096 1 445 /
// 1 469, and either way from table to table at 5 120 x 2 560 and 4 096 x 3 584 (5 120 x 5 120 2 522 / 2 429).
constexpr bool weights_as_pair(size_t n_out, size_t hidden, size_t room) {
    const size_t bytes = n_out * hidden * 2;
    return n_out * hidden <= size_t{128} * 256 * 256 && align_up(bytes, 256) + bytes <= room;
}

}  // namespace

extern "C" {

int psattn_layer_create(int32_t hidden, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, psattn_layer** out) {
    if (!out) return PSATTN_EINVAL;
    *out = nullptr;
    if (hidden <= 0 || n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0) return PSATTN_EINVAL;
    if (head_dim != 128) return PSATTN_EUNSUPPORTED;  // the rotary-embedding kernels
    psattn_layer* L = new (std::nothrow) psattn_layer();
    if (!L) return PSATTN_ENOMEM;
    L->hidden = hidden; L->Hq = n_q_heads; L->Hkv = n_kv_heads; L->d = head_dim;
    if (rocblas_create_handle(&L->blas) != rocblas_status_success) {
        delete L;
        return PSATTN_EHIP;
    }
    rocblas_set_pointer_mode(L->blas, rocblas_pointer_mode_host);
    *out = L;
    return PSATTN_OK;
}

int psattn_layer_free(psattn_layer* layer) {
    if (!layer) return PSATTN_OK;
    const bool ok = !layer->blas || rocblas_destroy_handle(layer->blas) == rocblas_status_success;
    delete layer;
    return ok ? PSATTN_OK : PSATTN_EHIP;
}

size_t psattn_layer_workspace_bytes(const psattn_layer* layer, const psattn_meta* meta, int32_t total_tokens) {
    if (!layer || !meta || total_tokens < 0) return 0;
    return carve(layer, meta, total_tokens, nullptr).total;
}

int psattn_layer_fwd(psattn_layer* L, const psattn_meta* meta, const psattn_rope* rope, int32_t total_tokens, float scale,
                     const void* X, const void* Wq, const void* Wk, const void* Wv, const void* Wo, void* Y,
                     void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!L || !meta || !rope) return PSATTN_EINVAL;
    const int32_t T = total_tokens;
    if (T < 0) return PSATTN_EINVAL;
    if (T == 0) return PSATTN_OK;
    if (!X || !Wq || !Wk || !Wv || !Wo || !Y || !workspace) return PSATTN_EINVAL;
    if (workspace_bytes < psattn_layer_workspace_bytes(L, meta, T)) return PSATTN_EINVAL;
    if (rocblas_set_stream(L->blas, static_cast<hipStream_t>(hip_stream)) != rocblas_status_success) return PSATTN_EHIP;
    const Slots s = carve(L, meta, T, workspace);
    const int64_t h = L->hidden, nq = static_cast<int64_t>(L->Hq) * L->d, nk = static_cast<int64_t>(L->Hkv) * L->d;
    int rc;
    if ((rc = gemm_rm(L->blas, false, true, T, nq, h, X, h, Wq, h, s.Q, nq, false)) != PSATTN_OK) return rc;
    if ((rc = gemm_rm(L->blas, false, true, T, nk, h, X, h, Wk, h, s.K, nk, false)) != PSATTN_OK) return rc;
    if ((rc = gemm_rm(L->blas, false, true, T, nk, h, X, h, Wv, h, s.V, nk, false)) != PSATTN_OK) return rc;
    rc = psattn_fwd_rope(meta, rope, PSATTN_BF16, L->Hq, L->Hkv, L->d, scale, s.Q, s.K, s.V, s.O, s.LSE, s.Qr, s.Kr, hip_stream);
    if (rc != PSATTN_OK) return rc;
    return gemm_rm(L->blas, false, true, T, h, nq, s.O, nq, Wo, nq, Y, h, false);
}

int psattn_layer_bwd(psattn_layer* L, const psattn_meta* meta, const psattn_rope* rope, int32_t total_tokens, float scale,
                     const void* X, const void* Wq, const void* Wk, const void* Wv, const void* Wo, const void* dY,
                     void* dX, void* dWq, void* dWk, void* dWv, void* dWo, void* workspace, size_t workspace_bytes,
                     void* hip_stream) {
    if (!L || !meta || !rope) return PSATTN_EINVAL;
    const int32_t T = total_tokens;
    if (T < 0) return PSATTN_EINVAL;
    if (!X || !Wq || !Wk || !Wv || !Wo || !dY || !dX || !dWq || !dWk || !dWv || !dWo || !workspace) return PSATTN_EINVAL;
    if (workspace_bytes < psattn_layer_workspace_bytes(L, meta, T)) return PSATTN_EINVAL;
    if (rocblas_set_stream(L->blas, static_cast<hipStream_t>(hip_stream)) != rocblas_status_success) return PSATTN_EHIP;
    const Slots s = carve(L, meta, T, workspace);
    const int64_t h = L->hidden, nq = static_cast<int64_t>(L->Hq) * L->d, nk = static_cast<int64_t>(L->Hkv) * L->d;
    int rc;
    // output projection: dO = dY Wo, dWo = dY^T O
    if ((rc = gemm_rm(L->blas, false, false, T, nq, h, dY, h, Wo, nq, s.dO, nq, false)) != PSATTN_OK) return rc;
    if ((rc = gemm_rm(L->blas, true, false, h, nq, T, dY, h, s.O, nq, dWo, nq, false)) != PSATTN_OK) return rc;
    // attention: gradients w.r.t. the unrotated Q, K
    rc = psattn_bwd_rope(meta, rope, PSATTN_BF16, L->Hq, L->Hkv, L->d, scale, s.Qr, s.Kr, s.V, s.O, s.dO, s.LSE, s.dQ, s.dK,
                         s.dV, s.attn_ws, s.attn_ws_bytes, hip_stream);
    if (rc != PSATTN_OK) return rc;
    // projections: dW = dP^T X, dX = dQ Wq + dK Wk + dV Wv
    if ((rc = gemm_rm(L->blas, true, false, nq, h, T, s.dQ, nq, X, h, dWq, h, false)) != PSATTN_OK) return rc;
    // dWk and dWv by themselves fill the chip poorly (63 us each for 31 us of products, 5 120 tokens, hidden 4 096, 8 kv heads).  As one
    // batch they go to the places of the unrotated Q and K, which the backward does not read; the caller's two matrices
    // lie anywhere, hence the copies.
    const size_t wk = static_cast<size_t>(nk) * h * 2, step = align_up(wk, 256);
    if (weights_as_pair(nk, h, s.V - s.Q)) {
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        if ((rc = gemm_rm_pair(L->blas, true, false, nk, h, T, s.dK, nk, (s.dV - s.dK) / 2, X, h, 0, s.Q, h, static_cast<int64_t>(step / 2))) != PSATTN_OK) return rc;
        if (hipMemcpyAsync(dWk, s.Q, wk, hipMemcpyDeviceToDevice, st) != hipSuccess) return PSATTN_EHIP;
        if (hipMemcpyAsync(dWv, s.Q + step, wk, hipMemcpyDeviceToDevice, st) != hipSuccess) return PSATTN_EHIP;
    } else {
        if ((rc = gemm_rm(L->blas, true, false, nk, h, T, s.dK, nk, X, h, dWk, h, false)) != PSATTN_OK) return rc;
        if ((rc = gemm_rm(L->blas, true, false, nk, h, T, s.dV, nk, X, h, dWv, h, false)) != PSATTN_OK) return rc;
    }
    if ((rc = gemm_rm(L->blas, false, false, T, h, nq, s.dQ, nq, Wq, h, dX, h, false)) != PSATTN_OK) return rc;
    if ((rc = gemm_rm(L->blas, false, false, T, h, nk, s.dK, nk, Wk, h, dX, h, true)) != PSATTN_OK) return rc;
    return gemm_rm(L->blas, false, false, T, h, nk, s.dV, nk, Wv, h, dX, h, true);
}

}  // extern "C"
