// Brings a block mask onto the device: one kernel that reads the pinned staging buffer over PCIe, expands the runs of
// equal token descriptors into one descriptor per token and copies the tile lists.
//
// Why a kernel and not hipMemcpyAsync: a copy of more than a few KB goes to a DMA engine, and handing the stream from
// the compute queue to it and back costs more than the copy (measured between two steps of 8 samples, 8 334 tokens:
// 9 us gap + 8 us copy + 16 us gap before the forward kernel; 8 + 27 + 12..30 us at 65 536 tokens).  A kernel stays in
// the queue.  Its time is PCIe latency, so everything is requested in one go: with up to 256 runs a block fetches them
// all without waiting for its index into them.
#include <hip/hip_runtime.h>

#include "psattn_internal.h"

namespace psattn {
namespace {

constexpr int kThreads = 256;
constexpr int kMostRuns = kUploadTokens + 1;  // runs that can touch one block's tokens (none is empty)

__global__ __launch_bounds__(kThreads) void psattn_meta_upload(UploadArgs a, int tok_blocks) {
    const int tid = threadIdx.x, b = blockIdx.x;
    if (b >= tok_blocks) {
        const uint32_t i = static_cast<uint32_t>(b - tok_blocks) * kThreads + tid;
        if (i < static_cast<uint32_t>(a.n_units)) a.dst[i] = a.src[i];
        return;
    }
    __shared__ int s_start[kMostRuns];
    __shared__ Tok4 s_tok[kMostRuns];
    int base = 0, n = a.n_seg;
    if (n > kThreads) {
        base = a.block_first[b];
        n = min(a.block_first[b + 1] - base + 1, kMostRuns);
    }
    for (int i = tid; i < n; i += kThreads) {
        s_start[i] = a.seg_start[base + i];
        s_tok[i] = a.seg_tok[base + i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kUploadTokens / kThreads; ++k) {
        const int t = b * kUploadTokens + k * kThreads + tid;
        if (t >= a.T) break;
        int lo = 0, hi = n;  // last run that starts at or before t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_start[mid] <= t) lo = mid;
            else hi = mid;
        }
        a.tok[t] = s_tok[lo];
    }
}

}  // namespace

int launch_upload(const UploadArgs& a, void* stream) {
    const int tok_blocks = upload_blocks(a.T), list_blocks = static_cast<int>((int64_t{a.n_units} + kThreads - 1) / kThreads);
    if (tok_blocks + list_blocks == 0) return 0;
    psattn_meta_upload<<<tok_blocks + list_blocks, kThreads, 0, static_cast<hipStream_t>(stream)>>>(a, tok_blocks);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
