// Internal declarations shared by the host metadata builder, the C-ABI entry
// points and the kernel launchers of libpsattn.  Not part of the public ABI.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include <hip/hip_vector_types.h>

#include "psattn.h"

namespace psattn {

constexpr int32_t kPadStart = INT32_MAX;
constexpr int kGridQ = 0, kGridK = 1;  // q-major, k-major grid

// Default tile grids = the shapes the bf16 MFMA kernels are built for.
constexpr int32_t kFwdTileQ = 128;
constexpr int32_t kFwdTileK = 64;
constexpr int32_t kBwdTileQ = 64;
constexpr int32_t kBwdTileK = 128;

// One CSR over a tile grid.  entry = (column tile index << 2) | class.
struct TileCsr {
    int32_t tile_q = 0, tile_k = 0;
    int32_t n_q_tiles = 0, n_k_tiles = 0;
    std::vector<int32_t> row_ptr;  // rows = q-tiles (FWD) or k-tiles (BWD)
    std::vector<int32_t> entry;    // (column tile index << 2) | class, ascending in a row
    std::vector<int32_t> order;    // rows in launch order
};

// What a workgroup of the MFMA kernels needs to start on its row, in launch order: one
// 16-byte scalar load instead of a chain of three dependent ones (launch order -> row ->
// list bounds -> first entry), which is a noticeable part of a short workgroup's life.
struct alignas(16) RowLaunch {
    int32_t row;          // tile row (q-tile for the q-major grid, k-tile for the k-major one)
    int32_t begin;        // first position of the row's tile list in `entry`
    int32_t count;        // its length
    int32_t first_entry;  // the entry the walk starts with: entry[begin] for the q-major grid,
                          // entry[begin + count - 1] for the k-major one (walked backwards)
};

// Per-token descriptor as the kernels read it (one 16-byte load).
struct alignas(16) Tok4 {
    int32_t s, hole_lo, hole_hi, key_hi;
};

// A block mask that is small enough to travel with every kernel's arguments instead of being brought onto the device first
// (psattn_mask.h reads it): at most kSmallTokens tokens in kSmallRuns runs of equal descriptors, kSmallRows rows of tiles in
// either grid and 16 tiles the other way.  Index 0: q-major grid, 1: k-major grid.
constexpr int kSmallTokens = 1024, kSmallRuns = 8, kSmallRows = 8, kSmallTiles = 16;
constexpr int kSmallField = 11;                            // bits of a token number; all set: none
constexpr uint32_t kSmallNone = (1u << kSmallField) - 1;
struct SmallMask {
    uint64_t run[kSmallRuns];           // first token | s | hole_lo | hole_hi | key_hi; s is none for padding, first token is none for an unused run
    uint32_t tiles[2][kSmallRows];      // in launch order: bits 0 - 15 the tiles of the row's list, 16 - 31 those that are FULL
    uint32_t row[2];                    // 4 bits for each position of the launch order
};

// Device-side view handed to kernels by value; grid 0: q-major, 1: k-major.
struct DeviceMeta {
    struct Lists {
        const Tok4* tok;             // [T]
        const int32_t* entry[2];     // (idx << 2) | cls
        const RowLaunch* launch[2];  // [n_rows], in launch order
    };
    int32_t T;
    int32_t in_args;
    int32_t n_rows[2];
    union {
        Lists list;
        SmallMask small;             // where in_args
    };
};

// What the launchers want to know of a grid.
struct GridSize {
    int32_t longest;    // entries of the longest row
    int64_t n_entries;  // of all rows
};

}  // namespace psattn

struct psattn_meta {
    int32_t T = 0;
    int32_t n_samples = 0;
    int64_t n_allowed = 0;
    int32_t n_positions = 0;        // 1 + the largest position id of any token (prompt length + longest response)
    // Runs of neighbouring tokens with the same descriptor (a prompt, a response, a stretch of padding), covering
    // [0, T): run i is tokens [seg_start[i], seg_start[i + 1]), seg_start.back() == T.
    std::vector<int32_t> seg_start;
    std::vector<psattn::Tok4> seg_tok;
    psattn::TileCsr fwd, bwd;
    // device copy
    bool on_device = false;
    int device = -1;
    void* d_blob = nullptr;   // device copy of the metadata (from the library's blob pool)
    void* h_stage = nullptr;  // pinned staging buffer, alive until release
    void* h_stage_dev = nullptr;  // its address on the device
    size_t blob_bytes = 0;    // bytes in use (0: the mask travels with the kernels' arguments)
    size_t blob_cap = 0;      // bytes allocated
    void* blob_idle = nullptr;  // hipEvent_t of the pooled pair
    psattn::DeviceMeta dev{};
    psattn::GridSize size[2] = {};
};

namespace psattn {

// Host-only construction (psattn_meta.cpp).  Returns a psattn_status.
int build_host(int32_t n_samples, const int32_t* offset, const int32_t* prefix_len,
               const int32_t* chosen_len, const int32_t* rejected_len, int32_t total_tokens,
               int32_t tile_q, int32_t tile_k, int32_t bwd_tile_q, int32_t bwd_tile_k,
               psattn_meta** out);

int build_host_multi(int32_t n_samples, const int32_t* offset, const int32_t* prefix_len,
                     const int32_t* resp_ptr, const int32_t* resp_len, int32_t total_tokens,
                     int32_t tile_q, int32_t tile_k, int32_t bwd_tile_q, int32_t bwd_tile_k,
                     psattn_meta** out);

// What every kernel starts with stands close together: each first access to 64 bytes of the arguments takes some 500 cycles, all of
// those that fetch_args makes at once as long as one.
struct AttnArgs {
    int32_t Hq, Hkv, d;
    float scale;
    const void *Q, *K, *V, *dO, *O;
    const float* LSE;
    // Rotary embedding (nullptr = none): table [positions][128] = cos[64] | sin[64] per position id.
    // Forward: Q arrives unrotated, is rotated in registers and, if Qr is set, saved rotated for the
    // backward; K arrives rotated.  Backward: Q and K arrive rotated, dQ and dK leave unrotated.
    const float* rope;
    DeviceMeta meta;
    float* delta;  // [Hq, T]  workspace: rowsum(dO o O); the MFMA kernels keep its negative here
    float* lse2;   // [Hq, T]  workspace: LSE * log2(e), written by the MFMA dQ pass for the dK/dV pass
    void *Oout, *dQ, *dK, *dV;
    float* LSEout;
    void* Qr;
    GridSize size[2];
};


// psattn_fwd with optional rotary embedding (rope_table == nullptr: none).
int fwd_checked(const psattn_meta* meta, int32_t dt, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                float scale, const void* Q, const void* K, const void* V, void* O, float* LSE,
                const float* rope_table, void* Qr, void* hip_stream);

// psattn_bwd without the workspace-size lookup: argument checks, then delta / dQ / dK/dV
// on `scratch_base` (device memory of at least bwd_scratch_bytes()).  Returns a psattn_status.
size_t bwd_scratch_bytes(const psattn_meta* meta, int32_t n_q_heads);
int bwd_checked(const psattn_meta* meta, int32_t dt, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                float scale, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                const float* LSE, void* dQ, void* dK, void* dV, void* scratch_base, size_t scratch_bytes,
                void* hip_stream, const float* rope_table = nullptr);

// Unpacks a staged block mask on the device (psattn_upload.hip): expands the runs of equal token descriptors into
// tok[T] and copies the lists.  All source pointers are pinned host memory as the device addresses it.
struct UploadArgs {
    const int32_t* seg_start;   // [n_seg + 1]
    const Tok4* seg_tok;        // [n_seg]
    const int32_t* block_first; // [blocks + 1]  run that holds the first token of block b (kUploadTokens tokens each)
    int32_t n_seg, T;
    Tok4* tok;
    const uint4* src;           // lists, 16-byte units
    uint4* dst;
    int32_t n_units;
};
constexpr int32_t kUploadTokens = 1024;
constexpr int32_t upload_blocks(int32_t T) { return static_cast<int32_t>((int64_t{T} + kUploadTokens - 1) / kUploadTokens); }
int launch_upload(const UploadArgs& a, void* stream);

// Launchers (each returns a hipError_t cast to int; 0 = success).
int launch_generic_fwd(int dt, const AttnArgs& a, void* stream);
int launch_generic_dq(int dt, const AttnArgs& a, void* stream);
int launch_generic_dkdv(int dt, const AttnArgs& a, void* stream);
int launch_generic_bwd(int dt, const AttnArgs& a, void* stream);  // dQ, dK, dV in one launch
bool generic_bwd_in_one(const AttnArgs& a);                       // where that is the faster way
int launch_mfma_fwd(const AttnArgs& a, void* stream);    // head_dim 128
int launch_mfma_fwd3(const AttnArgs& a, void* stream);   // the same with three workgroups to a CU
bool mfma_fwd_three(const AttnArgs& a);                  // where that is the faster way
int launch_mfma_fwd64(const AttnArgs& a, void* stream);
int launch_mfma_dq(const AttnArgs& a, void* stream);
int launch_mfma_dkdv(const AttnArgs& a, void* stream);
int launch_mfma_dkdv64(const AttnArgs& a, void* stream);

}  // namespace psattn
