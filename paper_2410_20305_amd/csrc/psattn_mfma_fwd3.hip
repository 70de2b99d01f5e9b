// bf16 MFMA forward at head_dim 128 with three workgroups to a CU (psattn_mfma_fwd.h), built without NaNs to honour like the one with two.
#include "psattn_mfma_fwd.h"

namespace psattn {

// From the grid on that fills the chip once with three workgroups to a CU; below, the second barrier and V's way stand uncovered.
// Measured, two / three to a CU, in us, 32 q / 8 kv heads unless said: 64 workgroups (one sample of 180 tokens) 7.8 / 8.0, 256 (900)
// 21.9 / 23.0, 512 27.9 / 28.9, 640 31.7 / 32.5, 700 (28 / 4 heads) 47.7 / 48.3, 768 38.7 / 38.4 and (16 / 16 heads, samples of
// 256) 27.4 / 23.3, 800 39.4 / 38.2, 1 024 (two full rounds of two) 46.1 / 46.4, 1 504 65.5 / 64.5, 2 080 89.2 / 87.4, 2 800 (28 / 4) 167 /
// 161, 64 / 8 heads, one sample of 8 000 tokens 953 / 934; 16 384 tokens of packed moderate samples 172 / 166, 65 536 of long ones
// at 64 / 8 heads 4.40 / 4.22 ms.  Fewer than 64 tokens have no 64 rows for a clipped tile to stand for.
bool mfma_fwd_three(const AttnArgs& a) { return a.meta.T >= 64 && static_cast<int64_t>(a.meta.n_rows[kGridQ]) * a.Hq >= 768; }

int launch_mfma_fwd3(const AttnArgs& a, void* stream) {
    const unsigned grid = static_cast<unsigned>(a.meta.n_rows[kGridQ]) * a.Hq;
    if (grid == 0) return 0;
    psattn_fwd_bf16_mfma<128, true><<<grid, 256, 0, static_cast<hipStream_t>(stream)>>>(a);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
