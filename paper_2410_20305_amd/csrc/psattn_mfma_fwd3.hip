// bf16 MFMA forward at head_dim 128 with three workgroups to a CU (psattn_mfma_fwd.h), built without NaNs to honour like the one with two.
#include "psattn_mfma_fwd.h"

namespace psattn {

// From the grid on that fills the chip once with three workgroups to a CU; below, the second barrier and V's way stand uncovered.
// Measured, two / three to a CU, in us, 32 q / 8 kv heads unless said: 64 workgroups (one sample of 180 tokens) 7.8 / 8.0, 256 (900)
// 21.9 / 23.0, 512 27.9 / 28.9, 640 31.7 / 32.5, 700 (28 / 4 heads) 47.7 / 48.3, 768 38.7 / 38.4 and (16 / 16 heads, samples of
// 256) 27.4 / 23.3, 800 39.4 / 38.2, 1 024 (two full rounds of two) 46.1 / 46.4, 1 504 65.5 / 64.5, 2 080 89.2 / 87.4, 2 800 (28 / 4) 167 /
// 161, 64 / 8 heads, one sample of 8 000 tokens 953 / 934; 16 384 tokens of packed moderate samples 172 / 166, 65 536 of long ones
// at 64 / 8 heads 4.40 / 4.22 ms.  Fewer than 64 tokens have no 64 rows for a clipped tile to stand for.
// Not where the launch is bound by a few long rows: the third workgroup takes its part of the CU while the longest row is still
// at work.  The line: rows of 12 and more k-tiles, the longest over 0.85 times a slot's share of all k-tiles.  Both forwards on 1 977
// random tables past the other two lines, three over two, mean and range by that ratio: rows under 12 tiles, any ratio, 0.96 (0.81 - 1.10, 2 %
// of them over 1.02); longer ones up to 0.85 0.99 (0.90 - 1.07), 0.85 - 1.1 0.99 (0.91 - 1.05), 1.1 - 1.5 1.01 (0.95 - 1.06), 1.5 - 2 1.03 (0.93 -
// 1.12), over 2 1.09 (1.03 - 1.14).  16 / 16 heads, one sample of 6 040 tokens 160 / 171.
constexpr bool three_to_a_cu(int32_t T, int64_t workgroups, int64_t longest, int64_t tiles) {
    return T >= 64 && workgroups >= 768 && (longest < 12 || 100 * 768 * longest <= 85 * tiles);
}

bool mfma_fwd_three(const AttnArgs& a) {
    return three_to_a_cu(a.meta.T, static_cast<int64_t>(a.meta.n_rows[kGridQ]) * a.Hq, a.size[kGridQ].longest, a.size[kGridQ].n_entries * a.Hq);
}

int launch_mfma_fwd3(const AttnArgs& a, void* stream) {
    const unsigned grid = static_cast<unsigned>(a.meta.n_rows[kGridQ]) * a.Hq;
    if (grid == 0) return 0;
    psattn_fwd_bf16_mfma<128, true><<<grid, 256, 0, static_cast<hipStream_t>(stream)>>>(a);
    return static_cast<int>(hipGetLastError());
}

}  // namespace psattn
