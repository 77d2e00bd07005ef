// pdssm_project_rule.h -- which kernel takes a layer product, and the extent of
// the block that a wave of the 256 x 256 tiles stores.  Plain constexpr
// arithmetic without HIP, shared by the kernels, their launches and host-side
// checks.
#pragma once
#include <stdint.h>

namespace pdssm {

enum ProjectKernel {
    kProjectThin1,   // k_project_thin<1>: at most 32 tokens a workgroup
    kProjectThin2,   // k_project_thin<2>: at most 64
    kProjectDma128,  // k_project_dma<128>
    kProjectDma256,  // k_project_dma<256>
    kProjectWide,    // k_project_wide
};

// where k_project_thin and the 128-token tiles of k_project_dma cross (see
// k_project_thin)
constexpr int kThinTokens = 64;

// T tokens of contraction Dm; routing (H heads of K maps) when route, and nproj
// projections of 2HN rows.
constexpr ProjectKernel project_kernel(long long T, long long Dm, long long H, long long K, long long N, bool route,
                                       int nproj) {
    const long long R = 2 * H * N, HK = route ? H * K : 0, hpb = route ? 256 / K : 1;
    const long long NT = (route ? (H + hpb - 1) / hpb : 0) + nproj * ((R + 255) / 256);
    const long long tiles256 = (T + 255) / 256 * NT;
    const bool below = ((R > HK ? R : HK) + 256) * Dm * 2 < (1LL << 31) && Dm < (1 << 20);  // weights below 2 GiB
    if (T <= kThinTokens && K <= 128 && below) return T <= 32 ? kProjectThin1 : kProjectThin2;
    // 256-token tiles when they still give every CU two of them
    if (tiles256 < 512) return kProjectDma128;
    // k_project_wide gains with every slice of the contraction and in the
    // projections' epilogue; its routing tiles' epilogue, with logits, costs
    // more than k_project_dma<256>'s, and a tile of few columns all of a tile's
    // products.  Time of k_project_dma<256> over k_project_wide's with logits, P
    // projection columns for each routing column:
    //   R < 64: 0.56-0.72 at Dm 32, 0.89-0.96 at 512, 0.97-1.03 beyond;
    //   R = 64, P 12 / 96: 0.86 / 0.87 at 32, 0.95 / 0.96 at 64, 1.02 / 1.03 at 128;
    //   P 4-8: 0.84-0.91 at 32, 0.90-1.02 at 64, 0.97-1.13 at 128, 1.04-1.25 at
    //     192 (of R 1024, 2048), 1.28 and more at 1024;
    //   P 9-16: 0.85-0.98 at 32, 0.92-1.05 at 64, 0.98-1.12 at 128;
    //   P 19 and more, R >= 128: 0.92 (a 7.03 rounds' tail), 1.02-1.36 at 32,
    //     1.00-1.47 at 64, 1.02-1.44 at 96.
    const long long P = HK ? nproj * R / HK : 1 << 20;
    const bool pays = R >= 64 && (Dm >= 192 ? P >= 4 : Dm >= 128 ? P >= 8 : R >= 128 && P >= 19);
    return below && R < (1 << 20) && nproj * R >= 4 * HK && pays ? kProjectWide : kProjectDma256;
}

// k_project_wide: a wave's block of 128 tokens x 128 columns of an output of R
// columns starts at column cr (past the last one in the second half of a tile
// whose remainder fits the first).
constexpr int wide_cols(int R, int cr) { return R <= cr ? 0 : R - cr < 128 ? R - cr : 128; }
// Bytes from the block's first entry to the end of its last token's last
// column: nothing of a block without tokens or columns.
constexpr uint32_t wide_block_bytes(int nt, int R, int ncol) {
    return nt <= 0 || ncol <= 0 ? 0u : ((uint32_t)(nt - 1) * (uint32_t)R + (uint32_t)ncol) * 4u;
}
// Byte offset of a lane's entries at column c of token row: one past the block's
// columns lies beyond every block (at most 2^29 bytes: R < 2^20), as do rows
// past its last token.
constexpr uint32_t kWidePast = 0xc0000000u;
constexpr uint32_t wide_pair_offset(int row, int c, int R, int ncol) {
    return c < ncol ? (uint32_t)(row * R + c) * 4u : kWidePast + (uint32_t)(row * R) * 4u;
}

}  // namespace pdssm
