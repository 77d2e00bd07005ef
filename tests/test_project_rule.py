"""Host checks of the layer product's dispatch rule and of the store extents of
its 256 x 256 tiles (csrc/pdssm_project_rule.h, compiled for the CPU)."""
import numpy as np
import pytest

from helpers import project_rule

CAP = 1 << 32  # byte offsets of a store are 32-bit


@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256])
def test_wide_store_extent(N):
    """Every remainder of the tokens (0 .. 128 of a wave's block) and every
    output width: each store that the descriptor lets through lands on a row
    and column of the block's own, and those are all let through."""
    rule = project_rule()
    tokens = np.arange(0, 129)
    rows = np.arange(128)
    for H in list(range(1, 33)) + [100, 2047]:
        R = 2 * H * N
        if R >= 1 << 20:
            continue
        for tile in {0, (R + 255) // 256 - 1}:
            for half in (0, 1):
                cr = 256 * tile + 128 * half
                ncol = rule.wide_cols(R, cr)
                assert ncol == min(max(R - cr, 0), 128), (R, cr)
                size = np.array([rule.wide_block_bytes(int(nt), R, ncol) for nt in tokens], np.int64)
                # never past the end of the rows that are left of the output
                assert (size <= np.maximum(tokens * R - cr, 0) * 4).all(), (R, cr)
                for c in (0, 2, max(ncol - 2, 0), ncol, 126):
                    first = rule.wide_pair_offset(0, c, R, ncol)
                    at = first + rows.astype(np.int64) * R * 4
                    assert at[-1] + 8 <= CAP
                    assert rule.wide_pair_offset(127, c, R, ncol) == at[-1]
                    passes = at[None, :] + 8 <= size[:, None]          # [tokens, rows]
                    inside = (rows[None, :] < tokens[:, None]) & (c < ncol)
                    np.testing.assert_array_equal(passes, inside, "R %d cr %d c %d" % (R, cr, c))


def test_project_kernel_rule():
    """The rule at its lines: 32, 64 tokens and K = 128; 512 tiles; the shares of
    projections and routing; few columns; weights of 2 GiB."""
    k = project_rule().kernel
    layer = dict(Dm=1024, H=16, K=16, N=64)
    assert [k(T=T, **layer) for T in (1, 32, 33, 64, 65)] == ["thin1", "thin1", "thin2", "thin2", "dma128"]
    assert k(T=1, Dm=64, H=2, K=128, N=8) == "thin1" and k(T=1, Dm=64, H=2, K=129, N=8) == "dma128"
    # 25 column tiles: 21 token tiles make 525
    assert k(T=20 * 256, **layer) == "dma128" and k(T=20 * 256 + 1, **layer) == "wide"
    # projection columns for each routing column, by the contraction's length
    big = dict(T=1 << 17, H=8, N=8)  # 3 R = 384
    for Dm, K in ((4096, 12), (192, 12), (160, 6), (128, 6), (96, 2), (32, 2)):
        assert k(Dm=Dm, K=K, **big) == "wide" and k(Dm=Dm, K=K + 1, **big) == "dma256", (Dm, K)
    assert k(T=1 << 17, Dm=1024, H=8, K=16, N=8, nproj=0) == "dma256"
    assert k(T=1 << 17, Dm=64, H=8, K=1, N=8, route=False, nproj=1) == "wide"
    # few columns
    assert [k(T=1 << 17, Dm=4096, H=H, K=1, N=8) for H in (3, 4)] == ["dma256", "wide"]
    assert [k(T=1 << 17, Dm=96, H=H, K=1, N=8) for H in (7, 8)] == ["dma256", "wide"]
    # rows (and 256 more) of 2 GiB
    assert k(T=1, Dm=16384, H=254, K=1, N=128) == "thin1" and k(T=1, Dm=16384, H=255, K=1, N=128) == "dma256"
