"""Launches with few output blocks (the kernel whose waves share out a column block's k-steps) against
the oracle at its edges: M around the 32-row block, kept-row lists around one k-step per wave, one round
of a wave's k-steps and several, empty tiles, all tile widths, M on both sides of the line where the
pipelined kernels take over (-m gpu)."""
import numpy as np
import pytest

import paper_2402_10876_amd as tw
from oracle import gemm as og
from tests.helpers import assert_C_close, random_tw_mask, random_tvw_mask
from tests import gpu_util as gu
import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [  # pattern, M, K, N, G, col_keep, row_keep
    ("tw", 1, 2, 1, 32, 1.0, 0.6), ("tw", 8, 128, 64, 64, 0.9, 1.0), ("tw", 31, 129, 33, 32, 0.9, 1.0),
    ("tw", 32, 512, 129, 128, 0.9, 1.0), ("tw", 33, 513, 300, 128, 0.8, 1.0), ("tw", 95, 1024, 130, 64, 0.9, 1.0),
    ("tw", 7, 1040, 500, 128, 0.5, 1.0), ("tw", 65, 2500, 700, 32, 0.9, 0.6), ("tw", 130, 768, 2304, 128, 0.9, 0.28),
    ("tw", 200, 300, 500, 64, 0.9, 0.01), ("tw", 577, 256, 256, 64, 0.9, 0.5), ("tw", 2080, 100, 120, 64, 0.9, 0.5),
    ("tw", 640, 768, 768, 128, 0.9, 0.28), ("tw", 704, 768, 768, 128, 0.9, 0.28),
    ("tvw", 1, 4, 1, 64, 1.0, 1.0), ("tvw", 31, 256, 65, 64, 1.0, 1.0), ("tvw", 33, 384, 129, 128, 0.9, 1.0),
    ("tvw", 40, 385, 300, 128, 0.8, 1.0), ("tvw", 64, 1100, 257, 64, 0.9, 1.0), ("tvw", 97, 2100, 600, 128, 0.9, 0.7),
    ("tvw", 520, 768, 700, 128, 0.9, 0.5), ("tvw", 290, 768, 3072, 128, 0.9, 0.25), ("tvw", 60, 200, 300, 64, 0.9, 0.02),
]


@pytest.mark.parametrize("pattern,M,K,N,G,col_keep,row_keep", CASES)
def test_few_blocks_edges(pattern, M, K, N, G, col_keep, row_keep):
    rng = np.random.default_rng(M * 7919 + K + N)
    if pattern == "tw":
        mask = tmask = random_tw_mask(rng, K, N, G, col_keep, row_keep)
    else:
        mask, tmask = random_tvw_mask(rng, K, N, G, col_keep, row_keep, full=False)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    print(f"case few blocks {pattern} M={M} K={K} N={N} G={G} keep={col_keep}/{row_keep}", flush=True)
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TW if pattern == "tw" else tw.PATTERN_TVW, tile_mask=tmask)
    lda, ldc = (M + 7) // 8 * 8 + 8, (M + 7) // 8 * 8 + 16
    C, raw = gu.run_tw(tw, p, A, N, lda=lda, ldc=ldc, fill=5.0)
    C2, raw2 = gu.run_tw(tw, p, A, N, lda=lda, ldc=ldc, fill=5.0)
    p.free()
    assert_C_close(C, og.gemm_oracle(A, B, mask), og.abs_bound(A, B, mask))
    assert not raw[~mask.any(0)][:, :M].view(np.uint16).any()          # pruned columns: exactly +0
    assert (raw[:, M:] == 5.0).all()                                   # nothing written past row M
    assert np.array_equal(raw.view(np.uint16), raw2.view(np.uint16))   # partial sums in a fixed order


def test_tvw_width_32_stays_refused():
    mask = np.zeros((8, 32), np.uint8)
    mask[:2] = 1
    p = tw.tw_pack(np.ones((8, 32), np.float16), mask, 32, tw.PATTERN_TVW, tile_mask=np.ones((8, 32), np.uint8))
    with pytest.raises(tw.TwError) as ei:
        gu.run_tw(tw, p, np.ones((8, 8), np.float16), 32)
    assert ei.value.status == 3
    p.free()


I8_CASES = [  # pattern, M, K, N, G, col_keep, row_keep, c_dtype
    ("tw", 1, 2, 1, 64, 1.0, 0.6, 0), ("tw", 15, 128, 64, 64, 0.9, 1.0, 1), ("tw", 31, 513, 129, 128, 0.9, 1.0, 0),
    ("tw", 33, 520, 300, 128, 0.8, 1.0, 1), ("tw", 97, 1500, 130, 64, 0.9, 1.0, 0), ("tw", 200, 300, 500, 64, 0.9, 0.01, 1),
    ("tw", 130, 768, 2304, 128, 0.9, 0.28, 1), ("tw", 700, 100, 70, 64, 0.9, 0.5, 0), ("tw", 704, 256, 1000, 128, 0.9, 0.5, 1),
    ("tvw", 1, 4, 1, 64, 1.0, 1.0, 1), ("tvw", 16, 256, 65, 64, 1.0, 1.0, 0), ("tvw", 47, 1030, 300, 128, 0.8, 1.0, 1),
    ("tvw", 64, 2100, 257, 64, 0.9, 1.0, 0), ("tvw", 290, 768, 600, 128, 0.9, 0.25, 1), ("tvw", 60, 200, 300, 64, 0.9, 0.02, 0),
    ("tvw", 1300, 500, 60, 64, 0.9, 0.5, 1),
]


@pytest.mark.parametrize("pattern,M,K,N,G,col_keep,row_keep,c_dtype", I8_CASES)
def test_few_blocks_i8_edges(pattern, M, K, N, G, col_keep, row_keep, c_dtype):
    """Sums are whole numbers: the same as the oracle's, and as the pipelined kernels' (which a forced tile size takes)."""
    rng = np.random.default_rng(M * 7919 + K + N)
    if pattern == "tw":
        mask = tmask = random_tw_mask(rng, K, N, G, col_keep, row_keep)
    else:
        mask, tmask = random_tvw_mask(rng, K, N, G, col_keep, row_keep, full=False)
    A, B, scale = wl.rng_i8(K, (M, K)), wl.rng_i8(K + 1, (K, N)), 1.0 / 331.0
    print(f"case few blocks i8 {pattern} M={M} K={K} N={N} G={G} keep={col_keep}/{row_keep} out={c_dtype}", flush=True)
    p = tw.tw_pack_i8(B, mask, G, tw.PATTERN_TW if pattern == "tw" else tw.PATTERN_TVW, tile_mask=tmask)
    lda, ldc = (M + 15) // 16 * 16 + 16, (M + 15) // 16 * 16 + 32
    C, raw = gu.run_tw_i8(tw, p, A, N, c_dtype=c_dtype, scale=scale, lda=lda, ldc=ldc)
    tw.tw_set_option("tile_m", 128)
    try:
        C2, _ = gu.run_tw_i8(tw, p, A, N, c_dtype=c_dtype, scale=scale, lda=lda, ldc=ldc)
    finally:
        tw.tw_set_option("tile_m", 0)
    p.free()
    want = og.gemm_i8_oracle(A, B, mask)
    if c_dtype:
        want = og.requantize_i8(want, scale).astype(np.int64)
    assert np.array_equal(C, want) and np.array_equal(C2, want)
    assert (raw[:, M:] == -77).all()                                   # nothing written past row M
