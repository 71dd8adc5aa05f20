"""Pipelined kernels that load the kept-row list two stages ahead, against the oracle: lists of no stage
up to seven (the loop runs in pairs and starts three loads early), tiles of different length in one launch,
every tile shape, and grids on both sides of the line between vector and scalar row loads (-m gpu)."""
import numpy as np
import pytest

import paper_2402_10876_amd as tw
from oracle import gemm as og
from tests.helpers import assert_C_close, random_tw_mask
from tests import gpu_util as gu
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_options():
    for name in ("tile_m", "ksplit", "idx_route"):
        tw.tw_set_option(name, 0)
    yield
    for name in ("tile_m", "ksplit", "idx_route"):
        tw.tw_set_option(name, 0)


def _uneven_tvw(rng, heights, G, N):
    """Tiles of G columns whose kept rows number heights[t]."""
    K = max(heights) + 3
    tmask, mask = np.zeros((K, N), np.uint8), np.zeros((K, N), np.uint8)
    for t, h in enumerate(heights):
        rows, cols = np.sort(rng.permutation(K)[:h]), np.arange(t * G, min((t + 1) * G, N))
        tmask[np.ix_(rows, cols)] = 1
        for q in range(0, h, 4):
            for c in cols:
                mask[rng.permutation(rows[q:q + 4])[:2], c] = 1
    return K, mask, tmask


@pytest.mark.parametrize("G,tile_m", [(128, 64), (128, 128), (128, 256), (64, 128)])
def test_tvw_lists_of_few_stages(G, tile_m):
    rng = np.random.default_rng(G + tile_m)
    heights = [64, 65, 130, 200, 256, 300, 384, 447, 3]
    N, M = G * len(heights) - 5, 2 * tile_m + 37
    K, mask, tmask = _uneven_tvw(rng, heights, G, N)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    print(f"case tvw row loads G={G} tile_m={tile_m}", flush=True)
    tw.tw_set_option("tile_m", tile_m)
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TVW, tile_mask=tmask)
    C, raw = gu.run_tw(tw, p, A, N, fill=5.0)
    p.free()
    assert_C_close(C, og.gemm_oracle(A, B, mask), og.abs_bound(A, B, mask))
    assert (raw[:, M:] == 5.0).all()


@pytest.mark.parametrize("pattern", ["tw", "tvw"])
@pytest.mark.parametrize("G,tile_m", [(128, 64), (128, 128), (64, 128)])
def test_i8_lists_of_few_stages(pattern, G, tile_m):
    rng = np.random.default_rng(7 * G + tile_m)
    heights = [128, 129, 260, 400, 512, 600, 800, 64, 3] if pattern == "tvw" else [64, 65, 130, 200, 256, 300, 384, 447, 3]
    N, M = G * len(heights) - 5, 2 * tile_m + 37
    K, mask, tmask = _uneven_tvw(rng, heights, G, N)
    A, B = wl.rng_i8(K, (M, K)), wl.rng_i8(K + 1, (K, N))
    print(f"case i8 row loads {pattern} G={G} tile_m={tile_m}", flush=True)
    tw.tw_set_option("tile_m", tile_m)
    if pattern == "tw":
        mask = tmask
        p = tw.tw_pack_i8(B, mask, G)
    else:
        p = tw.tw_pack_i8(B, mask, G, tw.PATTERN_TVW, tile_mask=tmask)
    for ksplit in ((0, 2) if pattern == "tw" else (0,)):
        tw.tw_set_option("ksplit", ksplit)
        C, raw = gu.run_tw_i8(tw, p, A, N)
        assert np.array_equal(C, og.gemm_i8_oracle(A, B, mask))
        assert (raw[:, M:] == -77).all()
    p.free()


@pytest.mark.parametrize("G,M,N", [(128, 4096, 2048), (128, 4224, 2048), (64, 4096, 1024), (64, 4224, 1024)])
def test_i8_both_sides_of_two_workgroups_per_CU(G, M, N):
    rng = np.random.default_rng(M + N)
    K = 150
    mask = random_tw_mask(rng, K, N, G, 1.0, 0.6)
    A, B = wl.rng_i8(M, (M, K)), wl.rng_i8(M + 1, (K, N))
    print(f"case i8 grid G={G} M={M} N={N}", flush=True)
    p = tw.tw_pack_i8(B, mask, G)
    C, _ = gu.run_tw_i8(tw, p, A, N)
    p.free()
    assert np.array_equal(C, og.gemm_i8_oracle(A, B, mask))


@pytest.mark.parametrize("G,tile_m", [(128, 128), (64, 256)])
def test_tw_scalar_and_vector_row_loads_agree(G, tile_m):
    rng = np.random.default_rng(G)
    heights = [32, 33, 70, 100, 128, 150, 200, 220, 3]
    N, M = G * len(heights) - 5, 2 * tile_m + 37
    K, _, mask = _uneven_tvw(rng, heights, G, N)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    print(f"case tw row loads G={G} tile_m={tile_m}", flush=True)
    tw.tw_set_option("tile_m", tile_m)
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TW)
    raws = []
    for route in (1, 2):
        tw.tw_set_option("idx_route", route)
        C, raw = gu.run_tw(tw, p, A, N, fill=5.0)
        assert_C_close(C, og.gemm_oracle(A, B, mask), og.abs_bound(A, B, mask))
        raws.append(raw.view(np.uint16))
    p.free()
    assert np.array_equal(raws[0], raws[1])
