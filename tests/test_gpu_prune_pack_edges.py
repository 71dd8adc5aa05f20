"""Device pruner and packer at the sizes where their kernels change path: segments around the register
limits of the selection (1024 and 4096 entries), widths with and without 16-byte mask rows, scores that
agree in all but their last bits (-m gpu)."""
import numpy as np
import pytest

import paper_2402_10876_amd as tw
from oracle import pack as opk
from oracle import prune as op
from tests.test_cabi_packer import _same
from tests.test_pack_dev import _pack_dev
from tests.test_prune_dev import _prune_on_device
import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [  # K, N, G, columns pruned, rows kept per tile
    (1024, 64, 64, 5, 300), (1025, 48, 32, 0, 256), (6, 4096, 128, 400, 4), (8, 4112, 64, 1, 8),
    (4100, 16, 32, 2, 1000), (33, 1040, 128, 1039, 1), (5, 17, 32, 3, 5), (64, 160, 32, 16, 32),
]


@pytest.mark.parametrize("K,N,G,cp,rk", CASES)
@pytest.mark.parametrize("pattern", ["tw", "tvw"])
def test_prune_then_pack_equals_oracle(K, N, G, cp, rk, pattern):
    B = wl.rng_fp16(K + N, (K, N), 0.5)
    pat = tw.PATTERN_TW if pattern == "tw" else tw.PATTERN_TVW
    print(f"case prune+pack {pattern} K={K} N={N} G={G} cp={cp} rk={rk}", flush=True)
    mask, tmask, _ = _prune_on_device(B, G, pat, cp, rk)
    want_t = op.tw(B, G, n_cols_pruned=cp, rows_kept_per_tile=rk, exact=True)
    want = op.vw24_condensed(B, want_t, G) if pattern == "tvw" else want_t
    assert np.array_equal(tmask, want_t) and np.array_equal(mask, want)
    tm = want_t if pattern == "tvw" else None
    p = _pack_dev(B, want, G, pat, tile_mask=tm)
    _same(p.export(), opk.ref_pack(B, want, G, pat, tile_mask=tm))
    p.free()


def test_scores_that_differ_in_the_last_bit_only():
    """Rows of equal sums but for one unit in the last place of one element: every digit of the
    threshold has to be followed, and what is equal to the end goes in index order."""
    K, N, G = 300, 32, 32
    B = np.full((K, N), 0.75, np.float16)
    up = np.random.default_rng(3).permutation(K)[:140]
    B[up, 5] = np.nextafter(np.float16(0.75), np.float16(1.0))
    mask, _, _ = _prune_on_device(B, G, tw.PATTERN_TW, 0, 200)
    want = op.tw(B, G, n_cols_pruned=0, rows_kept_per_tile=200, exact=True)
    assert want[up].all() and np.array_equal(mask, want)
