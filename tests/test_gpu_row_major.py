"""Row-major activations and outputs (TW_LAYOUT_MK) against the oracle at the edges of the kernel's
bands: K around one and two bands of 768 columns, M around the 64- and 32-row bands, column ranges of a tile
wider than one staged segment, tile widths 32, 64 and 128 (-m gpu)."""
import numpy as np
import pytest

import paper_2402_10876_amd as tw
from oracle import gemm as og
from tests.helpers import assert_C_close, random_tw_mask
from tests import gpu_util as gu
import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [  # M, K, N, G, col_keep, row_keep
    (1, 1, 1, 32, 1.0, 1.0), (1, 767, 130, 128, 0.9, 0.3), (63, 768, 384, 128, 0.9, 0.25),
    (64, 769, 257, 64, 0.9, 0.5), (65, 1535, 300, 32, 0.8, 0.6), (130, 1536, 640, 128, 0.3, 0.9),
    (200, 1537, 400, 64, 0.2, 0.05), (70, 2500, 900, 128, 0.9, 1.0), (129, 800, 2048, 128, 0.1, 0.02),
    (66, 3072, 768, 128, 0.9, 0.28), (1000, 96, 1200, 32, 0.9, 0.4), (5, 40, 700, 64, 0.02, 0.1),
    # 64-row bands (more than 128 blocks of them, lists of more than 96 rows), and 32-row ones by short lists
    (1665, 768, 1300, 128, 0.9, 0.25), (1727, 769, 1300, 128, 0.9, 0.4), (1700, 1537, 1300, 64, 0.9, 0.2),
    (1100, 767, 2300, 32, 0.9, 0.3), (1090, 513, 2300, 64, 0.9, 0.5), (2100, 700, 1300, 128, 0.9, 0.12),
    (33, 1024, 257, 64, 0.9, 0.5), (31, 767, 257, 64, 0.9, 0.5),
]


@pytest.mark.parametrize("M,K,N,G,col_keep,row_keep", CASES)
def test_row_major_edges(M, K, N, G, col_keep, row_keep):
    rng = np.random.default_rng(M * 7919 + K)
    mask = random_tw_mask(rng, K, N, G, col_keep, row_keep)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    print(f"case row-major M={M} K={K} N={N} G={G} keep={col_keep}/{row_keep}", flush=True)
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TW)
    ldc = (N + 7) // 8 * 8 + 8
    C, raw = gu.run_tw_mk(tw, p, A, N, ldc=ldc, fill=5.0)
    p.free()
    assert_C_close(C, og.gemm_oracle(A, B, mask), og.abs_bound(A, B, mask))
    assert not raw[:, :N][:, ~mask.any(0)].view(np.uint16).any()       # pruned columns: exactly +0
    assert (raw[:, N:] == 5.0).all()                                   # nothing written past column N


@pytest.mark.parametrize("M,K,N,G,lda", [(64, 64, 256, 128, 1024), (33, 61, 300, 64, 808), (70, 769, 257, 64, 4096),
                                         (1665, 700, 1300, 128, 1472), (130, 1537, 640, 128, 2048)])
def test_A_is_the_last_columns_of_a_wider_buffer(M, K, N, G, lda):
    """lda > K and A's last row ends where the buffer ends; everything around A is NaN."""
    import torch
    rng = np.random.default_rng(M + K)
    mask = random_tw_mask(rng, K, N, G, 0.9, 0.4)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    print(f"case row-major slice M={M} K={K} N={N} G={G} lda={lda}", flush=True)
    at = lda - (K + 7) // 8 * 8
    wide = torch.full((M, lda), float("nan"), dtype=torch.float16, device="cuda")
    wide[:, at:at + K] = torch.from_numpy(A).cuda()
    ldc = (N + 7) // 8 * 8
    C = torch.full((M, ldc), 5.0, dtype=torch.float16, device="cuda")
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TW)
    tw.tw_gemm(wide.data_ptr() + 2 * at, M, lda, tw.LAYOUT_MK, p, C.data_ptr(), ldc, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    p.free()
    got = C.cpu().numpy()
    assert_C_close(got[:, :N].astype(np.float64), og.gemm_oracle(A, B, mask), og.abs_bound(A, B, mask))
    assert (got[:, N:] == 5.0).all()


@pytest.mark.parametrize("M,K,N,G,lda", [(33, 96, 200, 64, 70_000_000), (64, 200, 33200, 128, (1 << 25) + 8), (33, 1600, 200, 128, 70_000_000),
                                         (64, 200, 33200, 128, 1 << 25)])       # the last one within 32 bits, 64-row bands
def test_last_row_of_a_band_past_32_bits(M, K, N, G, lda):
    """The band's last row starts up to 2^32 bytes and more behind its first: A is a column slice of 4.5 GB."""
    import torch
    mask = random_tw_mask(np.random.default_rng(5), K, N, G, 1.0, 0.6)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    print(f"case row-major M={M} N={N} lda={lda}", flush=True)
    wide = torch.empty((M, lda), dtype=torch.float16, device="cuda")
    wide[:, :K] = torch.from_numpy(A).cuda()
    C = torch.full((M, N), 5.0, dtype=torch.float16, device="cuda")
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TW)
    tw.tw_gemm(wide.data_ptr(), M, lda, tw.LAYOUT_MK, p, C.data_ptr(), N, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    p.free()
    del wide
    torch.cuda.empty_cache()
    assert_C_close(C.cpu().numpy().astype(np.float64), og.gemm_oracle(A, B, mask), og.abs_bound(A, B, mask))


@pytest.mark.parametrize("M,K,N,G,row_keep", [(40, 1537, 300, 128, 0.3), (130, 3072, 640, 64, 0.05), (33, 1537, 200, 32, 1.0),
                                              (1700, 1537, 1300, 64, 0.2), (1665, 3072, 1300, 128, 0.3)])
def test_infinite_weights_at_the_ends_of_the_bands(M, K, N, G, row_keep):
    """K in several bands: an infinite weight beside a band's end gives the infinity that its column's sum is, and
    infinite activations likewise; no other column changes."""
    import torch
    rng = np.random.default_rng(M + K + G)
    mask = random_tw_mask(rng, K, N, G, 0.9, row_keep)
    A, B = wl.make_A(K, M, K), wl.make_B(K, K, N, 0.1)
    A = np.where(A == 0, np.float16(0.5), A)
    B = np.where(B == 0, np.float16(0.5), B)
    cols = np.flatnonzero(mask.any(0))
    ends = [e for e in range(256, K, 256)]                       # every band end of 512 and 768 columns among them
    for i, c in enumerate(cols):                                 # one per column, within three kept rows of an end
        kept = np.flatnonzero(mask[:, c])
        at = np.searchsorted(kept, ends[i % len(ends)]) + i % 7 - 3
        if i % 3 and 0 <= at < len(kept):
            B[kept[at], c] = np.inf * (-1) ** i
    tail = {int(np.flatnonzero(mask[:, c])[-1]) for c in cols}   # (a padded list repeats its last row with weights of 0)
    free = [k for k in np.flatnonzero(mask.any(1)) if k not in tail and not np.isinf(B[k]).any()]
    A[M // 2, free[len(free) // 2]] = np.inf
    print(f"case row-major infinities M={M} K={K} N={N} G={G} keep={row_keep}", flush=True)
    p = tw.tw_pack(B, mask, G, tw.PATTERN_TW)
    C, raw = gu.run_tw_mk(tw, p, A, N)
    # the same weight packed on the device, and as the second of two joined ones
    Bd, md = torch.from_numpy(B).cuda(), torch.from_numpy(mask).cuda()
    q = tw.tw_pack_dev(Bd.data_ptr(), N, md.data_ptr(), 0, K, N, G, tw.PATTERN_TW, torch.cuda.current_stream().cuda_stream)
    one = tw.tw_pack(np.where(np.isinf(B), np.float16(1), B)[:, :64], mask[:, :64], G, tw.PATTERN_TW)
    both = tw.tw_concat([one, q])
    assert np.array_equal(gu.run_tw_mk(tw, q, A, N)[1].view(np.uint16), raw.view(np.uint16))
    D = gu.run_tw_mk(tw, both, A, N + 64)[0][:, 64:]
    assert np.array_equal(np.isnan(D), np.isnan(C)) and np.array_equal(np.isinf(D), np.isinf(C))
    for x in (p, q, one, both):
        x.free()
    rows = np.unique(np.r_[0:8, M // 2 - 2:M // 2 + 3, M - 8:M])
    A, C, kept = A[rows], C[rows], mask != 0
    with np.errstate(invalid="ignore"):
        want = np.stack([(A[:, kept[:, n]].astype(np.float64) * B[kept[:, n], n].astype(np.float64)).sum(1) for n in range(N)], 1)
    inf, nan = np.isinf(want), np.isnan(want)
    assert inf.sum() > len(rows) * len(cols) // 4
    assert np.array_equal(np.isnan(C), nan) and np.array_equal(C[inf], want[inf])
    fin = ~(inf | nan)
    Af, Bf = np.where(np.isfinite(A), A, 0).astype(np.float16), np.where(np.isfinite(B), B, 0).astype(np.float16)
    S = og.abs_bound(Af, Bf, mask)
    assert_C_close(np.where(fin, C, 0), np.where(fin, want, 0), S)
