"""Device pruner and packer at the sizes where their kernels change path: segments around the register
limits of the selection (1024 and 4096 entries), widths with and without 16-byte mask rows, masks at any
address, a tile that answers for very many columns, counts that fill more than one block of host memory, several
threads at once, scores that agree in all but their last bits (-m gpu)."""
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
    (600, 3008, 32, 8, 557), (601, 3001, 32, 1, 558), (400, 6016, 128, 0, 390), (130, 9000, 64, 8950, 20), (1, 1, 32, 0, 1), (130, 3, 64, 1, 70), (4097, 5, 128, 0, 4097), (2, 9000, 64, 8990, 1), (70, 143, 128, 143, 5),
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


@pytest.mark.parametrize("K,N,G,at,tile_at", [(37, 77, 32, 0, 0), (37, 77, 32, 3, 3), (64, 96, 32, 5, 12), (20, 200, 128, 15, 0)])
def test_masks_at_any_address(K, N, G, at, tile_at):
    """Masks that start `at` bytes behind a 16-byte boundary: what lies around them stays as it was, and they pack."""
    import torch
    B = wl.rng_fp16(K * N, (K, N), 0.5)
    rk = K // 3
    Bd = torch.from_numpy(B).cuda()
    buf = [torch.full((K * N + 64,), 7, dtype=torch.uint8, device="cuda") for _ in range(2)]
    md, td = buf[0][at:at + K * N], buf[1][tile_at:tile_at + K * N]
    ws = torch.empty(tw.tw_prune_workspace_bytes(K, N, G), dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    print(f"case mask address K={K} N={N} at={at},{tile_at}", flush=True)
    tw.tw_prune_dev(Bd.data_ptr(), K, N, N, G, tw.PATTERN_TVW, N // 8, rk, md.data_ptr(), td.data_ptr(), ws.data_ptr(),
                    ws.numel(), st)
    torch.cuda.synchronize()
    want_t = op.tw(B, G, n_cols_pruned=N // 8, rows_kept_per_tile=rk, exact=True)
    want = op.vw24_condensed(B, want_t, G)
    assert np.array_equal(md.cpu().numpy().reshape(K, N), want) and np.array_equal(td.cpu().numpy().reshape(K, N), want_t)
    for b, a in zip(buf, (at, tile_at)):
        assert (b[:a] == 7).all() and (b[a + K * N:] == 7).all()
    p = tw.tw_pack_dev(Bd.data_ptr(), N, md.data_ptr(), td.data_ptr(), K, N, G, tw.PATTERN_TVW, st)
    _same(p.export(), opk.ref_pack(B, want, G, opk.PATTERN_TVW, tile_mask=want_t))
    p.free()


@pytest.mark.parametrize("N", [20000, 90000])
def test_a_tile_of_very_many_columns(N):
    """100 kept columns: the last tile answers for all columns from 9000 on, shared by several workgroups, 90000 are more than
    its bits in LDS hold."""
    K, G = 6, 32
    B = np.zeros((K, N), np.float16)
    cols = np.r_[5:90, 9000:9015]
    B[:, cols] = wl.rng_fp16(1, (K, len(cols)), 0.5)
    B[:, cols] += np.sign(B[:, cols])
    mask, tmask, _ = _prune_on_device(B, G, tw.PATTERN_TVW, N - len(cols), 5)
    want_t = op.tw(B, G, n_cols_pruned=N - len(cols), rows_kept_per_tile=5, exact=True)
    want = op.vw24_condensed(B, want_t, G)
    assert np.array_equal(tmask, want_t) and np.array_equal(mask, want)
    p = _pack_dev(B, want, G, tw.PATTERN_TVW, tile_mask=want_t)
    _same(p.export(), opk.ref_pack(B, want, G, opk.PATTERN_TVW, tile_mask=want_t))
    p.free()


@pytest.mark.parametrize("K,N,G", [(4200, 3200, 32), (40, 90000, 32)])   # 66 x 100 counts; tables of 2813 tiles: a block of its own
def test_more_counts_than_one_block_of_host_memory(K, N, G):
    rng = np.random.default_rng(0)
    keep = rng.random((K, -(-N // G))) < 0.03
    mask = np.repeat(keep, G, axis=1)[:, :N].astype(np.uint8)
    mask[0] = 1
    B = wl.rng_fp16(3, (K, N))
    p, h = _pack_dev(B, mask, G, tw.PATTERN_TW), tw.tw_pack_host(B, mask, G, tw.PATTERN_TW)
    _same(p.export(), h.export())
    assert p.flop_counts() == h.flop_counts()
    p.free()
    h.free()


@pytest.mark.parametrize("K,N,G,pattern", [(1025, 70, 64, "tw"), (5000, 130, 32, "tvw"), (20011, 64, 64, "tw"), (2049, 700, 128, "tvw"),
                                           (17000, 17, 32, "tw")])
def test_tall_weights_in_slices(K, N, G, pattern):
    """Narrow and tall: the columns' bits come from several slices of the rows, a column from one of them or a few."""
    rng = np.random.default_rng(K + N)
    B = wl.rng_fp16(K, (K, N))
    tm = np.zeros((K, N), np.uint8)
    cols = np.sort(rng.choice(N, max(1, N * 2 // 3), replace=False))
    for t in range(0, len(cols), G):
        at = rng.integers(0, K, 5)                                   # rows of a tile in few places, the ends among them
        rows = np.unique(np.concatenate([at, (at + 1) % K, [0, K - 1] if t == 0 else at]))
        tm[np.ix_(rows, cols[t:t + G])] = 1
    mask, tile_mask, P = tm, None, tw.PATTERN_TW
    if pattern == "tvw":                                             # two of four: the first two rows of every group
        mask, tile_mask, P = np.zeros_like(tm), tm, tw.PATTERN_TVW
        for t in range(0, len(cols), G):
            rows = np.flatnonzero(tm[:, cols[t]])
            mask[np.ix_(rows[np.arange(len(rows)) % 4 < 2], cols[t:t + G])] = 1
    p = _pack_dev(B, mask, G, P, tile_mask=tile_mask)
    h = tw.tw_pack_host(B, mask, G, P, tile_mask=tile_mask)
    _same(p.export(), h.export())
    assert p.flop_counts() == h.flop_counts()
    p.free()
    h.free()


@pytest.mark.parametrize("K,N,G,cp,rk,pattern", [
    (4095, 66, 64, 3, 900, "tw"), (4096, 64, 64, 0, 1300, "tw"), (4097, 130, 32, 20, 700, "tvw"), (9001, 33, 32, 1, 4000, "tvw"),
    (40000, 5, 32, 1, 13, "tw"), (70, 8129, 128, 3000, 20, "tvw"), (33, 8128, 64, 5000, 9, "tw")])
def test_tall_weights_are_scored_in_slices(K, N, G, cp, rk, pattern):
    """Around the lines where columns are scored in slices and in whole lines of memory, with values on both sides of 1 (sums of 64 and of 128 bits)."""
    B = wl.rng_fp16(K + N, (K, N), 0.5)
    B[::37] *= np.float16(40)
    print(f"case tall prune {pattern} K={K} N={N} G={G} cp={cp} rk={rk}", flush=True)
    mask, tmask, _ = _prune_on_device(B, G, tw.PATTERN_TVW if pattern == "tvw" else tw.PATTERN_TW, cp, rk, ldb=N + 3)
    want_t = op.tw(B, G, n_cols_pruned=cp, rows_kept_per_tile=rk, exact=True)
    assert np.array_equal(tmask, want_t)
    assert np.array_equal(mask, op.vw24_condensed(B, want_t, G) if pattern == "tvw" else want_t)


@pytest.mark.parametrize("pattern,K,N,rk", [("tw", 5003, 3072, 2000), ("tvw", 5003, 3072, 2000), ("tvw", 1100, 4500, 500)])
def test_many_rows_for_each_workgroup_of_the_masks(pattern, K, N, rk):
    """2560 rows for a workgroup, or all of a tile, which are divided again; the selection as a whole is compared with one on the host in integers."""
    import torch
    G = 32
    q = torch.randint(-7, 8, (K, N), generator=torch.Generator().manual_seed(5), dtype=torch.int8)
    q[:, 0::2] *= 2
    B = (q.to(torch.float16) / 16).numpy()
    print(f"case masks with many rows {pattern} K={K} N={N}", flush=True)
    mask, tmask, _ = _prune_on_device(B, G, tw.PATTERN_TVW if pattern == "tvw" else tw.PATTERN_TW, 5, rk)
    sq = q.to(torch.int32) ** 2
    cols = torch.sort(torch.argsort(sq.sum(0), stable=True)[5:]).values
    want_t = np.zeros((K, N), np.uint8)
    want = np.zeros((K, N), np.uint8)
    for t in range(0, len(cols), G):
        c = cols[t:t + G]
        rows = torch.sort(torch.argsort(sq[:, c].sum(1), stable=True)[K - rk:]).values
        want_t[np.ix_(rows.numpy(), c.numpy())] = 1
        v = sq[rows][:, c].reshape(rk // 4, 4, len(c))                        # of four, the two largest; equal: the lower position
        two = torch.argsort(v, dim=1, descending=True, stable=True)[:, :2]
        keep = torch.zeros(v.shape, dtype=torch.uint8).scatter_(1, two, 1).reshape(rk, len(c))
        want[np.ix_(rows.numpy(), c.numpy())] = keep.numpy()
    assert np.array_equal(tmask, want_t) and np.array_equal(mask, want if pattern == "tvw" else want_t)


def test_several_threads_pack_at_once():
    """More threads than blocks of host memory are kept, each on a stream of its own, over and over."""
    import threading
    import torch
    rng = np.random.default_rng(1)
    jobs = []
    for i in range(6):
        K, N, G = 100 + 37 * i, 90 + 51 * i, 32
        keep = rng.random((K, (N + G - 1) // G)) < 0.4
        keep[0] = True
        mask = np.repeat(keep, G, axis=1)[:, :N].astype(np.uint8)
        B = wl.rng_fp16(i, (K, N))
        jobs.append((B, mask, G, opk.ref_pack(B, mask, G, opk.PATTERN_TW)))
    errors = []

    def work(B, mask, G, want):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(5):
                    p = _pack_dev(B, mask, G, tw.PATTERN_TW)
                    _same(p.export(), want)
                    p.free()
        except Exception as e:                                       # noqa: BLE001 (handed to the main thread)
            errors.append(e)
    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("mode", ["relaxed", "thread_local", "global"])
def test_packing_while_the_stream_is_captured_is_an_error(mode):
    """Refused before anything is allocated: outside the relaxed mode an allocation would end the caller's capture."""
    import torch
    B, mask = wl.rng_fp16(0, (64, 64)), np.ones((64, 64), np.uint8)
    Bd, md, x = torch.from_numpy(B).cuda(), torch.from_numpy(mask).cuda(), torch.zeros(8, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode=mode):
        x += 1
        with pytest.raises(tw.TwError) as ei:
            tw.tw_pack_dev(Bd.data_ptr(), 64, md.data_ptr(), None, 64, 64, 64, tw.PATTERN_TW,
                           torch.cuda.current_stream().cuda_stream)
    assert ei.value.status == 5
    g.replay()
    torch.cuda.synchronize()
    assert float(x[0]) == 1.0
