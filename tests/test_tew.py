"""TEW (tile-wise plus restored single elements): host side of the C ABI against
the oracle's canonical form (no GPU), and the product against the oracle on the GPU."""
import numpy as np
import pytest

import paper_2402_10876_amd as tw
from oracle import gemm as og
from oracle import pack as opk
from tests.helpers import assert_C_close, random_tw_mask
import workloads as wl


def random_tew_mask(rng, K, N, G, extra=0.05, **kw):
    tm = random_tw_mask(rng, K, N, G, **kw)
    m = tm | ((rng.random((K, N)) < extra) & (tm == 0)).astype(np.uint8)
    return m, tm


def _same_tew(e, r):
    assert e["n_kept"] == r["n_kept"] and e["n_tiles"] == r["n_tiles"]
    for key in ("col_idx", "cto_n", "ew_col_ptr", "ew_row", "ew_val"):
        assert np.array_equal(e[key], r[key]), key
    for t in range(r["n_tiles"]):
        assert np.array_equal(e["row_idx"][t], r["row_idx"][t])
        assert np.array_equal(e["cto_k"][t], r["cto_k"][t])
        assert np.array_equal(e["values"][t], r["values"][t])


@pytest.mark.parametrize("seed", range(8))
def test_tew_export_equals_oracle_pack(seed):
    rng = np.random.default_rng(300 + seed)
    K, N = int(rng.integers(1, 90)), int(rng.integers(1, 200))
    G = int(rng.choice([32, 64, 128]))
    m, tm = random_tew_mask(rng, K, N, G, extra=rng.uniform(0.0, 0.2), col_keep=rng.uniform(0.3, 1.0))
    B = wl.rng_fp16(seed, (K, N))
    p = tw.tw_pack_host(B, m, G, tw.PATTERN_TEW, tile_mask=tm)
    _same_tew(p.export(), opk.ref_pack(B, m, G, opk.PATTERN_TEW, tile_mask=tm))
    Bm, m2 = p.unpack()
    assert np.array_equal(m2, m)
    assert np.array_equal(Bm, np.where(m != 0, B.view(np.uint16), 0))
    skw, sk, ku = p.flop_counts()
    assert skw == int(tm.sum()) and ku == int(m.any(axis=1).sum())
    p.free()


def test_tew_configured_workload_export():
    c = wl.make_case(2, 0, pattern="tew", sparsity=0.75, delta=0.015, with_A=False)
    assert abs(c.mask.mean() - 0.25) < 2e-3 and int(c.mask.sum() - c.tile_mask.sum()) == int(0.015 * c.K * c.N)
    p = tw.tw_pack_host(c.B, c.mask, c.G, tw.PATTERN_TEW, tile_mask=c.tile_mask)
    _same_tew(p.export(), opk.ref_pack(c.B, c.mask, c.G, opk.PATTERN_TEW, tile_mask=c.tile_mask))
    p.free()


def test_tew_concat_is_the_side_by_side_weight():
    rng = np.random.default_rng(5)
    K, G = 70, 32
    mem = []
    for i, N in enumerate([50, 90, 33]):
        m, tm = random_tew_mask(rng, K, N, G, extra=0.1)
        mem.append((wl.make_B(50 + i, K, N, 1.0), m, tm))
    parts = [tw.tw_pack_host(B, m, G, tw.PATTERN_TEW, tile_mask=t) for B, m, t in mem]
    cat = tw.tw_concat(parts, upload=False)
    Bm, m2 = cat.unpack()
    B_all = np.concatenate([B for B, _, _ in mem], axis=1)
    m_all = np.concatenate([m for _, m, _ in mem], axis=1)
    t_all = np.concatenate([t for _, _, t in mem], axis=1)
    assert np.array_equal(m2, m_all) and np.array_equal(Bm, np.where(m_all != 0, B_all.view(np.uint16), 0))
    e = cat.export()
    # the restored elements are one CSC over the concatenated columns
    ptr = e["ew_col_ptr"]
    for n in range(B_all.shape[1]):
        assert np.array_equal(e["ew_row"][ptr[n]:ptr[n + 1]], np.flatnonzero((m_all[:, n] != 0) & (t_all[:, n] == 0)))
    for p in parts + [cat]:
        p.free()


def test_tew_pack_errors():
    rng = np.random.default_rng(6)
    m, tm = random_tew_mask(rng, 20, 40, 32)
    B = wl.rng_fp16(6, m.shape)
    with pytest.raises(tw.TwError) as ei:
        tw.tw_pack_host(B, m, 32, tw.PATTERN_TEW)                       # no tile mask
    assert ei.value.status == 1
    bad = m.copy()
    k, n = np.argwhere(tm != 0)[0]
    bad[k, n] = 0
    with pytest.raises(tw.TwError) as ei:
        tw.tw_pack_host(B, bad, 32, tw.PATTERN_TEW, tile_mask=tm)       # mask does not contain the tile mask
    assert ei.value.status == 2
    with pytest.raises(tw.TwError) as ei:
        tw.tw_pack_host(B, m, 32, tw.PATTERN_TEW, tile_mask=m)          # tile mask is not tile-wise
    assert ei.value.status == 2


# ---------------------------------------------------------------------------------------------
def _gpu_run(B, m, tm, G, A, **kw):
    from tests import gpu_util as gu
    p = tw.tw_pack(B, m, G, tw.PATTERN_TEW, tile_mask=tm)
    C, raw = gu.run_tw(tw, p, A, B.shape[1], **kw)
    p.free()
    return C, raw


@pytest.fixture
def _opts():
    keys = (("tile_m", 0), ("ksplit", 0), ("waves", 4))
    for k, v in keys:
        tw.tw_set_option(k, v)
    yield
    for k, v in keys:
        tw.tw_set_option(k, v)


@pytest.mark.gpu
@pytest.mark.parametrize("G,tile_m", [(128, 0), (128, 64), (128, 128), (128, 256), (64, 128), (64, 256)])
def test_tew_identity_A_is_bit_exact(G, tile_m, _opts):
    """A = I: every C element is one weight or zero, so C must equal fp16(B (.) mask) bit for
    bit: pins the restored elements' rows, columns and values, pruned columns included."""
    rng = np.random.default_rng(G + tile_m)
    K, N = 200, 330
    m, tm = random_tew_mask(rng, K, N, G, extra=0.06, col_keep=0.8)
    assert (m[:, ~tm.any(0)]).any()                     # restored elements in pruned columns too
    B = wl.make_B(5, K, N, 1.0)
    tw.tw_set_option("tile_m", tile_m)
    print(f"case tew identity G={G} tile_m={tile_m}", flush=True)
    C, raw = _gpu_run(B, m, tm, G, np.eye(K, dtype=np.float16))
    want = np.where(m != 0, B, np.float16(0)).astype(np.float16)
    assert np.array_equal(raw[:, :K].T.view(np.uint16), want.view(np.uint16))


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 8, 129, 333])
@pytest.mark.parametrize("G", [64, 128])
def test_tew_random_masks_and_M_tails(M, G, _opts):
    rng = np.random.default_rng(70 + M + G)
    K, N = 410, 300
    m, tm = random_tew_mask(rng, K, N, G, extra=0.04)
    A, B = wl.make_A(M, M, K), wl.make_B(M, K, N, 1.0)
    print(f"case tew random M={M} G={G}", flush=True)
    C, raw = _gpu_run(B, m, tm, G, A, fill=3.0, ldc=(M + 7) // 8 * 8 + 8)
    assert_C_close(C, og.gemm_oracle(A, B, m), og.abs_bound(A, B, m))
    dead = ~m.any(0)
    assert not raw[dead, :M].view(np.uint16).any()
    assert (raw[:, M:] == 3.0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("G,tile_m,ksplit", [(128, 64, 1), (128, 128, 1), (128, 256, 1), (128, 128, 2), (128, 64, 2), (64, 128, 1),
                                             (64, 256, 1)])
def test_tew_infinities_stay_in_the_columns_that_refer_to_them(G, tile_m, ksplit, _opts):
    """Rows with several restored elements are multiplied whole, zeros included; an infinity or NaN of A in such a row
    must reach the columns that hold one of its elements and no other."""
    rng = np.random.default_rng(G + tile_m + ksplit)
    K, N, M = 210, 300, 270
    m, tm = random_tew_mask(rng, K, N, G, extra=0.05, col_keep=0.9, row_keep=0.3)
    A, B = wl.make_A(4, M, K), wl.make_B(4, K, N, 1.0)
    B[B == 0] = 1
    restored = (m != 0) & (tm == 0)
    # (row 0 and the tiles' last kept rows also stand in, times +0, where a list is padded)
    padding = np.append(K - 1 - tm[::-1].argmax(0)[tm.any(0)], 0)
    ks = np.setdiff1d(np.flatnonzero(restored.any(1)), padding)[[0, 7, -1]]
    A[3, ks[0]], A[4, ks[1]], A[M - 1, ks[2]] = np.inf, np.nan, -np.inf
    tw.tw_set_option("tile_m", tile_m)
    tw.tw_set_option("ksplit", ksplit)
    print(f"case tew infinities G={G} tile_m={tile_m} ksplit={ksplit}", flush=True)
    _check_infinities(A, B, m, *_gpu_run(B, m, tm, G, A))


def _check_infinities(A, B, m, C, _raw):
    N = B.shape[1]
    with np.errstate(invalid="ignore"):
        want = np.stack([A[:, m[:, n] != 0].astype(np.float64) @ B[m[:, n] != 0, n].astype(np.float64) for n in range(N)], axis=1)
    fin = np.isfinite(want)
    assert not fin.all() and (~fin).sum() < fin.sum()
    assert np.array_equal(np.isfinite(C), fin) and np.array_equal(np.isnan(C), np.isnan(want))
    assert np.array_equal(C[~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)])
    F = np.where(np.isfinite(A), A, np.float16(0))
    ref, S = og.gemm_oracle(F, B, m), og.abs_bound(F, B, m)
    assert_C_close(np.where(fin, C, ref), ref, S)


@pytest.mark.gpu
@pytest.mark.parametrize("G,M,K,N,col_keep", [(128, 40, 210, 300, 0.9), (64, 5, 900, 190, 0.6), (64, 33, 100, 64, 1.0),
                                              (128, 1, 2000, 100, 0.1)])
def test_tew_few_blocks(G, M, K, N, col_keep, _opts):
    """The kernel for few output blocks, finite (also A = I, bit for bit) and with infinities."""
    rng = np.random.default_rng(G + M)
    m, tm = random_tew_mask(rng, K, N, G, extra=0.03, col_keep=col_keep, row_keep=0.3)
    A, B = wl.make_A(6, M, K), wl.make_B(6, K, N, 1.0)
    print(f"case tew few blocks G={G} M={M}", flush=True)
    C, _ = _gpu_run(B, m, tm, G, A)
    assert_C_close(C, og.gemm_oracle(A, B, m), og.abs_bound(A, B, m))
    eye = np.zeros((M, K), np.float16)
    at = rng.choice(K, M, replace=False)
    eye[np.arange(M), at] = 1
    _, raw = _gpu_run(B, m, tm, G, eye)
    want = np.where(m != 0, B, np.float16(0)).astype(np.float16)[at]
    assert np.array_equal(raw[:, :M].T.view(np.uint16), want.view(np.uint16))
    padding = np.append(K - 1 - tm[::-1].argmax(0)[tm.any(0)], 0)
    ks = np.setdiff1d(np.flatnonzero(((m != 0) & (tm == 0)).any(1)), padding)[[0, -1]]
    A[0, ks[0]], A[M - 1, ks[1]] = np.inf, -np.inf
    B[B == 0] = 1
    _check_infinities(A, B, m, *_gpu_run(B, m, tm, G, A))


@pytest.mark.gpu
@pytest.mark.parametrize("G,M,K,N,tile_m,ksplit", [
    (128, 1, 1500, 3000, 0, 0), (64, 33, 500, 2000, 0, 0),                                        # few output blocks
    (128, 333, 410, 900, 64, 1), (128, 333, 410, 900, 128, 1), (128, 333, 410, 900, 256, 1), (64, 333, 410, 900, 128, 1),
    (64, 333, 410, 900, 256, 1), (128, 129, 900, 900, 64, 2), (128, 131, 900, 900, 128, 2), (64, 1, 900, 2000, 128, 2)])
def test_tew_padding_of_A_is_no_input(G, M, K, N, tile_m, ksplit, _opts):
    """Rows past M of the last tile come from columns M .. round-up-8(M) of A, which a caller may leave as they are: the
    same bits whatever lies there, and those of the sums with the joined rows."""
    import torch
    rng = np.random.default_rng(G + M + tile_m)
    m, tm = random_tew_mask(rng, K, N, G, extra=0.04, col_keep=0.8, row_keep=0.3)
    A, B = wl.make_A(9, M, K), wl.make_B(9, K, N, 1.0)
    tw.tw_set_option("tile_m", tile_m)
    tw.tw_set_option("ksplit", ksplit)
    ld = (M + 7) // 8 * 8
    p = tw.tw_pack(B, m, G, tw.PATTERN_TEW, tile_mask=tm)
    out = []
    for pad in (0.0, 7.0, np.nan, -np.inf):
        print(f"case tew padding G={G} M={M} tile_m={tile_m} ksplit={ksplit} pad={pad}", flush=True)
        At = np.full((K, ld), pad, np.float16)
        At[:, :M] = A.T
        Ad = torch.from_numpy(At).cuda()
        C = torch.full((N, ld), 3.0, dtype=torch.float16, device="cuda")
        tw.tw_gemm(Ad.data_ptr(), M, ld, tw.LAYOUT_KM, p, C.data_ptr(), ld, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        out.append(C.cpu().numpy())
    p.free()
    assert_C_close(out[0][:, :M].T.astype(np.float64), og.gemm_oracle(A, B, m), og.abs_bound(A, B, m))
    assert (out[0][:, M:] == 3.0).all()
    for other in out[1:]:
        assert np.array_equal(out[0].view(np.uint16), other.view(np.uint16))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,tile_m,ksplit", [(512, 384, 64, 1), (500, 384, 128, 1), (129, 640, 64, 2), (1, 256, 128, 2), (700, 1024, 256, 1),
                                              (384, 3100, 0, 0)])
def test_tew_elements_one_by_one(M, N, tile_m, ksplit, _opts):
    """Long lists of joined rows with few elements each: the elements are added one by one (the host's rule holds for these
    shapes); A = I, bit for bit, random values and infinities."""
    import torch
    rng = np.random.default_rng(M + N)
    K, G = 3000, 128
    m, tm = random_tew_mask(rng, K, N, G, extra=0.003, col_keep=0.9, row_keep=0.1)
    A, B = wl.make_A(10, M, K), wl.make_B(10, K, N, 1.0)
    B[B == 0] = 1
    tw.tw_set_option("tile_m", tile_m)
    tw.tw_set_option("ksplit", ksplit)
    lda = (M + 63) // 64 * 64
    p = tw.tw_pack(B, m, G, tw.PATTERN_TEW, tile_mask=tm)

    def run(X):
        At = np.full((K, lda), np.nan, np.float16)
        At[:, :M] = X.T
        Ad = torch.from_numpy(At).cuda()
        C = torch.full((N, lda), 3.0, dtype=torch.float16, device="cuda")
        tw.tw_gemm(Ad.data_ptr(), M, lda, tw.LAYOUT_KM, p, C.data_ptr(), lda, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        raw = C.cpu().numpy()
        assert (raw[:, M:] == 3.0).all()
        return raw[:, :M].T

    print(f"case tew one by one M={M} N={N} tile_m={tile_m} ksplit={ksplit}", flush=True)
    assert_C_close(run(A).astype(np.float64), og.gemm_oracle(A, B, m), og.abs_bound(A, B, m))
    at = rng.choice(K, M, replace=False)
    eye = np.zeros((M, K), np.float16)
    eye[np.arange(M), at] = 1
    want = np.where(m != 0, B, np.float16(0)).astype(np.float16)[at]
    assert np.array_equal(run(eye).view(np.uint16), want.view(np.uint16))
    padding = np.append(K - 1 - tm[::-1].argmax(0)[tm.any(0)], 0)
    ks = np.setdiff1d(np.flatnonzero(((m != 0) & (tm == 0)).any(1)), padding)[[0, -1]]
    A[0, ks[0]], A[M - 1, ks[1]] = np.inf, -np.inf
    _check_infinities(A, B, m, run(A).astype(np.float64), None)
    p.free()


@pytest.mark.gpu
@pytest.mark.parametrize("G,M,K,tile_m,ksplit", [
    (64, 5, 210, 0, 0), (128, 5, 210, 0, 0),                                                      # few output blocks
    (64, 333, 210, 128, 1), (64, 333, 900, 128, 2), (128, 333, 210, 64, 1), (128, 333, 210, 256, 1), (128, 333, 900, 64, 2)])
def test_tew_concat_gemm(G, M, K, tile_m, ksplit, _opts):
    """Members' rows with restored elements join the tiles of the concatenated weight: narrow tiles in the middle, a member without
    restored elements and one without kept columns; random values, and A = I, bit for bit."""
    rng = np.random.default_rng(G + M + K)
    mem = []
    for i, (N, extra, kw) in enumerate([(150, 0.04, {}), (300, 0.0, {}), (77, 0.02, dict(col_keep=0.0)), (190, 0.08, dict(row_keep=0.1))]):
        m, tm = random_tew_mask(rng, K, N, G, extra=extra, **kw)
        mem.append((wl.make_B(60 + i, K, N, 1.0), m, tm))
    parts = [tw.tw_pack_host(B, m, G, tw.PATTERN_TEW, tile_mask=t) for B, m, t in mem]
    cat = tw.tw_concat(parts)
    B, m = (np.concatenate([x[i] for x in mem], axis=1) for i in (0, 1))
    A = wl.make_A(11, M, K)
    eye = np.zeros((M, K), np.float16)
    at = rng.permutation(np.arange(M) % K)
    eye[np.arange(M), at] = 1
    tw.tw_set_option("tile_m", tile_m)
    tw.tw_set_option("ksplit", ksplit)
    from tests import gpu_util as gu
    print(f"case tew concat G={G} M={M} tile_m={tile_m} ksplit={ksplit}", flush=True)
    C, _ = gu.run_tw(tw, cat, A, B.shape[1])
    _, raw = gu.run_tw(tw, cat, eye, B.shape[1])
    assert_C_close(C, og.gemm_oracle(A, B, m), og.abs_bound(A, B, m))
    want = np.where(m != 0, B, np.float16(0)).astype(np.float16)[at]
    want[want == 0] = 0                                                # (+0: a sum that starts at +0)
    assert np.array_equal(raw[:, :M].T.view(np.uint16), want.view(np.uint16))
    for p in parts + [cat]:
        p.free()


def test_tew_image_join_counts_only_shape_the_device_form():
    """tw_flop_counts, tw_export and tw_unpack know nothing of the rows that are multiplied whole."""
    rng = np.random.default_rng(31)
    m, tm = random_tew_mask(rng, 300, 200, 64, extra=0.05)
    B = wl.make_B(31, 300, 200, 1.0)
    p = tw.tw_pack_host(B, m, 64, tw.PATTERN_TEW, tile_mask=tm)
    assert p.flop_counts()[0] == int(tm.sum())
    _same_tew(p.export(), opk.ref_pack(B, m, 64, opk.PATTERN_TEW, tile_mask=tm))
    p.free()


@pytest.mark.gpu
@pytest.mark.parametrize("K,N,G,M", [(300, 260, 128, 200), (900, 1500, 128, 1700), (900, 1500, 64, 1333), (150, 3000, 128, 4100)])
def test_tew_without_restored_elements_equals_tw(K, N, G, M, _opts):
    from tests import gpu_util as gu
    rng = np.random.default_rng(77)
    tm = random_tw_mask(rng, K, N, G)
    A, B = wl.make_A(7, M, K), wl.make_B(7, K, N, 1.0)
    _, raw = _gpu_run(B, tm, tm, G, A)
    p = tw.tw_pack(B, tm, G, tw.PATTERN_TW)
    _, raw_tw = gu.run_tw(tw, p, A, N)
    p.free()
    assert np.array_equal(raw[:, :M].view(np.uint16), raw_tw[:, :M].view(np.uint16))


@pytest.mark.gpu
@pytest.mark.parametrize("ksplit,tile_m", [(2, 64), (2, 128)])
def test_tew_k_split_instances(ksplit, tile_m, _opts):
    rng = np.random.default_rng(80 + tile_m)
    K, N, G, M = 900, 200, 128, 260
    m, tm = random_tew_mask(rng, K, N, G, extra=0.03)
    A, B = wl.make_A(8, M, K), wl.make_B(8, K, N, 1.0)
    tw.tw_set_option("ksplit", ksplit); tw.tw_set_option("tile_m", tile_m)
    print(f"case tew ksplit tile_m={tile_m}", flush=True)
    C, _ = _gpu_run(B, m, tm, G, A)
    assert_C_close(C, og.gemm_oracle(A, B, m), og.abs_bound(A, B, m))


@pytest.mark.gpu
@pytest.mark.parametrize("shape_index", [0, 1, 2])
def test_tew_bert_base_sampled(shape_index, _opts):
    """BERT-base shapes, 75 % with delta = 1.5 %, in the launch configuration the heuristics
    pick at full size; the oracle on sampled rows of C."""
    c = wl.make_case(2, shape_index, pattern="tew", sparsity=0.75, delta=0.015)
    print(f"case {c.name}", flush=True)
    C, raw = _gpu_run(c.B, c.mask, c.tile_mask, c.G, c.A)
    rows = np.random.default_rng(1).choice(c.M, 48, replace=False)
    assert_C_close(C[rows], og.gemm_oracle(c.A[rows], c.B, c.mask), og.abs_bound(c.A[rows], c.B, c.mask))


@pytest.mark.gpu
def test_tew_unsupported_configurations_are_errors(_opts):
    import torch
    rng = np.random.default_rng(90)
    m, tm = random_tew_mask(rng, 64, 64, 32)
    p = tw.tw_pack(wl.make_B(1, 64, 64, 1.0), m, 32, tw.PATTERN_TEW, tile_mask=tm)
    A = torch.zeros((64, 64), dtype=torch.float16, device="cuda")
    Cd = torch.zeros((64, 64), dtype=torch.float16, device="cuda")
    for layout in (tw.LAYOUT_KM, tw.LAYOUT_MK):       # G = 32 has no TEW kernel; row-major has none either
        with pytest.raises(tw.TwError) as ei:
            tw.tw_gemm(A.data_ptr(), 64, 64, layout, p, Cd.data_ptr(), 64, 0)
        assert ei.value.status == 3
    p.free()
