"""GPU parity of the k-means codebook update against the CPU oracle: given the
same assignment, the updated binary16 books and the cluster counts must match
bit for bit (the sums are exact integers, so the order of the GPU's atomics does
not matter)."""
import numpy as np
import pytest
import torch

from paper_2607_07144_amd import workloads as w

pytestmark = pytest.mark.gpu


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("name", ["tiny", "gpt2"])
def test_lloyd_iterations_match_oracle(fkv, orc, name):
    cfg = w.CONFIGS[name]
    x, books, sb = w.make_group_numpy(cfg)
    xd, bd, sd = (torch.from_numpy(a).cuda() for a in (x, books, sb))
    S = books.shape[1]
    for it in range(2):
        for stage in range(S):
            sym, _ = fkv.fkv_rvq_assign(xd, bd, sd, cfg.t_begin, cfg.t_end)
            before = host(bd).copy()
            _, counts = fkv.fkv_kmeans_step(xd, bd, sd, cfg.t_begin, cfg.t_end, sym, stage)
            want, means, wc = orc.kmeans_update(x, before, sb, cfg.t_begin, cfg.t_end, host(sym), stage)
            assert np.array_equal(host(counts), wc), (it, stage)
            assert np.array_equal(host(bd).view(np.uint16), want.view(np.uint16)), (it, stage)


@pytest.mark.parametrize("d,S,K", [(64, 8, 32), (128, 3, 256), (48, 6, 20)])
def test_every_stage_matches_oracle(fkv, orc, d, S, K):
    """One update of every stage of deep books: stages 0-4 run kernels with the stage fixed at compile
    time, stages 5-7 the one that takes it at run time; each must match the oracle bit for bit."""
    rng = np.random.default_rng(d + S + K)
    ns, T, nb = 6, 120, 3
    x = (rng.standard_normal((ns, T, d)) * 1.3).astype(np.float16)
    books = (rng.standard_normal((nb, S, K, d)) * (0.6 ** np.arange(S))[None, :, None, None]).astype(np.float16)
    sb = rng.integers(0, nb, ns).astype(np.int32)
    xd, bd, sd = (torch.from_numpy(a).cuda() for a in (x, books, sb))
    sym, _ = fkv.fkv_rvq_assign(xd, bd, sd, 2, T - 1)
    symh = host(sym)
    for stage in range(S):
        before = host(bd).copy()
        _, counts = fkv.fkv_kmeans_step(xd, bd, sd, 2, T - 1, sym, stage)
        want, _, wc = orc.kmeans_update(x, before, sb, 2, T - 1, symh, stage)
        assert np.array_equal(host(counts), wc), stage
        assert np.array_equal(host(bd).view(np.uint16), want.view(np.uint16)), stage


@pytest.mark.parametrize("ns,T,d,S,K,stage,nb", [
    (2, 8193, 64, 1, 256, 0, 1),      # a chunk of 8192 tokens and one more
    (3, 8192, 16, 2, 5, 1, 2), (5, 4097, 8, 1, 256, 0, 1),     # chunks that straddle streams
    (1500, 1, 24, 2, 40, 1, 3), (1030, 17, 8, 1, 7, 0, 1),     # one-token streams; more streams than one scan
    (200, 100, 80, 3, 256, 2, 2), (4, 3000, 136, 2, 33, 1, 1), (2, 2500, 256, 6, 17, 5, 2), (9, 911, 72, 1, 1, 0, 1),
])
@pytest.mark.parametrize("extreme", [False, True])
def test_sorted_sums_match_oracle(fkv, orc, ns, T, d, S, K, stage, nb, extreme):
    """Chunks, stream boundaries, ragged slices and skipped tokens of the sorted accumulation; with the
    largest and smallest binary16 values, where the register sums come closest to their bound."""
    rng = np.random.default_rng(ns + T + d)
    x = (rng.standard_normal((ns, T, d)) * 1.5).astype(np.float16)
    books = (rng.standard_normal((nb, S, K, d)) * 0.5).astype(np.float16)
    if extreme:
        big, tiny = np.float16(65504), np.float16(2 ** -24)
        x = np.where(rng.random(x.shape) < 0.9, big, tiny).astype(np.float16)
        books = np.where(rng.random(books.shape) < 0.9, -big, -tiny).astype(np.float16)
    sb = rng.integers(0, nb, ns).astype(np.int32)
    sb[-1] = nb                                                    # no book
    sym = rng.integers(0, min(K + 1, 256), (ns, T * S)).astype(np.uint8)   # some symbols outside the book
    sym.reshape(-1, S)[: len(sym.reshape(-1, S)) // 2, stage] = K - 1      # one crowded cluster
    bd = torch.from_numpy(books).cuda()
    sums = torch.zeros((nb, K, d), dtype=torch.int64, device="cuda")
    _, counts = fkv.fkv_kmeans_step(torch.from_numpy(x).cuda(), bd, torch.from_numpy(sb).cuda(), 0, T,
                                    torch.from_numpy(sym).cuda(), stage, sums=sums)
    want, _, wc = orc.kmeans_update(x, books, sb, 0, T, sym, stage)
    assert np.array_equal(host(counts), wc)
    assert np.array_equal(host(bd).view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("d,S,K,stage", [
    (64, 2, 256, 1), (128, 3, 200, 2), (8, 1, 256, 0), (24, 8, 31, 7), (72, 5, 256, 4), (256, 4, 129, 3), (48, 6, 256, 5),
    (64, 1, 100, 0), (136, 2, 128, 0),
])
def test_direct_and_sorted_forms_agree(fkv, d, S, K, stage):
    """The same 1500 tokens of each book as one stream (fewer tokens than the sort repays, or a narrow row: added
    directly) and as six streams (sorted by cluster): sums and counts are equal bit for bit, with skipped
    symbols and non-finite elements among them."""
    rng = np.random.default_rng(d + S + K + stage)
    nb, T = 260, 1500
    x = (rng.standard_normal((nb, T, d)) * 1.5).astype(np.float16)
    x[rng.integers(0, nb, 40), rng.integers(0, T, 40), rng.integers(0, d, 40)] = np.inf
    x[rng.integers(0, nb, 40), rng.integers(0, T, 40), rng.integers(0, d, 40)] = np.nan
    books = (rng.standard_normal((nb, S, K, d)) * 0.5).astype(np.float16)
    sym = rng.integers(0, min(K + 1, 256), (nb, T * S)).astype(np.uint8)
    sym[:, :S * 700] = K - 1
    xd, sd = torch.from_numpy(x).cuda(), torch.from_numpy(sym).cuda()
    got = []
    for parts in (1, 6):
        sb = torch.arange(nb, dtype=torch.int32, device="cuda").repeat_interleave(parts)
        sums = torch.zeros((nb, K, d), dtype=torch.int64, device="cuda")
        bd = torch.from_numpy(books).cuda()
        _, counts = fkv.fkv_kmeans_step(xd.view(nb * parts, T // parts, d), bd, sb, 0, T // parts,
                                        sd.view(nb * parts, -1), stage, sums=sums)
        got.append((sums, counts, host(bd).view(np.uint16)))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert np.array_equal(got[0][2], got[1][2])


@pytest.mark.parametrize("ns,T,d,S,K,stage", [
    (3, 5000, 64, 1, 4, 0), (3, 900, 128, 3, 256, 2), (40, 30, 16, 6, 20, 5), (2, 700, 72, 5, 33, 4), (5, 37, 8, 1, 1, 0),
])
def test_non_finite_elements(fkv, ns, T, d, S, K, stage):
    """A NaN element of a stage input adds nothing to its sum and an infinite one 2^63 - 2^32 or -2^63
    (modulo 2^64); the finite elements of the same cluster, token and book still add up exactly, call after
    call.  NaN and infinities come from the vectors and from the earlier stages' codewords."""
    rng = np.random.default_rng(ns + T + d + S + K)
    x = (rng.standard_normal((ns, T, d)) * 1.5).astype(np.float16)
    books = (rng.standard_normal((2, S, K, d)) * 0.5).astype(np.float16)
    for v in (np.nan, np.inf, -np.inf):
        x[rng.integers(0, ns, 9), rng.integers(0, T, 9), rng.integers(0, d, 9)] = v
        if stage:
            books[rng.integers(0, 2, 3), rng.integers(0, stage, 3), rng.integers(0, K, 3), rng.integers(0, d, 3)] = v
    sb = (np.arange(ns) % 2).astype(np.int32)
    sym = rng.integers(0, K, (ns, T, S)).astype(np.uint8)
    with np.errstate(invalid="ignore"):
        r = x.astype(np.float64)
        for st in range(stage):
            r = r - books.astype(np.float64)[sb[:, None], st, sym[..., st]]
    fixed = np.zeros(r.shape, np.int64)
    fixed[np.isfinite(r)] = (r[np.isfinite(r)] * 2.0 ** 24).astype(np.int64)      # exact
    fixed[r == np.inf] = 2 ** 63 - 2 ** 32
    fixed[r == -np.inf] = -2 ** 63
    want, wc = np.zeros((2, K, d), np.int64), np.zeros((2, K), np.int64)
    where = (np.broadcast_to(sb[:, None], (ns, T)), sym[..., stage])
    np.add.at(want, where, fixed)                                                  # wraps modulo 2^64
    np.add.at(wc, where, 1)
    assert np.isnan(r).any() and np.isinf(r).any()
    for _ in range(3):
        sums = torch.zeros((2, K, d), dtype=torch.int64, device="cuda")
        _, counts = fkv.fkv_kmeans_step(torch.from_numpy(x).cuda(), torch.from_numpy(books).cuda(),
                                        torch.from_numpy(sb).cuda(), 0, T, torch.from_numpy(sym).cuda().view(ns, T * S),
                                        stage, sums=sums)
        assert np.array_equal(host(counts), wc) and np.array_equal(host(sums), want)


def test_skipped_tokens(fkv, orc):
    """Streams with an invalid book id and tokens whose symbols reach K contribute nothing."""
    rng = np.random.default_rng(4)
    ns, T, d, S, K = 6, 50, 24, 2, 8
    x = rng.standard_normal((ns, T, d)).astype(np.float16)
    books = rng.standard_normal((2, S, K, d)).astype(np.float16)
    sb = np.array([0, 1, 5, 0, -1, 1], np.int32)
    sym = rng.integers(0, K + 2, (ns, (T - 3) * S)).astype(np.uint8)       # some symbols >= K
    bd = torch.from_numpy(books).cuda()
    _, counts = fkv.fkv_kmeans_step(torch.from_numpy(x).cuda(), bd, torch.from_numpy(sb).cuda(), 3, T,
                                    torch.from_numpy(sym).cuda(), 1)
    want, _, wc = orc.kmeans_update(x, books, sb, 3, T, sym, 1)
    assert np.array_equal(host(counts), wc) and np.array_equal(host(bd).view(np.uint16), want.view(np.uint16))


def test_training_lowers_distortion(fkv):
    """Lloyd iterations on the GPU-shaped cache: the archive's reconstruction error falls."""
    cfg = w.CONFIGS["gpt2"]
    x, books, sb = w.make_group_numpy(cfg)
    xd, bd, sd = (torch.from_numpy(a).cuda() for a in (x, books, sb))
    errs = []
    for it in range(4):
        for stage in range(books.shape[1]):
            sym, res = fkv.fkv_rvq_assign(xd, bd, sd, cfg.t_begin, cfg.t_end, want_residual=True)
            if stage == 0:
                errs.append(float((res.double() ** 2).sum()))
            fkv.fkv_kmeans_step(xd, bd, sd, cfg.t_begin, cfg.t_end, sym, stage)
    assert errs[-1] < errs[0] and all(b <= a * 1.001 for a, b in zip(errs, errs[1:]))


def _train(fkv, xd, bd, sd, t0, t1, iters):
    S = bd.shape[1]
    for it in range(iters):
        for stage in range(S):
            sym, _ = fkv.fkv_rvq_assign(xd, bd, sd, t0, t1)
            fkv.fkv_kmeans_step(xd, bd, sd, t0, t1, sym, stage)


def _trained_parity(fkv, orc, x, bd, sb, t0, t1, idx):
    """Assignment on trained books against the oracle (teacher-forced near-ties); returns the
    near-ties per stage and the mean of D1/||x||^2 at the last stage."""
    xd, sd = torch.from_numpy(x).cuda(), torch.from_numpy(sb).cuda()
    sym, res = fkv.fkv_rvq_assign(xd, bd, sd, t0, t1, want_residual=True)
    fs, fp, fr = fkv.fkv_rvq_assign_encode(fkv.Codec(256), xd, bd, sd, t0, t1, want_residual=True)
    assert torch.equal(fs, sym) and torch.equal(fr, res)
    sym, res, books = host(sym), host(res), host(bd)
    o = orc.rvq_assign(x[idx], books, sb[idx], t0, t1, force=sym[idx], force_tol=1e-5)
    assert o["n_hard"] == 0, "index differs from the oracle outside the near-tie band on trained books"
    assert np.array_equal(o["symbols"], sym[idx])
    assert np.abs(o["residual"] - res[idx].astype(np.float64)).max() <= 1e-3
    S = books.shape[1]
    gaps = o["gaps"].reshape(len(idx), -1, S)
    ties = [int((gaps[:, :, st] < 1e-5).sum()) for st in range(S)]
    rel = float((o["residual"] ** 2).sum() / (x[idx][:, t0:t1].astype(np.float64) ** 2).sum())
    return ties, rel


def test_rvq_parity_on_trained_books_gpt2(fkv, orc):
    """Books after 10 Lloyd iterations (Sec. 3 "Setup": codebooks trained by k-means) at the GPT-2
    shape: the residual energy left after the stages is well below ||x||^2, which is where the
    score offsets and the fp32 accumulation are most stressed."""
    cfg = w.CONFIGS["gpt2"]
    x, books, sb = w.make_group_numpy(cfg)
    xd, bd, sd = (torch.from_numpy(a).cuda() for a in (x, books, sb))
    _train(fkv, xd, bd, sd, cfg.t_begin, cfg.t_end, 10)
    ties, rel = _trained_parity(fkv, orc, x, bd, sb, cfg.t_begin, cfg.t_end, np.arange(x.shape[0]))
    print("gpt2 trained books: near-ties per stage %s, residual energy %.3f of ||x||^2" % (ties, rel))
    assert rel < 0.9


def test_rvq_parity_on_trained_books_long_context_heads(fkv, orc):
    """The long-context head shape (d = 128, S = 3, K = 256, four x10 key-outlier channels) on 16
    streams of 4,096 tokens, one book each, after 10 Lloyd iterations."""
    cfg = w.Config(name="long_heads_sample", layers=1, heads=8, d=128, T=4096, batch=1, seed=1104,
                   groups=(w.Group(("K", "V"), S=3, K=256, N=256),))
    x, books, sb = w.make_group_numpy(cfg)
    xd, bd, sd = (torch.from_numpy(a).cuda() for a in (x, books, sb))
    _train(fkv, xd, bd, sd, cfg.t_begin, cfg.t_end, 10)
    ties, rel = _trained_parity(fkv, orc, x, bd, sb, cfg.t_begin, cfg.t_end, np.array([0, 5, 9, 15]))
    print("d128 trained books: near-ties per stage %s, residual energy %.3f of ||x||^2" % (ties, rel))
    assert rel < 0.95
