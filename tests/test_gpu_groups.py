"""GPU tests of the grouped assignment (fkv_rvq_assign_groups): one block serves the tokens of every stream
of a group that shares a book.  Each token's arithmetic is that of the per-stream assignment, so symbols and
residuals must equal fkv_rvq_assign's bit for bit; on the GPT-2-shaped eviction step (one leaving token per
stream) the oracle's bars (Sec. 3 "Setup": nearest codebook entries, greedy over the stages) apply directly."""
import numpy as np
import pytest
import torch

from paper_2607_07144_amd import workloads as w

pytestmark = pytest.mark.gpu

NEAR_TIE = 1e-5


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("d,S,K,T,t0,t1,G", [
    (128, 3, 256, 300, 299, 300, 4),    # an eviction step at the long-context head shape
    (128, 3, 256, 40, 3, 40, 8),        # several tokens per member, one block per group
    (64, 4, 256, 130, 2, 128, 3),       # 3 x 126 tokens: two blocks per group, members straddle them
    (64, 2, 64, 1, 0, 1, 4),            # a small book (the per-stream form has its own kernel for it)
    (256, 3, 256, 70, 69, 70, 16),      # single book buffer, hi/lo residual
    (16, 1, 16, 5, 0, 5, 1),            # one-member groups
    (32, 8, 33, 129, 1, 128, 2),        # padded book, eight stages
    (128, 2, 256, 10, 9, 10, 256),      # the largest group
    (80, 3, 130, 20, 0, 20, 5),
])
def test_groups_equal_per_stream(fkv, d, S, K, T, t0, t1, G):
    rng = np.random.default_rng(d + 7 * S + K + G)
    nb = 3
    ns = nb * G
    x = (rng.standard_normal((ns, T, d)) * 2).astype(np.float16)
    books = (rng.standard_normal((nb, S, K, d)) * (0.5 ** np.arange(S))[None, :, None, None]).astype(np.float16)
    sb = (np.arange(ns) % nb).astype(np.int32)          # a book's streams are strided, as batch entries are
    groups = fkv.book_groups(sb)
    assert groups.shape == (nb, G)
    xd, bd, sd = dev(x), dev(books), dev(sb)
    full, fres = fkv.fkv_rvq_assign(xd, bd, sd, t0, t1, want_residual=True)
    sym = torch.full_like(full, 0xA5)
    res = torch.full_like(fres, 7.0)
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(groups), t0, t1, symbols=sym, residual=res, n_bad=nbad)
    assert torch.equal(sym, full) and int(host(nbad)[0]) == 0
    assert np.array_equal(host(res).view(np.uint32), host(fres).view(np.uint32))
    # one group listed: the other streams keep their bytes
    sym.fill_(0xA5)
    fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(groups[1:2]), t0, t1, symbols=sym)
    got, want = host(sym), host(full)
    listed = np.zeros(ns, bool)
    listed[groups[1]] = True
    assert np.array_equal(got[listed], want[listed]) and (got[~listed] == 0xA5).all()


@pytest.mark.parametrize("d,S,K,n", [
    (16, 1, 1, 1), (32, 3, 33, 2), (48, 2, 64, 31), (64, 2, 256, 1), (64, 4, 256, 32), (80, 3, 97, 5), (96, 2, 100, 4),
    (112, 5, 129, 3), (128, 3, 256, 4), (128, 2, 200, 32), (128, 8, 256, 7), (144, 3, 255, 2), (192, 4, 64, 6),
    (208, 2, 160, 1), (256, 3, 256, 4), (256, 8, 31, 32),
])
def test_few_tokens_equal_bulk(fkv, d, S, K, n):
    """At most 32 tokens per work item (per stream, or per group of streams) against the bulk form over a
    longer range that holds them: the arithmetic of a token does not depend on the other tokens, so symbols
    and residuals are equal bit for bit.  Tied codewords, zero vectors, a stream and a group without a book,
    and fewer stages than the layout holds."""
    rng = np.random.default_rng(d + 5 * S + K + n)
    nb, ns, T, t0 = 3, 520, 75, 11                      # more streams than resident blocks of the staged form
    x = (rng.standard_normal((ns, T, d)) * 2).astype(np.float16)
    x[1, t0] = 0
    books = (rng.standard_normal((nb, S, K, d)) * (0.5 ** np.arange(S))[None, :, None, None]).astype(np.float16)
    books[1, :, K // 2] = books[1, :, 0]                # equal codewords: the lower index wins
    sb = np.tile(np.array([0, 1, 2, 1, 0, 2, 1, 2], np.int32), ns // 8)
    sb[5] = 9                                           # no book
    xd, bd, sd = dev(x), dev(books), dev(sb)
    full, fres = fkv.fkv_rvq_assign(xd, bd, sd, 0, T, want_residual=True)
    full, fres = host(full).reshape(ns, T, S)[:, t0:t0 + n], host(fres)[:, t0:t0 + n]
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    sym, res = fkv.fkv_rvq_assign(xd, bd, sd, t0, t0 + n, want_residual=True, n_bad=nbad)
    assert np.array_equal(host(sym).reshape(ns, n, S), full) and int(host(nbad)[0]) == 1
    assert np.array_equal(host(res).view(np.uint32), fres.view(np.uint32))
    k = max(1, S - 1)
    sym = torch.full((ns, n * S), 0xA5, dtype=torch.uint8, device="cuda")
    fkv.fkv_rvq_assign(xd, bd, sd, t0, t0 + n, symbols=sym, n_stages=k)
    got = host(sym).reshape(ns, n, S)
    valid = np.arange(ns) != 5
    assert np.array_equal(got[..., :k], full[..., :k]) and (got[valid][..., k:] == 0xA5).all()
    if 2 * n <= 32:
        some = np.array([[0, 4], [3, 6], [2, 7], [5, 1]], np.int32)   # the last one mixes books
        groups = dev(np.tile(some, (130, 1)))           # (the same bytes written again)
        nbad.zero_()
        sym = torch.full((ns, n * S), 0xA5, dtype=torch.uint8, device="cuda")
        res = torch.zeros((ns, n, d), dtype=torch.float32, device="cuda")
        fkv.fkv_rvq_assign_groups(xd, bd, sd, groups, t0, t0 + n, symbols=sym, residual=res, n_bad=nbad)
        got, gr, listed = host(sym).reshape(ns, n, S), host(res), [0, 4, 3, 6, 2, 7]
        assert np.array_equal(got[listed], full[listed]) and int(host(nbad)[0]) == 130
        assert np.array_equal(gr[listed].view(np.uint32), fres[listed].view(np.uint32))
        assert (got[[1, 5]] == 0xFF).all() and np.isnan(gr[[1, 5]]).all()


@pytest.mark.parametrize("d,S,K,n", [
    (16, 2, 100, 40), (32, 1, 256, 257), (48, 3, 65, 130), (64, 2, 256, 300), (64, 4, 200, 65), (80, 3, 100, 255),
    (96, 5, 129, 33), (112, 2, 256, 64), (128, 3, 256, 290), (128, 1, 70, 256), (128, 8, 256, 48),
    (48, 3, 65, 210), (64, 4, 200, 201), (96, 5, 129, 133), (128, 8, 256, 150), (80, 3, 100, 200), (80, 2, 256, 130),
])
def test_block_shapes_agree(fkv, d, S, K, n):
    """Large launches of full enough items (more than 256; 1536 at d <= 64 with at most two stages) take blocks
    of two token tiles per wave, smaller ones, and deep ones of half-empty items, blocks of one:
    symbols, residuals, points and counts are equal bit for bit, per stream, fused with the encode and grouped,
    with ragged items, a padded book, equal codewords and a stream without a book."""
    rng = np.random.default_rng(d + 3 * S + K + n)
    nb, t0 = 3, 2
    ns = 1560 if d <= 64 and S <= 2 else 280
    T = n + 5
    x = (rng.standard_normal((ns, T, d)) * 2).astype(np.float16)
    books = (rng.standard_normal((nb, S, K, d)) * (0.5 ** np.arange(S))[None, :, None, None]).astype(np.float16)
    books[1, :, K - 1] = books[1, :, K // 2]
    sb = rng.integers(0, nb, ns).astype(np.int32)
    sb[7] = -1
    xd, bd, sd = dev(x), dev(books), dev(sb)
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    sym, res = fkv.fkv_rvq_assign(xd, bd, sd, t0, t0 + n, want_residual=True, n_bad=nbad)
    assert int(host(nbad)[0]) == 1
    codec = fkv.Codec(256)
    fs, fp, fr = fkv.fkv_rvq_assign_encode(codec, xd, bd, sd, t0, t0 + n, want_residual=True)
    bits = lambda t: host(t).view(np.uint32)
    assert torch.equal(fs, sym) and np.array_equal(bits(fr), bits(res))
    some = slice(0, 100)                                # at most 200 items of 256 tokens
    s1, r1 = fkv.fkv_rvq_assign(xd[some], bd, sd[some], t0, t0 + n, want_residual=True)
    assert torch.equal(s1, sym[some]) and np.array_equal(bits(r1), bits(res[some]))
    s2, p2, r2 = fkv.fkv_rvq_assign_encode(codec, xd[some], bd, sd[some], t0, t0 + n, want_residual=True)
    assert torch.equal(s2, sym[some]) and np.array_equal(bits(r2), bits(res[some]))
    assert np.array_equal(host(p2).view(np.uint64), host(fp[some]).view(np.uint64))
    each = dev(np.delete(np.arange(ns, dtype=np.int32), 7)[:, None])
    s3 = sym.clone()
    s3[each[:, 0].long()] = 0x5A
    fkv.fkv_rvq_assign_groups(xd, bd, sd, each, t0, t0 + n, symbols=s3)
    assert torch.equal(s3, sym)


def test_groups_invalid(fkv):
    rng = np.random.default_rng(3)
    d, S, K, T, nb, ns = 64, 2, 64, 20, 2, 6
    x = rng.standard_normal((ns, T, d)).astype(np.float16)
    books = rng.standard_normal((nb, S, K, d)).astype(np.float16)
    sb = np.array([0, 1, 0, 1, 9, 9], np.int32)         # streams 4 and 5 have no book
    xd, bd, sd = dev(x), dev(books), dev(sb)
    full, _ = fkv.fkv_rvq_assign(xd, bd, sd, 2, 19)
    full = host(full)
    groups = np.array([[0, 2], [1, 0], [3, ns + 5], [4, 5], [1, 3]], np.int32)
    sym = torch.full((ns, 17 * S), 0xA5, dtype=torch.uint8, device="cuda")
    res = torch.zeros((ns, 17, d), dtype=torch.float32, device="cuda")
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    # groups 1 (books differ), 2 (a member out of range) and 3 (no valid book) are rejected; group 0 and 4
    # are assigned.  Stream 0 is in a good group and a rejected one, so only its rejection is checked when
    # the rejected group runs alone.
    fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(groups[[2, 3]]), 2, 19, symbols=sym, residual=res, n_bad=nbad)
    got = host(sym)
    assert int(host(nbad)[0]) == 2
    assert (got[[3, 4, 5]] == 0xFF).all() and (got[[0, 1, 2]] == 0xA5).all()
    assert np.isnan(host(res)[[3, 4, 5]]).all()
    nbad.zero_()
    sym.fill_(0xA5)
    fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(groups[[1]]), 2, 19, symbols=sym, n_bad=nbad)
    got = host(sym)
    assert int(host(nbad)[0]) == 1 and (got[[0, 1]] == 0xFF).all() and (got[[2, 3, 4, 5]] == 0xA5).all()
    nbad.zero_()
    sym.fill_(0xA5)
    fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(groups[[0, 4]]), 2, 19, symbols=sym, n_bad=nbad)
    got = host(sym)
    assert int(host(nbad)[0]) == 0
    assert np.array_equal(got[[0, 1, 2, 3]], full[[0, 1, 2, 3]]) and (got[[4, 5]] == 0xA5).all()
    # argument errors; no groups is a no-op
    with pytest.raises(fkv.FkvError):
        fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(np.zeros((1, 257), np.int32)), 2, 19)
    with pytest.raises(fkv.FkvError):
        fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(np.zeros((1, 0), np.int32)), 2, 19)
    sym.fill_(0xA5)
    fkv.fkv_rvq_assign_groups(xd, bd, sd, dev(np.zeros((0, 2), np.int32)), 2, 19, symbols=sym)
    assert (host(sym) == 0xA5).all()


def test_eviction_step_matches_oracle(fkv, orc):
    """The GPT-2-shaped eviction step (all 288 streams' leaving position, grouped by book) against the
    oracle, teacher-forced through near-ties."""
    cfg = w.CONFIGS["gpt2"]
    x, books, sb = w.make_group_numpy(cfg)
    groups = fkv.book_groups(sb)
    t = cfg.t_end - 1
    sym, res = fkv.fkv_rvq_assign_groups(dev(x), dev(books), dev(sb), dev(groups), t, t + 1, want_residual=True)
    sym, res = host(sym), host(res)
    o = orc.rvq_assign(x, books, sb, t, t + 1, force=sym, force_tol=NEAR_TIE)
    assert o["n_hard"] == 0 and np.array_equal(o["symbols"], sym)
    assert np.abs(o["residual"] - res.astype(np.float64)).max() <= 1e-3
    print("eviction step: %d streams, %d groups of %d, near-ties accepted %d"
          % (x.shape[0], groups.shape[0], groups.shape[1], o["n_forced"]))


def test_multi_item_blocks_match_single_item_blocks(fkv):
    """At 2^14 and more work items, three or more stages and d > 128 the per-stream form gives each block 16
    consecutive items and loads the next item's rows during the current item's last stage; the grouped form
    (one stream per group) keeps one item per block with the same arithmetic.  Symbols, residuals and the
    invalid-stream count must agree, with invalid streams between valid ones (an item that ends a block's run
    early)."""
    rng = np.random.default_rng(11)
    ns, T, d, S, K, nb = 128, 32800, 144, 3, 64, 4
    t0, t1 = 4, 32772                                   # 32,768 tokens: 128 items of 256 per stream
    x = torch.from_numpy((rng.standard_normal((ns, T, d)) * 1.2).astype(np.float16)).cuda()
    books = torch.from_numpy((rng.standard_normal((nb, S, K, d)) *
                              (0.5 ** np.arange(S))[None, :, None, None]).astype(np.float16)).cuda()
    sbh = rng.integers(0, nb, ns).astype(np.int32)
    sbh[[3, 40, 41, 127]] = 77                          # no valid book
    sb = torch.from_numpy(sbh).cuda()
    n1 = torch.zeros(1, dtype=torch.int32, device="cuda")
    n2 = torch.zeros(1, dtype=torch.int32, device="cuda")
    s1, r1 = fkv.fkv_rvq_assign(x, books, sb, t0, t1, want_residual=True, n_bad=n1)
    groups = torch.arange(ns, dtype=torch.int32, device="cuda").view(ns, 1)
    s2, r2 = fkv.fkv_rvq_assign_groups(x, books, sb, groups, t0, t1, want_residual=True, n_bad=n2)
    assert int(n1.item()) == int(n2.item()) == 4
    assert torch.equal(s1, s2)
    a, b = host(r1), host(r2)
    assert np.array_equal(np.isnan(a), np.isnan(b))
    assert np.array_equal(np.nan_to_num(a).view(np.uint32), np.nan_to_num(b).view(np.uint32))
    del x, s1, s2, r1, r2
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,S,K,ns,n", [(144, 3, 100, 16403, 33), (256, 4, 256, 16401, 35), (208, 3, 70, 8210, 300)])
def test_multi_item_blocks_of_short_streams(fkv, d, S, K, ns, n):
    """The same with blocks that cross from stream to stream (one ragged item, or a whole and a ragged one, per
    stream), an item count that 16 does not divide and streams without a book inside a block's run, against
    calls of few streams, which give each block one item."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d + n)
    nb, T, t0 = 5, n + 2, 1
    x = torch.randn((ns, T, d), generator=g, device="cuda").half()
    scale = 0.5 ** torch.arange(S, device="cuda")
    books = (torch.randn((nb, S, K, d), generator=g, device="cuda") * scale[None, :, None, None]).half()
    sb = (torch.arange(ns, device="cuda") * 7 % nb).int()
    sb[[0, 18, 19, 5000, ns - 1]] = nb
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    sym, res = fkv.fkv_rvq_assign(x, books, sb, t0, t0 + n, want_residual=True, n_bad=nbad)
    assert int(host(nbad)[0]) == 5
    for a in range(0, ns, 4096):
        s1, r1 = fkv.fkv_rvq_assign(x[a:a + 4096], books, sb[a:a + 4096], t0, t0 + n, want_residual=True)
        assert torch.equal(s1, sym[a:a + 4096])
        assert torch.equal(r1.view(torch.int32), res[a:a + 4096].view(torch.int32))


@pytest.mark.parametrize("d", [144, 160, 192, 208, 240, 256])
def test_first_stages_of_wide_heads(fkv, d):
    """Above d = 128, calls of one or two stages run blocks without the next item's rows, deeper ones with them:
    the first stages' symbols are the same."""
    rng = np.random.default_rng(d)
    ns, T, S, K, nb = 7, 300, 3, 200, 3
    x = (rng.standard_normal((ns, T, d)) * 2).astype(np.float16)
    books = (rng.standard_normal((nb, S, K, d)) * (0.5 ** np.arange(S))[None, :, None, None]).astype(np.float16)
    sb = rng.integers(0, nb, ns).astype(np.int32)
    xd, bd, sd = dev(x), dev(books), dev(sb)
    full = host(fkv.fkv_rvq_assign(xd, bd, sd, 0, T)[0]).reshape(ns, T, S)
    for k in (1, 2):
        sym = torch.full((ns, T * S), 0xA5, dtype=torch.uint8, device="cuda")
        _, res = fkv.fkv_rvq_assign(xd, bd, sd, 0, T, symbols=sym, n_stages=k, want_residual=True)
        got = host(sym).reshape(ns, T, S)
        assert np.array_equal(got[..., :k], full[..., :k]) and (got[..., k:] == 0xA5).all()
        r = x.astype(np.float64)
        for st in range(k):
            r = r - books.astype(np.float64)[sb[:, None], st, full[..., st]]
        assert np.abs(host(res) - r).max() <= 1e-3


@pytest.mark.parametrize("d,S,K,G,n,ng", [
    (128, 3, 130, 3, 75, 270), (128, 2, 256, 4, 100, 140), (96, 4, 256, 5, 45, 300), (80, 3, 256, 4, 37, 280),
    (112, 1, 33, 3, 50, 300), (64, 2, 256, 5, 45, 1540), (64, 4, 200, 3, 83, 280), (16, 3, 100, 3, 77, 300),
])
def test_large_grouped_launches(fkv, d, S, K, G, n, ng):
    """Grouped launches of more items than the wide shape's limits: two token tiles per wave, members that end
    inside a tile (n is not a multiple of 32) and items that hold several members or, at 4 x 100 tokens, split
    them, against the per-stream form a few streams at a time."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d + n)
    ns, nb, T, t0 = ng * G, 9, n + 3, 2
    x = torch.randn((ns, T, d), generator=g, device="cuda").half()
    scale = 0.5 ** torch.arange(S, device="cuda")
    books = (torch.randn((nb, S, K, d), generator=g, device="cuda") * scale[None, :, None, None]).half()
    groups = torch.randperm(ns, generator=g, device="cuda").int().view(ng, G)
    sb = torch.empty(ns, dtype=torch.int32, device="cuda")
    sb[groups.long()] = (torch.arange(ng, device="cuda") % nb).int()[:, None]
    bad = groups[11].long()
    sb[bad] = nb                                        # a group without a book
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    sym, res = fkv.fkv_rvq_assign_groups(x, books, sb, groups, t0, t0 + n, want_residual=True, n_bad=nbad)
    assert int(host(nbad)[0]) == 1 and bool((sym[bad] == 0xFF).all())
    for a in range(0, ns, 200):
        s1, r1 = fkv.fkv_rvq_assign(x[a:a + 200], books, sb[a:a + 200], t0, t0 + n, want_residual=True)
        assert torch.equal(s1, sym[a:a + 200])
        assert torch.equal(r1.view(torch.int32), res[a:a + 200].view(torch.int32))


def test_few_tokens_more_items_than_blocks(fkv):
    """More work items than the few-token kernel has blocks (2^20): a block takes a second item, after one with a
    book and after one without."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    ns, d, S, K, nb = (1 << 20) + 37, 16, 3, 100, 7
    x = torch.randn((ns, 1, d), generator=g, device="cuda").half()
    books = torch.randn((nb, S, K, d), generator=g, device="cuda").half()
    sb = torch.randint(0, nb, (ns,), generator=g, device="cuda", dtype=torch.int32)
    sb[[3, 9, (1 << 20) + 9, (1 << 20) + 12, ns - 1]] = -1
    nbad = torch.zeros(1, dtype=torch.int32, device="cuda")
    sym, res = fkv.fkv_rvq_assign(x, books, sb, 0, 1, want_residual=True, n_bad=nbad)
    assert int(host(nbad)[0]) == 5
    groups = torch.arange(ns, device="cuda", dtype=torch.int32)[:, None].contiguous()
    nbad.zero_()
    s2, r2 = fkv.fkv_rvq_assign_groups(x, books, sb, groups, 0, 1, want_residual=True, n_bad=nbad)
    assert int(host(nbad)[0]) == 5
    assert torch.equal(s2, sym) and torch.equal(r2.view(torch.int32), res.view(torch.int32))
    for a in range(0, ns, 1 << 18):
        s1, r1 = fkv.fkv_rvq_assign(x[a:a + (1 << 18)], books, sb[a:a + (1 << 18)], 0, 1, want_residual=True)
        assert torch.equal(s1, sym[a:a + (1 << 18)])
        assert torch.equal(r1.view(torch.int32), res[a:a + (1 << 18)].view(torch.int32))


@pytest.mark.parametrize("d,S,K,G,n,ng", [
    (16, 3, 100, 1, 32, 600), (16, 3, 64, 3, 4, 100), (64, 3, 64, 4, 4, 100), (64, 1, 192, 2, 1, 300), (64, 4, 33, 2, 5, 600),
    (80, 3, 192, 3, 6, 300), (80, 3, 64, 4, 2, 300), (80, 2, 100, 2, 16, 400), (96, 2, 64, 1, 32, 300), (128, 4, 40, 2, 16, 300),
    (192, 1, 200, 4, 8, 300), (192, 3, 32, 1, 30, 300), (208, 2, 64, 2, 15, 280), (256, 3, 64, 1, 32, 300),
    (16, 3, 192, 1, 20, 1100), (144, 2, 150, 2, 16, 300), (256, 1, 192, 4, 4, 300),
])
def test_few_tokens_of_small_books(fkv, d, S, K, G, n, ng):
    """Calls of at most 32 tokens per group on both sides of the choice between the few-token kernel and the
    staged form (small books, many tokens, one stage), against the staged form over a longer range."""
    rng = np.random.default_rng(d + 5 * S + K + n)
    ns, nb, t0 = ng * G, 4, 3
    T = max(n + 5, 38)
    x = (rng.standard_normal((ns, T, d)) * 2).astype(np.float16)
    books = (rng.standard_normal((nb, S, K, d)) * (0.5 ** np.arange(S))[None, :, None, None]).astype(np.float16)
    sb = np.repeat(rng.integers(0, nb, ng), G).astype(np.int32)
    xd, bd, sd = dev(x), dev(books), dev(sb)
    full, fres = fkv.fkv_rvq_assign(xd, bd, sd, 0, T, want_residual=True)
    full, fres = host(full).reshape(ns, T, S)[:, t0:t0 + n], host(fres)[:, t0:t0 + n]
    groups = dev(np.arange(ns, dtype=np.int32).reshape(ng, G))
    for sym, res in (fkv.fkv_rvq_assign(xd, bd, sd, t0, t0 + n, want_residual=True),
                     fkv.fkv_rvq_assign_groups(xd, bd, sd, groups, t0, t0 + n, want_residual=True)):
        assert np.array_equal(host(sym).reshape(ns, n, S), full)
        assert np.array_equal(host(res).view(np.uint32), fres.view(np.uint32))
