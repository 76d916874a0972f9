"""GPU parity of in-archive retrieval (Sec. 5) against the CPU oracle: the
per-position index bit for bit, and suffix-search hit sets, hit counts and
candidate counts exactly (hit order is unspecified on the GPU)."""
import numpy as np
import pytest
import torch

from paper_2607_07144_amd import workloads as w

pytestmark = pytest.mark.gpu


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _search(fkv, codec, traj, q, verify, max_hits=1 << 16):
    hits, nh, nc = fkv.fkv_suffix_search(codec, traj, torch.from_numpy(q).cuda(), verify=verify,
                                         max_hits=max_hits)
    n = int(nh.item())
    got = host(hits)[:min(n, max_hits)].view(np.uint32)
    return sorted(map(tuple, got.tolist())), n, int(nc.item())


@pytest.mark.parametrize("N,W", [(16, 0), (64, 0), (256, 0), (3, 64), (256, 11), (256, 1), (64, 16), (64, 17),
                                 (256, 8), (64, 5), (16, 2)])
def test_trajectory_matches_oracle(fkv, orc, N, W):
    rng = np.random.default_rng(N + W)
    sym = rng.integers(0, N, (5, 1000 + 37), dtype=np.uint8)     # a ragged last tile
    codec = fkv.Codec(N)
    Wv = W or codec.L
    tr = fkv.fkv_trajectory(codec, torch.from_numpy(sym).cuda(), Wv)
    want = orc.trajectory(orc.Codec(N), sym, Wv)
    assert np.array_equal(host(tr).view(np.uint64), want.view(np.uint64))


@pytest.mark.parametrize("n_sym,W", [(1, 6), (3, 6), (5, 6), (6, 6), (7, 8), (255, 6), (256, 6), (257, 8),
                                     (1023, 6), (1024, 3), (1025, 8)])
def test_trajectory_short_streams(fkv, orc, n_sym, W):
    """Streams shorter than, equal to and just past the window, and around the 256-position tile."""
    rng = np.random.default_rng(n_sym * 3 + W)
    sym = rng.integers(0, 256, (3, n_sym), dtype=np.uint8)
    codec = fkv.Codec(256)
    tr = fkv.fkv_trajectory(codec, torch.from_numpy(sym).cuda(), W)
    want = orc.trajectory(orc.Codec(256), sym, W)
    assert np.array_equal(host(tr).view(np.uint64), want.view(np.uint64))


@pytest.mark.parametrize("ns,n_sym,N,W", [(512, 37, 256, 6), (512, 3, 256, 6), (257, 2049, 256, 6), (171, 4100, 64, 9),
                                          (256, 2051, 16, 16), (130, 6145, 256, 7), (512, 2047, 3, 64)])
def test_trajectory_large_tiles(fkv, orc, ns, n_sym, N, W):
    """Streams around the length of a 2048-position tile, shorter than a tile or the window, odd stream lengths
    (every byte alignment), symbols outside the alphabet."""
    rng = np.random.default_rng(ns + n_sym)
    sym = rng.integers(0, N, (ns, n_sym), dtype=np.uint8)
    want = orc.trajectory(orc.Codec(N), sym, W)
    if N < 256:
        sym[1, n_sym // 2] = N          # NaN points while it is in the window
        want[1, n_sym // 2:n_sym // 2 + W] = np.nan
    tr = host(fkv.fkv_trajectory(fkv.Codec(N), torch.from_numpy(sym).cuda(), W))
    bad = np.isnan(want)
    assert np.array_equal(np.isnan(tr), bad)
    assert np.array_equal(tr.view(np.uint64)[~bad], want.view(np.uint64)[~bad])


@pytest.mark.parametrize("ns,n_sym,N,W", [
    (171, 5400, 16, 16), (171, 5400, 64, 9),              # tiles without, with and next to a stream's start
    (400000, 3, 256, 6), (100003, 17, 16, 16), (24001, 40, 64, 9), (1000003, 1, 256, 6),   # many starts per tile
    (4490, 2047, 256, 6), (4600, 2049, 64, 9), (449, 2048, 16, 16),                        # around the tile's length
    (66000, 70, 256, 64), (1000, 9, 256, 64), (3, 255, 16, 16), (5, 257, 64, 9), (90, 31, 16, 16),   # long windows, small tiles
])
def test_trajectory_tiles_cross_streams(fkv, orc, ns, n_sym, N, W):
    """Tiles run over the streams as they lie: short windows at every place of a tile, 256- and 2048-position
    tiles, a symbol outside the alphabet at a stream's end (the next stream's windows do not hold it)."""
    rng = np.random.default_rng(ns + 3 * n_sym + N)
    sym = rng.integers(0, N, (ns, n_sym), dtype=np.uint8)
    want = orc.trajectory(orc.Codec(N), sym, W)
    if N < 256:
        sym[ns // 2, -1] = N
        want[ns // 2, -1] = np.nan
    tr = host(fkv.fkv_trajectory(fkv.Codec(N), torch.from_numpy(sym).cuda(), W))
    bad = np.isnan(want)
    assert np.array_equal(np.isnan(tr), bad)
    assert np.array_equal(tr.view(np.uint64)[~bad], want.view(np.uint64)[~bad])


@pytest.mark.parametrize("N", [16, 64, 256])
def test_suffix_search_matches_oracle(fkv, orc, N):
    rng = np.random.default_rng(7 * N)
    used = min(N, 8)
    sym = rng.integers(0, used, (6, 5000), dtype=np.uint8)
    codec = fkv.Codec(N)
    oc = orc.Codec(N)
    tr = fkv.fkv_trajectory(codec, torch.from_numpy(sym).cuda())
    trh = orc.trajectory(oc, sym, oc.L)
    for ell in range(1, codec.L + 1):
        s, k = int(rng.integers(0, 6)), int(rng.integers(ell - 1, 5000))
        q = sym[s, k - ell + 1:k + 1].copy()
        for verify in (True, False):
            got, n, nc = _search(fkv, codec, tr, q, verify)
            wh, wn, wc = orc.suffix_search(oc, trh, q, verify=verify)
            assert n == wn and nc == wc and got == sorted(map(tuple, wh.tolist())), (ell, verify)
            if verify:
                assert (s, k) in got


def test_suffix_search_limits(fkv, orc):
    codec = fkv.Codec(16)
    rng = np.random.default_rng(2)
    sym = rng.integers(0, 2, (2, 3000), dtype=np.uint8)             # a two-letter stream: many hits
    tr = fkv.fkv_trajectory(codec, torch.from_numpy(sym).cuda())
    q = np.array([1, 0], np.uint8)
    full, n, _ = _search(fkv, codec, tr, q, True)
    capped, n2, _ = _search(fkv, codec, tr, q, True, max_hits=100)
    assert n2 == n > 100 and len(capped) == 100 and set(capped) <= set(full)
    none, n3, c3 = _search(fkv, codec, tr, np.array([1, 99], np.uint8), True)   # symbol >= N
    assert n3 == 0 and c3 == 0 and none == []


def test_read_stress_index_and_search(fkv, orc):
    """The read-side stress archive (144 streams x 262,144 symbols): the whole index on the GPU,
    a sample of streams bit for bit, and suffix queries over the full index."""
    c = w.READ_STRESS
    sym_h, _, _ = w.read_stress_inputs()
    codec = fkv.Codec(c["N"])
    oc = orc.Codec(c["N"])
    tr = fkv.fkv_trajectory(codec, torch.from_numpy(sym_h).cuda())
    sample = [0, 77, 143]
    trd = host(tr[torch.as_tensor(sample, device="cuda")])
    assert np.array_equal(trd.view(np.uint64), orc.trajectory(oc, sym_h[sample], oc.L).view(np.uint64))
    trh = host(tr)
    rng = np.random.default_rng(c["seed"] + 3)
    for ell in (2, 3, 4):
        s, k = int(rng.integers(0, 144)), int(rng.integers(ell, sym_h.shape[1]))
        q = sym_h[s, k - ell + 1:k + 1].copy()
        got, n, nc = _search(fkv, codec, tr, q, True)
        wh, wn, wc = orc.suffix_search(oc, trh, q, verify=True)
        assert n == wn and nc == wc and got == sorted(map(tuple, wh.tolist())) and (s, k) in got
