"""GPU parity: topk_select against the oracle -- indices, values and counts bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2411_18873_amd import eck, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _same(got, want):
    gi, ge, gc = got
    wi, we, wc = want
    assert np.array_equal(gc, wc)
    assert np.array_equal(gi, wi)
    assert np.array_equal(ge.view(np.uint32), we.view(np.uint32))


@pytest.mark.parametrize("n,S,k,ties", [(6400, 1, 16, 0.0), (1 << 16, 1, 64, 0.3), ((1 << 16) + 8 * 13, 8, 32, 0.5),
                                        (50000, 1, 1024, 0.9), (4096, 64, 32, 0.2), (100, 1, 100, 0.0), (7, 7, 1, 0.0)])
def test_threshold_mode(G, n, S, k, ties):
    e = synth.gaussian_scores(n, 1, ties=ties, quantum=0.01 if ties else None)
    lat = synth.gaussian_scores(n, 2, ties=ties / 2) * 0.3 + 2.0
    legal = synth.legal_mask(n, 3, 0.4)
    for alpha in (1.1, 1.0, 2.5, float("inf")):
        _same(G.topk_gpu(e, lat, legal, S, k, alpha=alpha), oracle.topk(e, lat, legal, S, k, alpha=alpha))
    _same(G.topk_gpu(e, lat, None, S, k), oracle.topk(e, lat, None, S, k))
    _same(G.topk_gpu(e, None, legal, S, k), oracle.topk(e, None, legal, S, k))
    _same(G.topk_gpu(e, None, None, S, k), oracle.topk(e, None, None, S, k))


def test_negative_latencies_and_mixed_signs(G):
    n = 30000
    e = synth.gaussian_scores(n, 5)
    for shift in (-3.0, 0.0):
        lat = synth.gaussian_scores(n, 6) * 0.2 + shift
        legal = synth.legal_mask(n, 7, 0.5)
        _same(G.topk_gpu(e, lat, legal, 1, 64, alpha=1.1), oracle.topk(e, lat, legal, 1, 64, alpha=1.1))


def test_degenerate_inputs(G):
    n = 20000
    const = np.full(n, 2.5, dtype=np.float32)
    _same(G.topk_gpu(const, None, None, 1, 100), oracle.topk(const, None, None, 1, 100))           # all equal
    _same(G.topk_gpu(const, const, None, 4, 50), oracle.topk(const, const, None, 4, 50))
    e = synth.gaussian_scores(n, 8)
    none_legal = np.zeros(n, dtype=np.uint8)
    _same(G.topk_gpu(e, e, none_legal, 2, 10), oracle.topk(e, e, none_legal, 2, 10))                 # nothing feasible
    few = none_legal.copy()
    few[[5, 77, 19999]] = 1
    _same(G.topk_gpu(e, None, few, 1, 10), oracle.topk(e, None, few, 1, 10))                         # fewer than k
    # NaN, infinities, signed zeros, denormals
    sp = e.copy()
    sp[::7] = np.nan
    sp[1::11] = -0.0
    sp[2::11] = 0.0
    sp[3::13] = -np.inf
    sp[4::13] = np.inf
    sp[5::17] = 1e-42
    lat = np.abs(synth.gaussian_scores(n, 9)) + 0.5
    lat[::5] = np.nan
    _same(G.topk_gpu(sp, lat, None, 1, 4000, alpha=3.0), oracle.topk(sp, lat, None, 1, 4000, alpha=3.0))
    _same(G.topk_gpu(sp, None, None, 1, 4096), oracle.topk(sp, None, None, 1, 4096))
    # two distinct values only: the k-th falls inside a huge tie
    two = (np.arange(n) % 3 == 0).astype(np.float32)
    _same(G.topk_gpu(two, None, None, 1, 4096), oracle.topk(two, None, None, 1, 4096))


@pytest.mark.parametrize("n,S,k,m", [(20000, 1, 50, 500), (1 << 15, 4, 64, 128), (3000, 1, 16, 5000), (5000, 1, 100, 100)])
def test_rank_mode(G, n, S, k, m):
    e = synth.gaussian_scores(n, 11, ties=0.3, quantum=0.05)
    lat = synth.gaussian_scores(n, 12, ties=0.3, quantum=0.05)
    legal = synth.legal_mask(n, 13, 0.6)
    _same(G.topk_gpu(e, lat, legal, S, k, mode=eck.SELECT_RANK, m_latency=m),
          oracle.topk(e, lat, legal, S, k, mode=oracle.SEL_RANK, m_latency=m))
    _same(G.topk_gpu(e, lat, None, S, k, mode=eck.SELECT_RANK, m_latency=m),
          oracle.topk(e, lat, None, S, k, mode=oracle.SEL_RANK, m_latency=m))


def test_children_of_few_parents_tie_heavily(G):
    # like an evolutionary round: 2^18 children of 1024 parents, most of them exact copies
    rng = np.random.default_rng(0)
    parents_e = synth.gaussian_scores(1024, 14)
    parents_l = np.abs(synth.gaussian_scores(1024, 15)) + 1
    n = 1 << 18
    who = np.arange(n) % 1024
    mutated = rng.random(n) < 0.47
    e = np.where(mutated, synth.gaussian_scores(n, 16), parents_e[who]).astype(np.float32)
    lat = np.where(mutated, np.abs(synth.gaussian_scores(n, 17)) + 1, parents_l[who]).astype(np.float32)
    legal = synth.legal_mask(n, 18, 0.8)
    _same(G.topk_gpu(e, lat, legal, 1, 1024, alpha=1.1), oracle.topk(e, lat, legal, 1, 1024, alpha=1.1))


def test_repeatable(G):
    n = 1 << 18
    e = synth.gaussian_scores(n, 21, ties=0.5, quantum=0.001)
    lat = np.abs(synth.gaussian_scores(n, 22)) + 1
    a = G.topk_gpu(e, lat, None, 4, 512)
    b = G.topk_gpu(e, lat, None, 4, 512)
    _same(a, b)


def test_scalar_and_vector_streaming_paths_agree_with_the_oracle(G):
    """The streaming kernels read four candidates per load when segment length and pointers allow it and one
    per load otherwise: odd segment lengths, and score / flag arrays that start one element into an allocation,
    take the scalar path at a size that spans many blocks; the result is the oracle's either way."""
    import torch
    S, seg = 3, 123457                                   # odd segment length
    n = S * seg
    e = synth.gaussian_scores(n, 11, ties=0.2, quantum=0.01)
    lat = synth.gaussian_scores(n, 12) * 0.3 + 2.0
    legal = synth.legal_mask(n, 13, 0.5)
    want = oracle.topk(e, lat, legal, S, 200, alpha=1.1)
    _same(G.topk_gpu(e, lat, legal, S, 200, alpha=1.1), want)
    # aligned length, misaligned pointers: views that start at element 1
    n2 = 1 << 18
    e2, l2, g2 = e[:n2], lat[:n2], legal[:n2]
    want2 = oracle.topk(e2, l2, g2, 4, 77, alpha=1.1)
    pad_f = lambda a: torch.cat([torch.zeros(1, dtype=torch.float32), torch.from_numpy(a.copy())]).cuda()[1:]
    pad_b = torch.cat([torch.zeros(1, dtype=torch.uint8), torch.from_numpy(g2.copy())]).cuda()[1:]
    assert pad_f(e2).data_ptr() % 16 != 0
    _same(G.topk_dev(pad_f(e2), pad_f(l2), pad_b, 4, 77, alpha=1.1), want2)
    # and the aligned (vector) path on the same data
    _same(G.topk_gpu(e2, l2, g2, 4, 77, alpha=1.1), want2)


@pytest.mark.parametrize("n,S,k", [(1 << 22, 1, 4096), (1 << 22, 1, 300), (1 << 22, 1, 1), (3 * ((1 << 20) + 4), 3, 257),
                                   (1 << 21, 512, 16), (40000, 1, 4096)])
def test_selections_that_take_several_levels(G, n, S, k):
    """A block selects among 4096 (k <= 256 on a full chip) or 16384 candidates; longer segments go through
    further levels over the lists of the level before.  Sizes here take one to four levels, with k from 1 to the
    largest the library accepts, ties included so that index digits decide."""
    e = synth.gaussian_scores(n, 31, ties=0.4, quantum=0.02)
    lat = synth.gaussian_scores(n, 32) * 0.3 + 2.0
    legal = synth.legal_mask(n, 33, 0.7)
    _same(G.topk_gpu(e, None, legal, S, k), oracle.topk(e, None, legal, S, k))
    _same(G.topk_gpu(e, lat, legal, S, k, alpha=1.3), oracle.topk(e, lat, legal, S, k, alpha=1.3))
    m = min(4096, max(k, 1000))
    _same(G.topk_gpu(e, lat, legal, S, k, mode=eck.SELECT_RANK, m_latency=m),
          oracle.topk(e, lat, legal, S, k, mode=oracle.SEL_RANK, m_latency=m))


def test_rank_gate_limits_and_workspace(G):
    import ctypes as C
    import torch
    L = eck.lib()
    n = 1 << 16
    # a gate wider than the library's largest selection is refused unless it admits the whole segment anyway
    assert L.topk_select_rank_workspace_bytes(n, 1, 16, 5000) == 0
    assert L.topk_select_rank_workspace_bytes(n, 1, 16, n) > 0
    assert L.topk_select_rank_workspace_bytes(n, 1, 16, 0) == 0
    need = eck.topk_select_workspace_bytes(n, 1, 16, m_latency=4096)
    assert need >= eck.topk_select_workspace_bytes(n, 1, 16)
    e = torch.zeros(n, dtype=torch.float32, device="cuda")
    idx = torch.zeros(16, dtype=torch.int32, device="cuda")
    eo = torch.zeros(16, dtype=torch.float32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    p = lambda t: C.c_void_p(t.data_ptr())
    call = lambda m, ws_bytes: L.topk_select(p(e), p(e), None, n, 1, 16, eck.SELECT_RANK, 1.1, m, p(idx), p(eo), p(cnt),
                                             p(ws), ws_bytes, None)
    assert call(5000, need) == eck.EUNSUPPORTED
    assert call(4096, eck.topk_select_workspace_bytes(n, 1, 16) - 8) == eck.EWORKSPACE
    assert call(4096, need) == eck.OK and call(n, need) == eck.OK
    torch.cuda.synchronize()
    assert cnt.item() == 16 and idx.cpu().numpy().tolist() == list(range(16))


@pytest.mark.parametrize("segments,seg_len,k,m", [(1, 40, 1, 1), (3, 1000, 511, 512), (1, 16384, 512, 513), (1, 16385, 513, 514),
                                                  (2, 70001, 100, 2000), (1, 300000, 1500, 4096), (5, 4097, 300, 256),
                                                  (64, 20000, 7, 255), (1, 9000, 4000, 4096)])
@pytest.mark.parametrize("odd", [False, True])
def test_rank_gate_and_energies_in_one_tournament(G, segments, seg_len, k, m, odd):
    """gates around the sizes where the block's method changes, segments that one block holds and segments of several
    levels; ties in latency and energy; odd: few legal candidates (fewer than the gate in some segments, none in the last),
    NaN energies among the fastest, infinities, NaN latencies"""
    rng = np.random.default_rng(seg_len + k)
    n = segments * seg_len
    energy = (np.round(rng.standard_normal(n) * 50) / 50).astype(np.float32)
    latency = (np.round(rng.standard_normal(n) * 200) / 200).astype(np.float32)
    legal = None
    if odd:
        legal = (rng.random(n) < min(1.0, 0.7 * m / seg_len)).astype(np.uint8)
        legal[n - seg_len:] = 0
        for values in (energy, latency):
            where = rng.random(n) < 0.1
            values[where] = rng.choice(np.array([np.nan, np.inf, -np.inf, -0.0, 0.0], dtype=np.float32), int(where.sum()))
    got = G.topk_gpu(energy, latency, legal, segments, k, mode=eck.SELECT_RANK, m_latency=m)
    want = oracle.topk(energy, latency, legal, segments, k, mode=oracle.SEL_RANK, m_latency=m)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    # and the gate of the threshold mode where one block finds the least latency of its segment itself
    with np.errstate(invalid="ignore"):
        got = G.topk_gpu(energy, latency, legal, segments, k, alpha=1.3)
        want = oracle.topk(energy, latency, legal, segments, k, alpha=1.3)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("segments,seg_len,k,m", [(1, 6400, 1, 4096), (1, 16384, 64, 513), (3, 16384, 512, 4096), (64, 4096, 33, 600),
                                                  (1, 1 << 18, 64, 4096), (5, 700, 17, 640)])
@pytest.mark.parametrize("few", [False, True])
def test_energies_of_wide_gates(G, segments, seg_len, k, m, few):
    """More gated candidates than are ranked directly, of which the block bounds the energies before it selects: distinct
    energies, and few distinct ones (ties by the thousand at the bound); NaN energies and unlaunchable candidates, by which a
    segment may have fewer than the gate admits or than are asked for."""
    rng = np.random.default_rng(seg_len + k + m)
    n = segments * seg_len
    e = rng.standard_normal(n).astype(np.float32)
    lat = (rng.random(n) + 0.5).astype(np.float32)
    if few:
        e = np.round(e).astype(np.float32)
        lat = np.round(lat * 8).astype(np.float32)
        e[rng.random(n) < 0.3] = np.nan
    legal = (rng.random(n) < 0.8).astype(np.uint8)
    legal[n - seg_len // 2:] = 0
    _same(G.topk_gpu(e, lat, legal, segments, k, mode=eck.SELECT_RANK, m_latency=m),
          oracle.topk(e, lat, legal, segments, k, mode=oracle.SEL_RANK, m_latency=m))


@pytest.mark.parametrize("segments,seg_len,k", [(1, 16385, 7), (3, 20000, 512), (64, 65536, 32), (2, 70001, 1), (5, 40000, 600)])
@pytest.mark.parametrize("kind", ["few", "all", "rising", "falling", "negative", "none"])
def test_candidates_listed_under_the_gate(G, segments, seg_len, k, kind):
    """The pass that finds the least latency also lists what lies under the gate of each chunk's own minimum.  few: short
    lists; all: every list overflows; rising, falling: only the first or the last chunk holds anything under the segment's
    gate; negative latencies under alpha = 3.5, where a smaller minimum has the higher gate; no legal candidate in some
    segments.  With the workspace of the query, and with one that does not hold the lists."""
    import torch
    rng = np.random.default_rng(seg_len + k)
    n = segments * seg_len
    e = rng.standard_normal(n).astype(np.float32)
    lat = {"few": 2.0 + 0.4 * rng.standard_normal(n), "all": 10.0 + 0.05 * rng.standard_normal(n),
           "negative": -3.0 + rng.standard_normal(n)}.get(kind, 1.0 + rng.random(n)).astype(np.float32)
    if kind in ("rising", "falling"):
        lat = np.sort(lat.reshape(segments, -1), axis=1)[:, ::1 if kind == "rising" else -1].reshape(-1).copy()
    lat[rng.random(n) < 0.01] = np.nan
    e[rng.random(n) < 0.01] = np.nan
    legal = (rng.random(n) < 0.3).astype(np.uint8)
    if kind == "none":
        legal[:seg_len] = 0
    alpha = 3.5 if kind == "negative" else 1.1
    want = oracle.topk(e, lat, legal, segments, k, alpha=alpha)
    _same(G.topk_gpu(e, lat, legal, segments, k, alpha=alpha), want)
    _same(G.topk_gpu(e, lat, None, segments, k, alpha=alpha), oracle.topk(e, lat, None, segments, k, alpha=alpha))
    # the call takes the smaller workspace that a selection without the lists needs
    full = eck.topk_select_workspace_bytes(n, segments, k)
    chunks = segments * -(-seg_len // 4096)
    ed, ld, gd = G.to_dev(e), G.to_dev(lat), G.to_dev(legal)
    idx = torch.zeros((segments, k), dtype=torch.int32, device="cuda")
    eo = torch.zeros((segments, k), device="cuda")
    cnt = torch.zeros(segments, dtype=torch.int32, device="cuda")
    ws = torch.empty(full - chunks * (8 * 128 + 8), dtype=torch.uint8, device="cuda")
    eck.topk_select(ed, ld, gd, segments, k, idx, eo, cnt, ws, alpha=alpha)
    torch.cuda.synchronize()
    _same((idx.cpu().numpy().view(np.uint32), eo.cpu().numpy(), cnt.cpu().numpy().view(np.uint32)), want)


@pytest.mark.parametrize("segments,seg_len,k", [(1, 4096, 64), (1, 4096, 65), (1, 4097, 33), (2, 8192, 256), (2, 8193, 257), (1, 16385, 48),
                                                (1, 16388, 49), (1, 300000, 100), (3, 70000, 250), (1, 200004, 513), (2, 150000, 1000),
                                                (130, 16400, 3), (1, 1 << 20, 128), (1, (1 << 20) + 1, 129), (1, 16384, 1024), (4, 1030, 1025)])
@pytest.mark.parametrize("order", ["random", "rising", "falling", "few"])
def test_block_sizes_and_list_shares(G, segments, seg_len, k, order):
    """Both sides of the lines between block sizes, lists that go into the threads of the next level evenly and not, and
    pools of more entries than a block has threads.  In ascending or descending order one block holds the whole selection
    and no bound is tight; few distinct values tie by the thousand."""
    rng = np.random.default_rng(seg_len + k)
    n = segments * seg_len
    e = rng.standard_normal(n).astype(np.float32)
    lat = (1.0 + rng.random(n)).astype(np.float32)
    if order == "few":
        e, lat = np.round(e).astype(np.float32), np.round(lat * 8).astype(np.float32)
    elif order != "random":
        step = 1 if order == "rising" else -1
        e, lat = (np.sort(v.reshape(segments, -1), axis=1)[:, ::step].reshape(-1).copy() for v in (e, lat))
    legal = (rng.random(n) < 0.5).astype(np.uint8)
    _same(G.topk_gpu(e, None, legal, segments, k), oracle.topk(e, None, legal, segments, k))
    _same(G.topk_gpu(e, lat, None, segments, k, alpha=1.2), oracle.topk(e, lat, None, segments, k, alpha=1.2))
    if k <= 1000:
        _same(G.topk_gpu(e, lat, legal, segments, max(1, k // 2), mode=eck.SELECT_RANK, m_latency=k),
              oracle.topk(e, lat, legal, segments, max(1, k // 2), mode=oracle.SEL_RANK, m_latency=k))


@pytest.mark.parametrize("segments,seg_len", [(131, 16388), (131, 16385), (20, 16388), (1, 70000), (300, 4100), (2, 1500000)])
@pytest.mark.parametrize("k", [5, 300, 1100])
@pytest.mark.parametrize("alpha", [1.0, 1.1, 3.5])
def test_long_lists_above_the_gate(G, segments, seg_len, k, alpha):
    """Chunks whose own minimum admits more than a list holds, but which lie above the segment's gate; next to them segments that
    admit everything, little, nothing legal, or have no gate (an infinite least latency, negative ones); launches of more blocks
    than compute units, where those of 1024 threads share one, and of fewer."""
    rng = np.random.default_rng(seg_len + k)
    n = segments * seg_len
    e = rng.standard_normal(n).astype(np.float32)
    lat = (1.0 + rng.random((segments, seg_len))).astype(np.float32)
    legal = (rng.random((segments, seg_len)) < 0.3).astype(np.uint8)
    for s in range(segments):
        kind = (s + seg_len) % 7
        if kind < 2:
            lat[s] = np.sort(lat[s])[::1 if kind == 0 else -1]
        elif kind == 2:
            lat[s] = 10 + lat[s] / 100
        elif kind == 3:
            lat[s] -= 3
        elif kind == 4:
            lat[s, rng.random(seg_len) < 0.9] = np.inf
            lat[s, rng.random(seg_len) < 0.5] = np.nan
        elif kind == 5:
            (lat if s % 2 else legal)[s] = np.inf if s % 2 else 0
    lat, legal = lat.reshape(-1), legal.reshape(-1)
    _same(G.topk_gpu(e, lat, legal, segments, k, alpha=alpha), oracle.topk(e, lat, legal, segments, k, alpha=alpha))
