"""GPU parity: candidate_enumerate and features_compute against the oracle, bit for bit."""
import itertools
import math

import numpy as np
import pytest

import oracle
from paper_2411_18873_amd import eck, synth

pytestmark = pytest.mark.gpu



@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _spaces(name_or_pb, kind):
    pb = synth.CONFIGS[name_or_pb]["problem"] if isinstance(name_or_pb, str) else name_or_pb
    return eck.Space(pb, kind), oracle.Space(pb, kind)


def test_exhaustive_c1(G):
    mine, ref = _spaces("c1", eck.SPACE_KNOB)
    got = G.enumerate_gpu(mine, eck.MODE_EXHAUSTIVE, 6400)
    want = oracle.enumerate_candidates(ref, oracle.MODE_EXHAUSTIVE, 6400)
    assert np.array_equal(got[:, :6400], want)
    got = G.enumerate_gpu(mine, eck.MODE_EXHAUSTIVE, 777, first_index=5000, ld=1000)
    assert np.array_equal(got[:, :777], want[:, 5000:5777])
    assert np.all(got[:, 777:] == 0xFFFF)  # nothing written past n


@pytest.mark.parametrize("cfg,n,first", [("c2", (1 << 16) + 37, 0), ("c3", 5001, (1 << 40) + 3), ("c1", 3000, 10)])
def test_sample(G, cfg, n, first):
    kind = eck.SPACE_KNOB if cfg == "c1" else eck.SPACE_SPLIT
    mine, ref = _spaces(cfg, kind)
    got = G.enumerate_gpu(mine, eck.MODE_SAMPLE, n, seed=2024, rnd=3, first_index=first)
    want = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, n, seed=2024, rnd=3, first_index=first)
    assert np.array_equal(got[:, :n], want)


def test_sample_sweep_shapes(G):
    for i, (m, n_, k) in enumerate(synth.sweep_shapes()[::9]):
        mine, ref = _spaces(synth.gemm(m, n_, k), eck.SPACE_SPLIT)
        got = G.enumerate_gpu(mine, eck.MODE_SAMPLE, 4099, seed=100 + i)
        want = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, 4099, seed=100 + i)
        assert np.array_equal(got[:, :4099], want)


@pytest.mark.parametrize("p_mut", [synth.P_MUT_Q32, 0, 0xFFFFFFFF])
def test_mutate(G, p_mut):
    mine, ref = _spaces("c3", eck.SPACE_SPLIT)
    parents = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, 1024, seed=7)
    n = (1 << 16) + 11
    for rnd, first in [(1, 0), (5, 123457)]:
        got = G.enumerate_gpu(mine, eck.MODE_MUTATE, n, seed=7, rnd=rnd, first_index=first, parents=parents,
                              p_mut_q32=p_mut)
        want = oracle.enumerate_candidates(ref, oracle.MODE_MUTATE, n, seed=7, rnd=rnd, first_index=first,
                                           parents=parents, p_mut_q32=p_mut)
        assert np.array_equal(got[:, :n], want)


def _check_features(G, mine, ref, genes, n_feat):
    n = genes.shape[1]
    if n & 1:
        genes = np.concatenate([genes, genes[:, :1]], axis=1)
    raw_o, f32_o, b16_o, legal_o = oracle.features(ref, genes, n_feat, n=n)
    raw_g, f32_g, legal_g = G.features_gpu(mine, genes, n, n_feat, eck.F32)
    _, b16_g, legal_g2 = G.features_gpu(mine, genes, n, n_feat, eck.BF16, want_raw=False)
    differs = np.nonzero((raw_g[:, :n] != raw_o[:, :n]).any(axis=1))[0]
    assert differs.size == 0, "raw features that differ: %s" % differs
    assert np.array_equal(f32_g[:, :n].view(np.uint32), f32_o[:, :n].view(np.uint32))
    assert np.array_equal(b16_g[:, :n], b16_o[:, :n])
    assert np.array_equal(legal_g, legal_o) and np.array_equal(legal_g2, legal_o)
    return raw_o, legal_o


def test_features_c1_all(G):
    mine, ref = _spaces("c1", eck.SPACE_KNOB)
    genes = oracle.enumerate_candidates(ref, oracle.MODE_EXHAUSTIVE, 6400)
    _check_features(G, mine, ref, genes, 32)
    _check_features(G, mine, ref, genes, 64)
    # fp32 elements and the case-study machine (Table 5 configuration)
    pb = synth.gemm(512, 512, 512, elem_bytes=4, hw=synth.HW_CASE_STUDY)
    _check_features(G, *_spaces(pb, eck.SPACE_KNOB), genes, 64)
    # a problem that is not a multiple of any tile
    _check_features(G, *_spaces(synth.bgemm(3, 100, 77, 130), eck.SPACE_KNOB), genes, 64)


@pytest.mark.parametrize("cfg,n", [("c2", (1 << 16) + 37), ("c3", (1 << 15) + 1)])
def test_features_split_spaces(G, cfg, n):
    mine, ref = _spaces(cfg, eck.SPACE_SPLIT)
    genes = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, n, seed=11)
    raw, legal = _check_features(G, mine, ref, genes, 64)
    assert 0 < legal.mean() < 1


def test_features_sweep_shapes_and_odd_problems(G):
    for i, (m, n_, k) in enumerate(synth.sweep_shapes()[::7]):
        mine, ref = _spaces(synth.gemm(m, n_, k), eck.SPACE_SPLIT)
        genes = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, 2048, seed=i)
        _check_features(G, mine, ref, genes, 64)
    odd = [synth.conv2d(2, 4, 8, 6, 6, 3, 3, 1, 1, elem_bytes=4, hw=(8, 64, 65536, 1024, 16)),
           synth.conv2d(4, 96, 60, 30, 27, 5, 3, 2, 2),
           synth.conv2d(16, 64, 64, 56, 56, 1, 1, 1, 0, elem_bytes=4),
           synth.bgemm(2, 8, 12, 6, elem_bytes=2, hw=(4, 64, 1024, 256, 8)),
           synth.gemm(1, 4096, 1024, elem_bytes=4),
           synth.gemm(60060, 2, 2)]  # 10240 factorisations: the table stays in global memory
    for pb in odd:
        mine, ref = _spaces(pb, eck.SPACE_SPLIT)
        n = min(ref.size, 3001)
        mode = oracle.MODE_EXHAUSTIVE if ref.size <= 3001 else oracle.MODE_SAMPLE
        genes = oracle.enumerate_candidates(ref, mode, n, seed=5)
        _check_features(G, mine, ref, genes, 64)


def test_features_hand_worked_schedules(G, golden):
    def gene_of(extent, tup):
        divs = [d for d in range(1, extent + 1) if extent % d == 0]
        return sorted(t for t in itertools.product(divs, repeat=4) if math.prod(t) == extent).index(tuple(tup))
    rows = golden("hand_conv.txt")
    pb = synth.conv2d(2, 4, 8, 6, 6, 3, 3, 1, 1, elem_bytes=4, hw=(8, 64, 65536, 1024, 16))
    mine = eck.Space(pb, eck.SPACE_SPLIT)
    g = [gene_of(2, (1, 2, 1, 1)), gene_of(8, (1, 4, 2, 1)), gene_of(6, (3, 2, 1, 1)), gene_of(6, (1, 3, 1, 2)),
         gene_of(4, (2, 1, 1, 2)), 2, 1]
    genes = np.array([g, g], dtype=np.uint16).T.copy()
    raw, _, legal = G.features_gpu(mine, genes, 2, 64, eck.F32)
    assert [int(v) for v in raw[:, 0]] == [int(t) for t in rows[0]] and legal[0] == int(rows[1][0])
    rows = golden("hand_bgemm.txt")
    pb = synth.bgemm(2, 8, 12, 6, elem_bytes=2, hw=(4, 64, 1024, 256, 8))
    mine = eck.Space(pb, eck.SPACE_SPLIT)
    g = [gene_of(2, (1, 1, 2, 1)), gene_of(8, (2, 2, 1, 2)), gene_of(12, (1, 3, 2, 2)), gene_of(6, (3, 1, 2, 1)), 1, 1]
    genes = np.array([g, g], dtype=np.uint16).T.copy()
    raw, _, legal = G.features_gpu(mine, genes, 2, 64, eck.F32)
    assert [int(v) for v in raw[:, 1]] == [int(t) for t in rows[0]] and legal[1] == int(rows[1][0])


def test_table5_counters_on_gpu(G, golden):
    pb = synth.gemm(512, 512, 512, elem_bytes=4, hw=synth.HW_CASE_STUDY)
    mine = eck.Space(pb, eck.SPACE_KNOB)
    tiles, threads = [16, 32, 64, 128, 256], [64, 128, 256, 512]
    for row in golden("table5_case_study.txt"):
        tm, tn, thr, grid, block, glb_ld, glb_st, _, shared_st = (int(t) for t in row[1:])
        g = [tiles.index(tm), tiles.index(tn), 1, threads.index(thr), 0, 0]
        raw, _, _ = G.features_gpu(mine, np.array([g, g], dtype=np.uint16).T.copy(), 2, 32, eck.F32)
        assert (raw[6, 0], raw[7, 0], raw[15, 0], raw[19, 0]) == (grid, block, glb_ld, shared_st)
        if row[0] == "K2":
            assert raw[16, 0] == glb_st


@pytest.mark.parametrize("mode", [eck.MODE_SAMPLE, eck.MODE_MUTATE])
def test_batched_spaces_match_the_oracle_space_by_space(G, mode):
    """One launch over several spaces: each space's column block equals the oracle's output for that space,
    seed and parent block; the padding columns beyond n_spaces*n stay untouched."""
    import torch
    problems = [synth.gemm(*s) for s in synth.sweep_shapes()[::13]] + [synth.gemm(100, 77, 130)]
    mine = [eck.Space(pb, eck.SPACE_SPLIT) for pb in problems]
    refs = [oracle.Space(pb, oracle.SPACE_SPLIT) for pb in problems]
    S, n, P = len(problems), 1537, 24      # n spans several blocks with a ragged tail; odd on purpose
    ld = S * n + 5
    ld += ld & 1
    seeds = [900 + 17 * s for s in range(S)]
    parents = None
    if mode == eck.MODE_MUTATE:
        parents = np.concatenate([oracle.enumerate_candidates(r, oracle.MODE_SAMPLE, P, seed=3 + s)
                                  for s, r in enumerate(refs)], axis=1)
    genes = torch.full((mine[0].n_genes, ld), -1, dtype=torch.int16, device="cuda")
    eck.candidate_enumerate_batch(mine, mode, n, genes, seeds, round=2, first_index=77,
                                  parents=None if parents is None else G.to_dev(parents),
                                  p_mut_q32=synth.P_MUT_Q32)
    feat = torch.zeros((64, ld), dtype=torch.bfloat16, device="cuda")
    raw = torch.zeros((64, ld), dtype=torch.int64, device="cuda")
    legal = torch.full((ld,), 7, dtype=torch.uint8, device="cuda")
    eck.features_compute_batch(mine, genes, n, 64, eck.BF16, feat_out=feat, raw_out=raw, legal_out=legal)
    torch.cuda.synchronize()
    genes_h = genes.cpu().numpy().view(np.uint16)
    feat_h = feat.view(torch.int16).cpu().numpy().view(np.uint16)
    raw_h, legal_h = raw.cpu().numpy().view(np.uint64), legal.cpu().numpy()
    for s, ref in enumerate(refs):
        cols = slice(s * n, (s + 1) * n)
        want = oracle.enumerate_candidates(ref, mode, n, seed=seeds[s], rnd=2, first_index=77,
                                           parents=None if parents is None else parents[:, s * P:(s + 1) * P],
                                           p_mut_q32=synth.P_MUT_Q32)
        assert np.array_equal(genes_h[:, cols], want), "space %d" % s
        padded = np.concatenate([want, want[:, :1]], axis=1)
        raw_o, _, b16_o, legal_o = oracle.features(ref, padded, 64, n=n)
        assert np.array_equal(raw_h[:, cols], raw_o[:, :n]), "space %d" % s
        assert np.array_equal(feat_h[:, cols], b16_o[:, :n]), "space %d" % s
        assert np.array_equal(legal_h[cols], legal_o), "space %d" % s
    assert np.all(genes_h[:, S * n:] == 0xFFFF) and np.all(legal_h[S * n:] == 7) and np.all(raw_h[:, S * n:] == 0)


def test_batched_knob_spaces_and_single_space_batch(G):
    import torch
    pbs = [synth.gemm(512, 512, 512), synth.gemm(384, 1000, 96)]
    mine = [eck.Space(pb, eck.SPACE_KNOB) for pb in pbs]
    refs = [oracle.Space(pb, oracle.SPACE_KNOB) for pb in pbs]
    n = 700
    genes = torch.zeros((mine[0].n_genes, 2 * n), dtype=torch.int16, device="cuda")
    eck.candidate_enumerate_batch(mine, eck.MODE_EXHAUSTIVE, n, genes, [0, 0], first_index=1000)
    feat = torch.zeros((32, 2 * n), dtype=torch.float32, device="cuda")
    eck.features_compute_batch(mine, genes, n, 32, eck.F32, feat_out=feat)
    one = torch.zeros((mine[0].n_genes, n), dtype=torch.int16, device="cuda")
    eck.candidate_enumerate_batch(mine[1:], eck.MODE_SAMPLE, n, one, [5])
    torch.cuda.synchronize()
    genes_h = genes.cpu().numpy().view(np.uint16)
    for s, ref in enumerate(refs):
        want = oracle.enumerate_candidates(ref, oracle.MODE_EXHAUSTIVE, n, first_index=1000)
        assert np.array_equal(genes_h[:, s * n:(s + 1) * n], want)
        _, f32_o, _, _ = oracle.features(ref, want, 32, n=n)
        assert np.array_equal(feat.cpu().numpy()[:, s * n:(s + 1) * n].view(np.uint32), f32_o[:, :n].view(np.uint32))
    assert np.array_equal(one.cpu().numpy().view(np.uint16),
                          oracle.enumerate_candidates(refs[1], oracle.MODE_SAMPLE, n, seed=5))


@pytest.mark.parametrize("p_mut", [synth.P_MUT_Q32, 0])
def test_crossover(G, p_mut):
    mine, ref = _spaces("c3", eck.SPACE_SPLIT)
    parents = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, 100, seed=7)
    n = (1 << 16) + 11
    for rnd, first in [(1, 0), (5, 123457)]:
        got = G.enumerate_gpu(mine, eck.MODE_CROSSOVER, n, seed=9, rnd=rnd, first_index=first, parents=parents,
                              p_mut_q32=p_mut)
        want = oracle.enumerate_candidates(ref, oracle.MODE_CROSSOVER, n, seed=9, rnd=rnd, first_index=first,
                                           parents=parents, p_mut_q32=p_mut)
        assert np.array_equal(got[:, :n], want)


def test_crossover_batched_over_spaces(G):
    import torch
    problems = [synth.gemm(*s) for s in synth.sweep_shapes()[::21]]
    mine = [eck.Space(pb, eck.SPACE_SPLIT) for pb in problems]
    refs = [oracle.Space(pb, oracle.SPACE_SPLIT) for pb in problems]
    S, n, P = len(problems), 2049, 17
    parents = np.concatenate([oracle.enumerate_candidates(r, oracle.MODE_SAMPLE, P, seed=3 + s)
                              for s, r in enumerate(refs)], axis=1)
    ld = S * n + (S * n & 1)
    genes = torch.full((mine[0].n_genes, ld), -1, dtype=torch.int16, device="cuda")
    seeds = [40 + s for s in range(S)]
    eck.candidate_enumerate_batch(mine, eck.MODE_CROSSOVER, n, genes, seeds, round=3, parents=G.to_dev(parents),
                                  p_mut_q32=synth.P_MUT_Q32)
    torch.cuda.synchronize()
    got = genes.cpu().numpy().view(np.uint16)
    for s, ref in enumerate(refs):
        want = oracle.enumerate_candidates(ref, oracle.MODE_CROSSOVER, n, seed=seeds[s], rnd=3,
                                           parents=parents[:, s * P:(s + 1) * P], p_mut_q32=synth.P_MUT_Q32)
        assert np.array_equal(got[:, s * n:(s + 1) * n], want), "space %d" % s


def test_dedup_marks_first_occurrences(G):
    import torch
    mine, ref = _spaces("c3", eck.SPACE_SPLIT)
    parents = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, 8, seed=7)
    n = 20000 + 1   # children of 8 parents with a low mutation rate: mostly repeats
    kids = oracle.enumerate_candidates(ref, oracle.MODE_MUTATE, n, seed=1, rnd=1, parents=parents, p_mut_q32=1 << 28)
    want = oracle.dedup(kids)
    assert 0.02 < want.mean() < 0.9
    genes = G.to_dev(np.concatenate([kids, kids[:, :1]], axis=1))      # ld = n + 1
    flags = torch.full((n + 1,), 9, dtype=torch.uint8, device="cuda")
    eck.candidates_dedup(genes, n, flags, overwrite=True)
    torch.cuda.synchronize()
    got = flags.cpu().numpy()
    assert np.array_equal(got[:n], want) and got[n] == 9
    # AND-ed into existing flags (e.g. legality)
    legal = (np.arange(n) % 3 != 0).astype(np.uint8)
    flags = torch.from_numpy(legal).cuda()
    eck.candidates_dedup(genes, n, flags)
    torch.cuda.synchronize()
    assert np.array_equal(flags.cpu().numpy(), legal & want)
    # all distinct and all equal
    distinct = np.arange(5000, dtype=np.uint16)[None, :].repeat(2, axis=0)
    flags = torch.zeros(5000, dtype=torch.uint8, device="cuda")
    eck.candidates_dedup(G.to_dev(distinct), 5000, flags, overwrite=True)
    same = np.zeros((6, 4096), dtype=np.uint16)
    flags2 = torch.ones(4096, dtype=torch.uint8, device="cuda")
    eck.candidates_dedup(G.to_dev(same), 4096, flags2, overwrite=True)
    torch.cuda.synchronize()
    assert flags.cpu().numpy().all() and list(flags2.cpu().numpy()[:3]) == [1, 0, 0] and flags2.sum().item() == 1


def test_paper_operator_shapes(G):
    """The eleven operators of the paper's evaluation (Sec. 7.2: MM1-4, MV1-4, CONV1-3): sampled schedules,
    all 64 features, both output types, bit for bit."""
    for i, (name, pb) in enumerate(synth.paper_operators().items()):
        mine, ref = _spaces(pb, eck.SPACE_SPLIT)
        n = 3001
        got = G.enumerate_gpu(mine, eck.MODE_SAMPLE, n, seed=300 + i)
        want = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, n, seed=300 + i)
        assert np.array_equal(got[:, :n], want), name
        _check_features(G, mine, ref, want, 64)


def test_features_random_problems(G):
    """Seeded random operators across the library's accepted range (both space kinds, all three operator
    classes, both element sizes, odd extents, strides and paddings): whatever the oracle accepts the library
    must accept, and every raw feature, transformed feature and legality flag must agree."""
    rng = np.random.default_rng(2024)
    dims = [1, 2, 3, 7, 12, 30, 64, 100, 255, 256, 500, 1024, 2047, 4096]
    checked = 0
    for trial in range(60):
        kind_op = rng.integers(0, 4)
        eb = int(rng.choice([2, 4]))
        hw = synth.HW_MI355X if trial % 3 else synth.HW_CASE_STUDY
        if kind_op == 0:
            pb, kind = synth.gemm(*(int(rng.choice(dims)) for _ in range(3)), elem_bytes=eb, hw=hw), eck.SPACE_KNOB
        elif kind_op == 1:
            pb, kind = synth.gemm(*(int(rng.choice(dims)) for _ in range(3)), elem_bytes=eb, hw=hw), eck.SPACE_SPLIT
        elif kind_op == 2:
            pb = synth.bgemm(int(rng.choice([2, 3, 8, 32])), *(int(rng.choice(dims[:12])) for _ in range(3)),
                             elem_bytes=eb, hw=hw)
            kind = eck.SPACE_SPLIT if trial % 2 else eck.SPACE_KNOB
        else:
            r, s_ = int(rng.choice([1, 3, 5])), int(rng.choice([1, 3]))
            pb = synth.conv2d(int(rng.choice([1, 2, 8])), int(rng.choice([3, 16, 64, 96])), int(rng.choice([8, 32, 100])),
                              int(rng.choice([7, 14, 28, 57])), int(rng.choice([7, 14, 30])), r, s_,
                              int(rng.choice([1, 2])), int(rng.choice([0, 1, 2])), elem_bytes=eb, hw=hw)
            kind = eck.SPACE_SPLIT
        try:
            ref = oracle.Space(pb, kind)
        except Exception:
            continue                                   # outside the accepted range on the oracle's side too
        try:
            mine = eck.Space(pb, kind)
        except eck.EckError:
            continue                                   # the library's range limits are tighter in places
        assert mine.radix == ref.radix
        n = int(min(ref.size, 1500)) if ref.size else 1500
        mode = oracle.MODE_EXHAUSTIVE if ref.size and ref.size <= 1500 else oracle.MODE_SAMPLE
        genes = oracle.enumerate_candidates(ref, mode, n, seed=trial)
        _check_features(G, mine, ref, genes, 64)
        checked += 1
    assert checked >= 40


def test_reduction_parallel_hand_worked_schedule(G, golden):
    rows = golden("hand_mv_xred.txt")
    pb = synth.gemm(1, 8, 32, elem_bytes=2, hw=(4, 64, 1024, 256, 8))
    mine, ref = _spaces(pb, eck.SPACE_SPLIT_XRED)
    tabs = [[tuple(int(v) for v in t) for t in oracle.split_table(e)] for e in (1, 8, 32)]
    g = [tabs[0].index((1, 1, 1, 1)), tabs[1].index((2, 2, 1, 2)), tabs[2].index((2, 4, 2, 2)), 1, 1]
    genes = np.array([g, g], dtype=np.uint16).T.copy()
    raw, _, legal = G.features_gpu(mine, genes, 2, 64, eck.F32)
    assert [int(v) for v in raw[:, 0]] == [int(t) for t in rows[0]] and legal[0] == int(rows[1][0])


def test_reduction_parallel_features_of_the_paper_operators(G):
    """Space kind SPLIT_XRED (the reduction split across threads) on the eleven operators of Sec. 7.2, the
    matrix-vector products it is meant for among them: every feature and flag bit for bit."""
    share = {}
    for i, (name, pb) in enumerate(synth.paper_operators().items()):
        mine, ref = _spaces(pb, eck.SPACE_SPLIT_XRED)
        assert mine.radix == ref.radix
        n = 4097
        got = G.enumerate_gpu(mine, eck.MODE_SAMPLE, n, seed=500 + i)
        want = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, n, seed=500 + i)
        assert np.array_equal(got[:, :n], want), name
        _, legal = _check_features(G, mine, ref, want, 64)
        _check_features(G, mine, ref, want[:, :1001], 32)
        share[name] = legal.mean()
    assert all(share[k] > 0.02 for k in ("MV1", "MV2", "MV3", "MV4")), share


def test_reduction_parallel_features_random_problems(G):
    rng = np.random.default_rng(77)
    dims = [1, 2, 3, 7, 12, 30, 64, 100, 255, 256, 500, 1024, 2047, 4096, 12288, 49512]
    checked = 0
    for trial in range(50):
        eb = int(rng.choice([2, 4]))
        hw = synth.HW_MI355X if trial % 3 else synth.HW_CASE_STUDY
        which = trial % 3
        if which == 0:
            pb = synth.gemm(*(int(rng.choice(dims)) for _ in range(3)), elem_bytes=eb, hw=hw)
        elif which == 1:
            pb = synth.bgemm(int(rng.choice([2, 3, 8, 32])), *(int(rng.choice(dims[:13])) for _ in range(3)),
                             elem_bytes=eb, hw=hw)
        else:
            pb = synth.conv2d(int(rng.choice([1, 2, 8])), int(rng.choice([3, 16, 64, 96, 512])),
                              int(rng.choice([8, 32, 100])), int(rng.choice([7, 14, 28, 57])),
                              int(rng.choice([7, 14, 30])), int(rng.choice([1, 3, 5])), int(rng.choice([1, 3])),
                              int(rng.choice([1, 2])), int(rng.choice([0, 1, 2])), elem_bytes=eb, hw=hw)
        try:
            ref = oracle.Space(pb, oracle.SPACE_SPLIT_XRED)
        except Exception:
            continue
        try:
            mine = eck.Space(pb, eck.SPACE_SPLIT_XRED)
        except eck.EckError:
            continue
        n = int(min(ref.size, 1500)) if ref.size else 1500
        mode = oracle.MODE_EXHAUSTIVE if ref.size and ref.size <= 1500 else oracle.MODE_SAMPLE
        genes = oracle.enumerate_candidates(ref, mode, n, seed=trial)
        _check_features(G, mine, ref, genes, 64)
        checked += 1
    assert checked >= 30


def test_reduction_parallel_spaces_batched(G):
    """A batch of SPLIT_XRED spaces through the batched calls; kinds cannot be mixed in one batch."""
    import torch
    problems = [synth.gemm(1, n_, k) for n_, k in ((4096, 1024), (8192, 2048), (1024, 4096))]
    mine = [eck.Space(pb, eck.SPACE_SPLIT_XRED) for pb in problems]
    refs = [oracle.Space(pb, oracle.SPACE_SPLIT_XRED) for pb in problems]
    n = 2050
    seeds = [31, 32, 33]
    genes = torch.zeros((mine[0].n_genes, 3 * n), dtype=torch.int16, device="cuda")
    eck.candidate_enumerate_batch(mine, eck.MODE_SAMPLE, n, genes, seeds)
    feat = torch.zeros((64, 3 * n), dtype=torch.float32, device="cuda")
    legal = torch.zeros(3 * n, dtype=torch.uint8, device="cuda")
    eck.features_compute_batch(mine, genes, n, 64, eck.F32, feat, None, legal)
    torch.cuda.synchronize()
    g_h = genes.cpu().numpy().view(np.uint16)
    for s in range(3):
        want = oracle.enumerate_candidates(refs[s], oracle.MODE_SAMPLE, n, seed=seeds[s])
        assert np.array_equal(g_h[:, s * n:(s + 1) * n], want)
        _, f32_o, _, legal_o = oracle.features(refs[s], want, 64)
        assert np.array_equal(feat[:, s * n:(s + 1) * n].cpu().numpy().view(np.uint32), f32_o.view(np.uint32))
        assert np.array_equal(legal[s * n:(s + 1) * n].cpu().numpy(), legal_o)
    mixed = [mine[0], eck.Space(problems[1], eck.SPACE_SPLIT)]
    with pytest.raises(eck.EckError):
        eck.features_compute_batch(mixed, genes, n, 64, eck.F32, feat, None, legal)


@pytest.mark.parametrize("n,ld,kinds", [(1, 1, 1), (2, 5, 1), (257, 300, 1), (4099, 4099, 3), (70001, 70008, 900), (1 << 18, 1 << 18, 1 << 17)])
def test_dedup_clears_flags_of_many_and_few_occurrences(G, n, ld, kinds):
    """Many candidates of few tuples, lower indices arriving late, tuples that differ in the last gene only; flags that
    were any non-zero value come out as one."""
    import torch
    rng = np.random.default_rng(n)
    genes = np.zeros((5, ld), dtype=np.uint16)
    genes[1] = 7
    which = rng.integers(0, kinds, ld)
    genes[3], genes[4] = which >> 8, which & 255
    want = oracle.dedup(np.ascontiguousarray(genes[:, :n]))
    dev = G.to_dev(genes)
    for overwrite in (True, False):
        before = rng.choice(np.array([0, 1, 2, 255], dtype=np.uint8), n)
        flags = G.to_dev(before)
        eck.candidates_dedup(dev, n, flags, overwrite=overwrite)
        torch.cuda.synchronize()
        expected = want if overwrite else (want != 0) & (before != 0)
        assert np.array_equal(flags.cpu().numpy(), np.asarray(expected, dtype=np.uint8))


@pytest.mark.parametrize("n,kinds,n_genes", [(16384, 1, 3), (40001, 1, 3)] + [  # (one tuple: other sizes say nothing more)
    (n, *form) for n in (16383, 16384, 16385, 40001, 524288, 524289, (1 << 20) - 1, 1 << 20, (1 << 20) + 1)
    for form in ((1500, 8), (1500, 9), (200000, 1), (1 << 30, 5))])
def test_dedup_by_parts_and_by_one_table(G, n, kinds, n_genes):
    """Candidates sorted by hash with a table per part (16384 to 2^20 candidates of up to eight genes, in the workspace of the
    query) and one table for all: few tuples of many occurrences, whose part is far larger than the others, and nearly all
    distinct; genes over all sixteen bits; rows longer than n; a workspace of the table's size only, and one that starts 4
    bytes into a 16-byte line."""
    import torch
    rng = np.random.default_rng(n + kinds)
    ld = n + 3
    base = rng.integers(0, 65536, size=(n_genes, min(kinds, n)), dtype=np.uint16)
    genes = np.ascontiguousarray(base[:, rng.integers(0, base.shape[1], size=ld)])
    # (the oracle compares every pair; numpy's first occurrences, which the oracle is pinned by, for more than a few thousand)
    want = np.zeros(n, dtype=np.uint8)
    want[np.unique(np.ascontiguousarray(genes[:, :n].T).view("V%d" % (2 * n_genes)).ravel(), return_index=True)[1]] = 1
    assert np.array_equal(oracle.dedup(np.ascontiguousarray(genes[:, :3000])), want[:3000])
    dev = G.to_dev(genes)
    table = 4
    while table < 8 * n:
        table *= 2
    full = eck.candidates_dedup_workspace_bytes(n)
    ws = torch.full((max(full, table) + 32,), 255, dtype=torch.uint8, device="cuda")
    for room in (ws[:full], ws[:table], ws[4:4 + full]):
        for overwrite in (True, False):
            flags = G.to_dev((rng.random(n) < 0.7).astype(np.uint8) * 2)
            before = flags.cpu().numpy()
            eck.candidates_dedup(dev, n, flags, overwrite=overwrite, ws=room)
            torch.cuda.synchronize()
            got = flags.cpu().numpy()
            assert np.array_equal(got, want if overwrite else (want & (before != 0)).astype(np.uint8))


def genes_hash(genes):
    """What candidates are sorted by: a SplitMix64 chain over the genes."""
    gamma, h = np.uint64(0x9E3779B97F4A7C15), np.zeros(genes.shape[1], dtype=np.uint64)
    for row in genes:
        z = h + gamma + row.astype(np.uint64)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        h = z ^ (z >> np.uint64(31))
    return h


@pytest.mark.parametrize("n,n_genes,distinct", [(20000, 8, 6000), (20000, 8, 8192), (20000, 8, 8193), (40001, 3, 9000), (600001, 3, 20000)])
def test_dedup_of_genes_chosen_against_the_parts(G, n, n_genes, distinct):
    """Parts of more tuples than a block's table in LDS has slots (8192), or nearly as many: half of the candidates' tuples hash into
    one part, a third into another, the rest anywhere."""
    import torch
    rng = np.random.default_rng(n + distinct)
    shift = np.uint64(64 - (8 if n <= 1 << 19 else 9))
    pools = [[], []]
    while any(sum(g.shape[1] for g in p) < distinct for p in pools):
        draw = rng.integers(0, 65536, size=(n_genes, 1 << 19), dtype=np.uint16)
        part = genes_hash(draw) >> shift
        for p, which in zip(pools, (3, 200)):
            p.append(draw[:, part == which])
    pools = [np.concatenate(p, axis=1)[:, :distinct] for p in pools]
    one, two = n // 2, n // 3
    pick = lambda count: np.concatenate([np.arange(min(count, distinct)), rng.integers(0, distinct, size=max(0, count - distinct))])
    genes = np.concatenate([pools[0][:, pick(one)], pools[1][:, pick(two)],
                            rng.integers(0, 65536, size=(n_genes, n - one - two), dtype=np.uint16)], axis=1)
    genes = np.ascontiguousarray(genes[:, rng.permutation(n)])
    want = np.zeros(n, dtype=np.uint8)
    want[np.unique(np.ascontiguousarray(genes.T).view("V%d" % (2 * n_genes)).ravel(), return_index=True)[1]] = 1
    ws = torch.full((eck.candidates_dedup_workspace_bytes(n) + 256,), 255, dtype=torch.uint8, device="cuda")
    flags = torch.zeros(n, dtype=torch.uint8, device="cuda")
    eck.candidates_dedup(G.to_dev(genes), n, flags, overwrite=True, ws=ws[:-256])
    torch.cuda.synchronize()
    assert np.array_equal(flags.cpu().numpy(), want)
    assert bool((ws[-256:] == 255).all())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_features_streamed_and_through_the_caches(G, dtype):
    """Rows that start on 64 bytes are stored past the caches (of fp32 as long as the matrix is small), others through them:
    the same values, nothing beside the columns asked for, and the oracle's at both ends."""
    import torch
    mine, ref = _spaces("c2", eck.SPACE_SPLIT)
    code, kind = (eck.F32, torch.float32) if dtype == "f32" else (eck.BF16, torch.bfloat16)
    n = 268800  # fp32: past the line; rows of either type a multiple of 64 bytes; with the parts, every size of block
    genes = torch.zeros((mine.n_genes, n), dtype=torch.int16, device="cuda")
    eck.candidate_enumerate(mine, eck.MODE_SAMPLE, n, genes, seed=7)
    whole = torch.full((64, n), -1.0, dtype=kind, device="cuda")
    eck.features_compute(mine, genes, n, 64, code, feat_out=whole)
    for col0, part in ((0, 1000), (0, 190001), (0, 201600), (2, n - 2), (33, 4097)):
        got = torch.full((64, n), -1.0, dtype=kind, device="cuda")
        eck.features_compute(mine, genes, part, 64, code, feat_out=got, col0=col0)
        assert torch.equal(got[:, col0:col0 + part], whole[:, col0:col0 + part])
        assert bool((got[:, :col0] == -1.0).all()) and bool((got[:, col0 + part:] == -1.0).all())
    for at in (0, n - 1500):
        _, want, bits, _ = oracle.features(ref, np.ascontiguousarray(genes[:, at:at + 1500].cpu().numpy().view(np.uint16)), 64)
        mine_bits = whole[:, at:at + 1500].contiguous().cpu()
        if dtype == "f32":
            assert np.array_equal(mine_bits.numpy(), want)
        else:
            assert np.array_equal(mine_bits.view(torch.int16).numpy().view(np.uint16), bits)


@pytest.mark.parametrize("n_feat", [32, 64])
@pytest.mark.parametrize("n", [140000, 262144, 524288, 1 << 20])
def test_features_beside_raw_ones(G, n, n_feat):
    """Sizes at which transformed and raw features, together or alone, are stored by different blocks and by the caches or past
    them: the same values in every form, and the oracle's at both ends."""
    import torch
    mine, ref = _spaces("c2", eck.SPACE_SPLIT)
    genes = torch.zeros((mine.n_genes, n), dtype=torch.int16, device="cuda")
    eck.candidate_enumerate(mine, eck.MODE_SAMPLE, n, genes, seed=7)
    raw_alone = torch.zeros((n_feat, n), dtype=torch.int64, device="cuda")
    eck.features_compute(mine, genes, n, n_feat, eck.F32, raw_out=raw_alone)
    for code, kind in ((eck.F32, torch.float32), (eck.BF16, torch.bfloat16)):
        alone, beside = (torch.full((n_feat, n), -1.0, dtype=kind, device="cuda") for _ in range(2))
        raw = torch.zeros_like(raw_alone)
        eck.features_compute(mine, genes, n, n_feat, code, feat_out=alone)
        eck.features_compute(mine, genes, n, n_feat, code, feat_out=beside, raw_out=raw)
        assert torch.equal(alone, beside) and torch.equal(raw, raw_alone)
        for at in (0, n - 1500):
            want_raw, want, bits, _ = oracle.features(ref, np.ascontiguousarray(genes[:, at:at + 1500].cpu().numpy().view(np.uint16)), n_feat)
            assert np.array_equal(raw[:, at:at + 1500].cpu().numpy().view(np.uint64), want_raw)
            got = alone[:, at:at + 1500].contiguous().cpu()
            if code == eck.F32:
                assert np.array_equal(got.numpy(), want)
            else:
                assert np.array_equal(got.view(torch.int16).numpy().view(np.uint16), bits)
