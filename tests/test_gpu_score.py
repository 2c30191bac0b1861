"""GPU parity: costmodel_score against the fp64 oracle.

Tolerance: |g - o| <= rtol * M per candidate, rtol = 1e-5 for fp32 models and 1e-2 for bf16 models, where
M = |b3| + sum_j |w3_j| h2_j is the magnitude of the output sum (from the oracle).  The output of these
networks is a small difference of large terms (|o| is often 10-60x below M, and for some weight seeds its
mean over the space is ~0), so relating the error to |o| or to rms(o) would measure the cancellation, not the
arithmetic; M is what a relative error of a floating-point sum refers to.  A second, tighter check compares with
the oracle mode that rounds the first hidden layer to bf16 exactly where the kernel does: 1e-4 * M
(what remains is fp32 accumulation order and rare rounding flips of single activations; measured < 1e-6 * M)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2411_18873_amd import eck, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _features(cfg, n, n_feat, seed=3):
    pb = synth.CONFIGS[cfg]["problem"] if isinstance(cfg, str) else cfg
    is_c1 = isinstance(cfg, str) and cfg == "c1"
    kind = oracle.SPACE_KNOB if is_c1 else oracle.SPACE_SPLIT
    ref = oracle.Space(pb, kind)
    mode = oracle.MODE_EXHAUSTIVE if is_c1 else oracle.MODE_SAMPLE
    genes = oracle.enumerate_candidates(ref, mode, n, seed=seed)
    _, f32, b16, _ = oracle.features(ref, genes, n_feat)
    return f32, b16


def test_fp32_model_c1(G):
    widths = synth.CONFIGS["c1"]["widths"]
    f32, _ = _features("c1", 6400, 32)
    for seed in synth.CONFIGS["c1"]["weight_seeds"]:
        theta = synth.mlp_theta(widths, seed, bias_scale=0.3 * (seed == 2))
        model = G.make_model(widths, eck.F32, theta)
        got = G.score_gpu(model, G.to_dev(f32), 6400)
        want = oracle.score(widths, theta, f32)
        assert G.within(got, want, oracle.score_magnitude(widths, theta, f32), 1e-5) <= 1.0
        assert np.isfinite(got).all()


def test_fp32_model_wide_and_ragged(G):
    widths = [64, 256, 256, 1]
    f32, _ = _features("c2", 2000, 64)
    theta = synth.mlp_theta(widths, 5, bias_scale=0.5)
    model = G.make_model(widths, eck.F32, theta)
    n = 1987  # ld = 2000 > n, last block partly empty
    got = G.score_gpu(model, G.to_dev(f32), n)
    want = oracle.score(widths, theta, f32, n=n)
    assert G.within(got, want, oracle.score_magnitude(widths, theta, f32, n=n), 1e-5) <= 1.0


@pytest.mark.parametrize("widths", [[32, 50, 30, 1], [32, 52, 36, 1], [64, 7, 1, 1], [64, 512, 4, 1]])
def test_fp32_model_widths_with_and_without_four_units_per_thread(G, widths):
    """hidden widths that are and are not multiples of four, and one unit: whole and partial tiles in either layer"""
    n = 1000 + 37
    f32, _ = _features("c1" if widths[0] == 32 else "c2", n + 1, widths[0])
    theta = synth.mlp_theta(widths, 6, bias_scale=0.4)
    model = G.make_model(widths, eck.F32, theta)
    got = G.score_gpu(model, G.to_dev(f32), n)
    want = oracle.score(widths, theta, f32, n=n)
    assert np.isfinite(got).all()
    assert G.within(got, want, oracle.score_magnitude(widths, theta, f32, n=n), 1e-5) <= 1.0


@pytest.mark.parametrize("widths", [[32, 1, 1, 1], [64, 17, 48, 1], [32, 33, 5, 1], [64, 304, 80, 1], [64, 500, 497, 1]])
def test_fp32_model_tile_edges(G, widths):
    """hidden widths that leave 1-4 tiles of 16 units to a wavefront, remainders in both layers and in the reduction;
    candidate counts around a tile and around each change of the block's size.  A candidate's score is the same bits
    whatever its place and n; the least legal key of a segment is numpy's, also where a tile straddles segments."""
    counts = [1, 15, 16, 17, 63, 65, 1000]
    if max(widths[1:]) <= 64:
        counts += [512 * 16 - 3, 512 * 16 * 4 + 1, 512 * 16 * 8 + 16, 512 * 16 * 16 + 5]
    most = counts[-1]
    f32, _ = _features("c1" if widths[0] == 32 else "c2", 6400 if widths[0] == 32 else most + (most & 1), widths[0])
    f32 = np.ascontiguousarray(np.tile(f32, (1, -(-most // f32.shape[1]) + 1))[:, :most + (most & 1)])
    theta = synth.mlp_theta(widths, 7, bias_scale=0.4)
    model = G.make_model(widths, eck.F32, theta)
    dev = G.to_dev(f32)
    full = G.score_gpu(model, dev, most)
    want = oracle.score(widths, theta, f32, n=most)
    assert G.within(full, want, oracle.score_magnitude(widths, theta, f32, n=most), 1e-5) <= 1.0
    for n in counts[:-1]:
        assert np.array_equal(G.score_gpu(model, dev, n), full[:n]), n
    rng = np.random.default_rng(3)
    for n, segments in ((1000, 1), (1000, 8), (999, 37), (most, 1)):
        legal = (rng.random(n) < 0.2).astype(np.uint8)
        score = torch.zeros(n, dtype=torch.float32, device="cuda")
        key = torch.zeros(segments, dtype=torch.int32, device="cuda")
        eck.costmodel_score_min(model, dev, n, score, G.to_dev(legal), segments, key)
        torch.cuda.synchronize()
        assert np.array_equal(score.cpu().numpy(), full[:n])
        for s in range(segments):
            of = slice(s * (n // segments), (s + 1) * (n // segments))
            least = full[:n][of][legal[of] != 0]
            got = int(key[s].item()) & 0xFFFFFFFF
            if least.size == 0:
                assert got == 0xFFFFFFFF
            else:
                bits = int(np.float32(least.min()).view(np.uint32))
                assert got == bits ^ (0xFFFFFFFF if bits >> 31 else 0x80000000)


@pytest.mark.parametrize("widths,cfg,n", [([64, 256, 256, 1], "c2", 5000), ([64, 512, 512, 1], None, 4133),
                                          ([64, 128, 128, 1], "c3", 1500), ([32, 64, 64, 1], "c1", 6400)])
def test_bf16_model(G, widths, cfg, n):
    if cfg is None:
        cfg = synth.gemm(4096, 8192, 1024)
    f32, b16 = _features(cfg, n + (n & 1), widths[0])
    theta = synth.mlp_theta(widths, 8, bf16=True, bias_scale=0.5)
    model = G.make_model(widths, eck.BF16, theta)
    feat_as_f32 = oracle.bf16_bits_to_f32(b16)
    want = oracle.score(widths, theta, feat_as_f32, n=n)
    got = G.score_gpu(model, G.bf16_dev(b16), n)
    assert np.isfinite(got).all()
    mag = oracle.score_magnitude(widths, theta, feat_as_f32, n=n)
    worst = G.within(got, want, mag, 1e-2)
    assert worst <= 1.0, worst
    # rounding the first hidden layer to bf16 is the only modelled difference: with it emulated the gap shrinks
    emu = oracle.score(widths, theta, feat_as_f32, n=n, emulate_bf16=True)
    worst_emu = G.within(got, emu, mag, 1e-4)
    assert worst_emu <= 1.0, worst_emu
    print("bf16 score parity %s: worst/1e-2 = %.3f, vs bf16-activation oracle worst/1e-4 = %.4f" % (widths, worst, worst_emu))
    # fp32 features are rounded to bf16 on load: same result as feeding the bf16 features
    got32 = G.score_gpu(model, G.to_dev(f32), n)
    assert np.array_equal(got32, got)


def test_bf16_model_determinism_and_tail_tiles(G):
    widths = [64, 256, 256, 1]
    f32, b16 = _features("c2", 1 << 15, 64)
    theta = synth.mlp_theta(widths, 3, bf16=True)
    model = G.make_model(widths, eck.BF16, theta)
    dev = G.bf16_dev(b16)
    full = G.score_gpu(model, dev, 1 << 15)
    again = G.score_gpu(model, dev, 1 << 15)
    assert np.array_equal(full, again)
    for n in (1, 31, 32, 33, 255, 256, 257, 1000):
        part = G.score_gpu(model, dev, n)
        assert np.array_equal(part, full[:n])
    # the output past n is not written
    out = torch.full((300,), 123.0, dtype=torch.float32, device="cuda")
    eck.costmodel_score(model, dev, 257, out)
    torch.cuda.synchronize()
    assert np.all(out.cpu().numpy()[257:] == 123.0)


def test_bf16_model_leading_dimensions_that_do_not_fit_the_wide_loads(G):
    """A lane loads the 2 or 4 neighbouring candidates it owns at once, so ld must be a multiple of that for the
    last group of a row to end inside the row.  ld = n = 1002 (even, not a multiple of 4) must take the
    two-candidate kernel and give the scores of the padded matrix bit for bit; an odd ld, a misaligned pointer
    and a model shape without a kernel are refused on the host."""
    import ctypes as C
    widths = [64, 256, 256, 1]
    n = 1002
    f32, b16 = _features("c2", 1004, 64)
    theta = synth.mlp_theta(widths, 3, bf16=True, bias_scale=0.5)
    model = G.make_model(widths, eck.BF16, theta)
    padded = G.score_gpu(model, G.bf16_dev(b16), n)                       # ld = 1004: four candidates per load
    tight = G.score_gpu(model, G.bf16_dev(b16[:, :n]), n)                 # ld = n = 1002: two per load
    tight32 = G.score_gpu(model, G.to_dev(f32[:, :n]), n)                 # fp32 features, 8-byte loads
    assert np.array_equal(tight, padded) and np.array_equal(tight32, padded)
    L = eck.lib()
    out = torch.zeros(1024, dtype=torch.float32, device="cuda")
    odd = G.bf16_dev(b16[:, :1001])
    odd32 = G.to_dev(f32[:, :1001])
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    po = C.c_void_p(out.data_ptr())
    assert L.costmodel_score(model.h, C.c_void_p(odd.data_ptr()), eck.BF16, 1001, 1001, po, None, 0, stream) == eck.EALIGN
    assert L.costmodel_score(model.h, C.c_void_p(odd.data_ptr()), eck.BF16, 1001, 999, po, None, 0, stream) == eck.EALIGN
    assert L.costmodel_score(model.h, C.c_void_p(odd32.data_ptr()), eck.F32, 1001, 1001, po, None, 0, stream) == eck.EALIGN
    even = G.bf16_dev(b16)
    assert L.costmodel_score(model.h, C.c_void_p(even.data_ptr() + 2), eck.BF16, 1004, 1000, po, None, 0, stream) == eck.EALIGN
    even32 = G.to_dev(f32)
    assert L.costmodel_score(model.h, C.c_void_p(even32.data_ptr() + 4), eck.F32, 1004, 1000, po, None, 0, stream) == eck.EALIGN
    torch.cuda.synchronize()
    assert np.all(out.cpu().numpy() == 0)                                  # a refused call touches nothing
    # a bf16 model is refused at creation when no matrix-core kernel exists for its shape
    h = C.c_void_p()
    w = (C.c_int32 * 4)(64, 384, 384, 1)
    assert L.eck_model_create(3, w, eck.BF16, C.byref(h)) == eck.EUNSUPPORTED and h.value is None
    assert L.eck_model_create(3, w, eck.F32, C.byref(h)) == eck.OK
    L.eck_model_destroy(h)


def test_bf16_model_rows_wider_than_a_32bit_lane_offset(G):
    """A leading dimension so large that eight feature rows span more than 4 GiB selects the kernel variant
    with 64-bit per-lane addresses; the scores must be those of the compact matrix.  (17 GB of device memory,
    of which only the first columns are written and read.)"""
    widths = [32, 64, 64, 1]
    n = 1500
    _, b16 = _features("c1", n, 32)
    theta = synth.mlp_theta(widths, 4, bf16=True, bias_scale=0.5)
    model = G.make_model(widths, eck.BF16, theta)
    compact = G.score_gpu(model, G.bf16_dev(b16), n)
    ld = (1 << 28) + 2
    wide = torch.empty((32, ld), dtype=torch.bfloat16, device="cuda")
    wide[:, :n] = G.bf16_dev(b16)[:, :n]
    got = G.score_gpu(model, wide, n)
    del wide
    torch.cuda.empty_cache()
    assert np.array_equal(got, compact)


@pytest.mark.parametrize("widths,ld_extra", [([64, 512, 512, 1], 2), ([64, 256, 256, 1], 4)])
def test_bf16_model_wide_rows_over_several_tiles_per_block(G, widths, ld_extra):
    """The same for the 64-feature kernels, with more tiles than blocks and a ragged last one: the features of a
    block's next tile are requested load by load while the current tile computes, through 64-bit per-lane
    addresses here.  (34 GB of device memory, of which only the first columns are written and read.)"""
    n = 256 * 512 + 3 * 256 + 36
    _, b16 = _features("c2", n, 64)
    theta = synth.mlp_theta(widths, 5, bf16=True, bias_scale=0.5)
    model = G.make_model(widths, eck.BF16, theta)
    compact = G.score_gpu(model, G.bf16_dev(b16), n)
    ld = (1 << 28) + ld_extra
    wide = torch.empty((64, ld), dtype=torch.bfloat16, device="cuda")
    wide[:, :n] = G.bf16_dev(b16)[:, :n]
    got = G.score_gpu(model, wide, n)
    del wide
    torch.cuda.empty_cache()
    assert np.array_equal(got, compact)


def test_set_get_state_roundtrip(G):
    widths = [64, 256, 256, 1]
    P = synth.param_count(widths)
    rng = np.random.default_rng(0)
    blob = rng.standard_normal(3 * P + 1).astype(np.float32)
    model = eck.Model(widths, eck.BF16)
    model.set_state(G.to_dev(blob))
    assert np.array_equal(model.get_state().cpu().numpy(), blob)
    model.set_state(G.to_dev(blob[:P]))
    back = model.get_state().cpu().numpy()
    assert np.array_equal(back[:P], blob[:P]) and np.all(back[P:] == 0)


@pytest.mark.parametrize("widths", [[32, 1, 1, 1], [64, 50, 30, 1], [32, 64, 64, 1]])
def test_narrow_fp32_models_on_many_candidates(G, widths):
    """Two candidate tiles per wavefront from 2^18 - 15 candidates on, four below: each candidate has the bits it has in a
    call of few, checked against the oracle."""
    some = 5003
    f32, _ = _features("c1" if widths[0] == 32 else "c2", some + 1, widths[0])
    theta = synth.mlp_theta(widths, 6, bias_scale=0.4)
    model = G.make_model(widths, eck.F32, theta)
    few = G.score_gpu(model, G.to_dev(f32), some)
    assert G.within(few, oracle.score(widths, theta, f32, n=some), oracle.score_magnitude(widths, theta, f32, n=some), 1e-5) <= 1.0
    for n in (262128, 262129, 300001):
        feat = G.to_dev(np.ascontiguousarray(f32[:, np.arange(n + 1) % some]))
        assert np.array_equal(G.score_gpu(model, feat, n), few[np.arange(n) % some]), n


@pytest.mark.parametrize("widths,block,blocks_a_unit", [([64, 256, 256, 1], 64, 1), ([64, 130, 17, 1], 64, 1), ([64, 128, 100, 1], 64, 2),
                                                        ([64, 300, 40, 1], 32, 1), ([32, 16, 512, 1], 64, 1)])
def test_fp32_last_round_of_smaller_blocks(G, widths, block, blocks_a_unit):
    """A launch whose last round of blocks would leave most of the chip idle gives that round's candidates to smaller blocks:
    from no candidate over whole rounds to just past half a round, each has the bits it has in a call of few (checked against
    the oracle), and every segment, blocks of both sizes in it or not, the least of its scores."""
    some = 1009
    f32, _ = _features("c1" if widths[0] == 32 else "c2", some + 1, widths[0])
    theta = synth.mlp_theta(widths, 6, bias_scale=0.4)
    model = G.make_model(widths, eck.F32, theta)
    few = G.score_gpu(model, G.to_dev(f32), some)
    assert G.within(few, oracle.score(widths, theta, f32, n=some), oracle.score_magnitude(widths, theta, f32, n=some), 1e-5) <= 1.0
    units = torch.cuda.get_device_properties(0).multi_processor_count * blocks_a_unit
    left = [0, 1, units // 8 * block, units // 8 * block + 1, units // 4 * block - 17, units // 4 * block + 1, units // 2 * block,
            units // 2 * block + 1]
    for n in [2 * units * block + more for more in left]:
        feat = G.to_dev(np.ascontiguousarray(f32[:, np.arange(n + (n & 1)) % some]))
        want = few[np.arange(n) % some]
        assert np.array_equal(G.score_gpu(model, feat, n), want), n
        segments = max(s for s in range(1, 60) if n % s == 0)
        out, keys = torch.zeros(n, device="cuda"), torch.zeros(segments, dtype=torch.int32, device="cuda")
        eck.costmodel_score_min(model, feat, n, out, None, segments, keys)
        bits = want.reshape(segments, -1).min(axis=1).view(np.uint32)
        order = np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31))
        assert np.array_equal(out.cpu().numpy(), want) and np.array_equal(keys.cpu().numpy().view(np.uint32), order), n


@pytest.mark.parametrize("widths,n", [((32, 64, 64, 1), 777), ((64, 50, 30, 1), 40001), ((64, 128, 128, 1), 9000), ((64, 256, 256, 1), 5000),
                                      ((64, 300, 17, 1), 9000), ((64, 16, 512, 1), 9000), ((32, 512, 512, 1), 1000), ((64, 9, 1, 1), 200000)])
def test_fp32_scores_of_numbers_that_are_not_finite(G, widths, n):
    """A number that is infinite, a NaN or above bfloat16's range has no parts to multiply: its candidate is worked out in plain
    fp32 sums, with the infinities and NaNs those have (a NaN sum leaves the ReLU as zero); every other candidate keeps its
    bits.  Huge finite features, which do have parts, are as close as ordinary ones (weights of one sign where they are, so that no
    cancellation decides between a number and an infinity)."""
    rng = np.random.default_rng(widths[1] + n)
    F, H1, H2, _ = widths
    w1, w2, w3 = (rng.standard_normal(s).astype(np.float32) / np.float32(s[0] ** 0.5) for s in ((F, H1), (H1, H2), (H2, 1)))
    b1, b2, b3 = (rng.standard_normal(s).astype(np.float32) * np.float32(0.1) for s in (H1, H2, 1))
    theta = np.concatenate([t.ravel() for t in (w1, b1, w2, b2, w3, b3)])
    model = G.make_model(widths, eck.F32, theta)
    x = rng.random((F, n + (n & 1))).astype(np.float32)
    clean = G.score_gpu(model, G.to_dev(x), n)
    odd = {0: np.inf, 5: -np.inf, 17: np.nan, n // 2: 3.4e38, n - 1: np.inf, n // 3: 1e30, n // 4: -2.5e37}
    for at, value in odd.items():
        x[rng.integers(F), at] = value
    got = G.score_gpu(model, G.to_dev(x), n)
    same = np.ones(n, dtype=bool)
    same[list(odd)] = False
    assert np.array_equal(got[same].view(np.uint32), clean[same].view(np.uint32))
    with np.errstate(all="ignore"):
        for at in odd:
            h1 = np.fmax((x[:, at].astype(np.float64) @ w1.astype(np.float64) + b1), 0.0)
            h2 = np.fmax(h1 @ w2.astype(np.float64) + b2, 0.0)
            want = float((h2 @ w3.astype(np.float64))[0] + b3[0])
            size = float(h2 @ np.abs(w3[:, 0].astype(np.float64)) + abs(b3[0]))
            if np.isfinite(want):
                assert abs(float(got[at]) - want) <= 1e-5 * size, (at, got[at], want)
            else:
                assert (np.isnan(got[at]) and np.isnan(want)) or got[at] == want, (at, got[at], want)
    # weights that are not finite: every candidate takes the plain sums
    w2[rng.integers(H1), rng.integers(H2)] = np.inf
    bad = G.make_model(widths, eck.F32, np.concatenate([t.ravel() for t in (w1, b1, w2, b2, w3, b3)]))
    few = 300
    got = G.score_gpu(bad, G.to_dev(np.ascontiguousarray(x[:, 20:20 + few])), few)
    with np.errstate(all="ignore"):
        h1 = np.fmax(w1.T @ x[:, 20:20 + few] + b1[:, None], 0)
        terms = np.where(h1[:, None, :] == 0, np.where(np.isinf(w2)[:, :, None], np.nan, 0.0), w2[:, :, None] * h1[:, None, :])
        want = (np.fmax(terms.sum(0) + b2[:, None], 0) * w3).sum(0) + b3[0] if H1 * H2 * few < 3e7 else None
    if want is not None:
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))


@pytest.mark.parametrize("widths,n", [((64, 512, 512, 1), 1 << 14), ((64, 256, 256, 1), 1 << 15), ((32, 64, 64, 1), 1 << 17)])
@pytest.mark.parametrize("where", ["first", "second", "bias", "all"])
def test_fp32_models_that_are_not_finite_take_no_path_of_their_own_per_candidate(G, widths, n, where):
    """A refit that diverged leaves NaNs and infinities in the weights, so that every candidate's sums hold some: they are worked
    out in fp32 matrix instructions, at a sixth of the rate or more, not candidate by candidate (a hundredth and less)."""
    F, H1, H2, _ = widths
    rng = np.random.default_rng(H1)
    theta = synth.mlp_theta(list(widths), 6, bias_scale=0.4)
    bad = theta.copy()
    first, second = F * H1, F * H1 + H1 + H1 * H2
    if where == "first":
        bad[rng.integers(first)] = np.nan
    elif where == "second":
        bad[first + H1 + rng.integers(H1 * H2)] = np.inf
    elif where == "bias":
        bad[first + rng.integers(H1)] = -np.inf
    else:
        bad[:] = np.nan
    x = (rng.random((F, n)) * 8).astype(np.float32)
    feat, out = G.to_dev(x), torch.zeros(n, device="cuda")
    took = []
    for th in (theta, bad):
        model = G.make_model(list(widths), eck.F32, th)
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        eck.costmodel_score(model, feat, n, out)
        start.record()
        for _ in range(8):
            eck.costmodel_score(model, feat, n, out)
        end.record()
        torch.cuda.synchronize()
        took.append(start.elapsed_time(end))
    assert took[1] < 6 * took[0], took
    some = 64
    with np.errstate(all="ignore"):
        w1, b1 = bad[:first].reshape(F, H1).astype(np.float64), bad[first:first + H1]
        w2, b2 = bad[first + H1:second].reshape(H1, H2).astype(np.float64), bad[second:second + H2]
        w3, b3 = bad[second + H2:-1].astype(np.float64), bad[-1]
        h1 = np.fmax((x[:, :some, None] * w1[:, None, :]).sum(0) + b1, 0)
        want = np.stack([np.fmax((h[:, None] * w2).sum(0) + b2, 0) @ w3 + b3 for h in h1])
        size = np.stack([np.fmax((h[:, None] * w2).sum(0) + b2, 0) @ np.abs(w3) + abs(b3) for h in h1])
    got = out[:some].cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    fine = np.isfinite(want)
    assert np.all(np.abs(got[fine] - want[fine]) <= 1e-5 * size[fine])


@pytest.mark.parametrize("widths", [(64, 256, 256, 1), (32, 64, 64, 1), (64, 300, 40, 1), (64, 20, 100, 1)])
@pytest.mark.parametrize("inputs,first,bias,second", [(-122, 100, None, 0), (-124, 90, None, 30), (8, -124, None, 120), (8, 40, None, -122),
                                                      (None, 0, -124, 110), (-62, -62, None, 110), (-39, -49, -99, 90)])
def test_fp32_scores_of_small_numbers(G, widths, inputs, first, bias, second):
    """Numbers below 2^-110 are no sums of three bfloat16 ones.  Features, weights, biases and, from products of small ones,
    activations of such sizes (powers of two; None: zeros), scaled up again behind, are as close as ordinary ones; candidates with
    ordinary features beside small ones keep the bits they have alone."""
    F, H1, H2, _ = widths
    n = 777
    number = np.float32(1 + 0.45 / 512) # (at 2^-124 the parts miss 9e-4 of it, at 2^-122 1e-4)
    sized = lambda shape, power: np.full(shape, 0 if power is None else number * 2.0 ** power, dtype=np.float32)
    x, w1, b1, w2, w3 = sized((F, n), inputs), sized((F, H1), first), sized(H1, bias), sized((H1, H2), second), sized((H2, 1), 0)
    x[2:] = 0
    theta = np.concatenate([t.ravel() for t in (w1, b1, w2, np.zeros(H2, np.float32), w3, np.zeros(1, np.float32))])
    model = G.make_model(list(widths), eck.F32, theta)
    got = G.score_gpu(model, G.to_dev(np.ascontiguousarray(np.pad(x, ((0, 0), (0, 1))))), n)
    d = np.float64
    want = (w3.T.astype(d) @ (w2.T.astype(d) @ (w1.T.astype(d) @ x.astype(d) + b1[:, None].astype(d))))[0]
    # sums of positive terms: a rounding for each addition and each product
    assert np.all(np.abs(got - want) <= (F + H1 + H2 + 4) * 2.0 ** -24 * want), float(np.max(np.abs(got / want - 1)))
    if inputs is not None:
        plain = np.random.default_rng(H1).random((F, n + 1)).astype(np.float32)
        alone = G.score_gpu(model, G.to_dev(plain), n)
        mixed = plain.copy()
        mixed[:, 5::7] = np.pad(x, ((0, 0), (0, 1)))[:, 5::7]
        both = G.score_gpu(model, G.to_dev(mixed), n)
        ordinary = np.ones(n, dtype=bool)
        ordinary[5::7] = False
        assert np.array_equal(both[ordinary], alone[ordinary]) and np.array_equal(both[5::7], got[5::7])


@pytest.mark.parametrize("widths", [(32, 1, 1, 1), (64, 16, 16, 1), (64, 9, 17, 1), (32, 16, 64, 1), (64, 5, 128, 1), (64, 16, 130, 1),
                                    (32, 12, 257, 1), (64, 16, 512, 1)])
def test_fp32_models_of_a_first_layer_of_one_tile(G, widths):
    """First layers of up to sixteen units are worked out in fp32 products, in blocks whose form depends on the candidates, the
    features and the second layer: on both sides of every line each candidate has the bits it has in a call of few, checked
    against the oracle, and every segment the least of its scores."""
    widths = list(widths)
    some = 1009
    f32, _ = _features("c1" if widths[0] == 32 else "c2", some + 1, widths[0])
    theta = synth.mlp_theta(widths, 6, bias_scale=0.4)
    model = G.make_model(widths, eck.F32, theta)
    few = G.score_gpu(model, G.to_dev(f32), some)
    assert G.within(few, oracle.score(widths, theta, f32, n=some), oracle.score_magnitude(widths, theta, f32, n=some), 1e-5) <= 1.0
    for tiles in (1, 4, 256, 512, 1024, 1536, 3072, 5632, 8192):
        for n in (16 * tiles - 15, 16 * tiles, 16 * tiles + 1):
            feat = G.to_dev(np.ascontiguousarray(f32[:, np.arange(n + (n & 1)) % some]))
            want = few[np.arange(n) % some]
            assert np.array_equal(G.score_gpu(model, feat, n), want), n
            segments = max(s for s in range(1, 60) if n % s == 0)
            out, keys = torch.zeros(n, device="cuda"), torch.zeros(segments, dtype=torch.int32, device="cuda")
            eck.costmodel_score_min(model, feat, n, out, None, segments, keys)
            bits = want.reshape(segments, -1).min(axis=1).view(np.uint32)
            order = np.where(bits >> 31, ~bits, bits | np.uint32(1 << 31))
            assert np.array_equal(out.cpu().numpy(), want) and np.array_equal(keys.cpu().numpy().view(np.uint32), order), n
