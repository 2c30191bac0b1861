"""GPU parity: costmodel_update (SNR, Eq.-(1) Adam refit) against the oracle."""
import math

import numpy as np
import pytest
from scipy.stats import spearmanr

import oracle
from paper_2411_18873_amd import eck, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    return gpu_util


def _pairs(n, seed=11):
    cfg = synth.CONFIGS["c4"]
    ref = oracle.Space(cfg["problem"], oracle.SPACE_SPLIT)
    genes = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, n, seed=seed)
    _, f32, b16, _ = oracle.features(ref, genes, 64)
    e = synth.measured_energy(f32, cfg["label_seed"])
    return f32, b16, e


def _oracle_state(theta):
    P = theta.size
    return np.concatenate([theta.astype(np.float64), np.zeros(2 * P + 1)])


def test_fp32_trajectory(G):
    widths = [64, 256, 256, 1]
    P = synth.param_count(widths)
    f32, _, e = _pairs(2048)
    theta = synth.mlp_theta(widths, 3, bias_scale=0.1)
    model = G.make_model(widths, eck.F32, theta)
    st = _oracle_state(theta)
    feat = G.to_dev(f32)
    # one step
    snr_g, loss_g = G.update_gpu(model, feat, e, 1, 512)
    snr_o, loss_o = oracle.update(widths, st, f32, e, 1, 512)
    assert abs(snr_g - snr_o) <= 1e-4 * snr_o and abs(loss_g - loss_o) <= 1e-4 * loss_o
    got = model.get_state().cpu().numpy().astype(np.float64)
    # first Adam step is lr*sign(g): exact wherever the gradient is not vanishing
    d = np.abs(got[:P] - st[:P])
    assert np.mean(d > 1e-5) < 1e-3 and d.max() <= 2.001e-3
    assert np.allclose(got[P:2 * P], st[P:2 * P], rtol=2e-3, atol=1e-7)      # first moment = 0.1 g
    assert got[3 * P] == 1.0
    # 19 more steps, minibatches wrap around the 4 blocks of the buffer
    snr_g, loss_g = G.update_gpu(model, feat, e, 19, 512)
    snr_o, loss_o = oracle.update(widths, st, f32, e, 19, 512)
    assert abs(snr_g - snr_o) <= 2e-3 * snr_o and abs(loss_g - loss_o) <= 2e-3 * loss_o
    got = model.get_state().cpu().numpy().astype(np.float64)
    d = np.abs(got[:P] - st[:P])
    assert np.quantile(d, 0.999) < 2e-4 and got[3 * P] == 20.0
    pred_g = G.score_gpu(model, feat, 2048)
    pred_o = oracle.score(widths, st[:P].astype(np.float32), f32)
    assert G.within(pred_g, pred_o, oracle.score_magnitude(widths, st[:P].astype(np.float32), f32), 1e-3) <= 1.0


@pytest.mark.parametrize("widths,n_pairs,minibatch", [([32, 1, 1, 1], 8, 1), ([64, 17, 48, 1], 45, 15), ([32, 33, 5, 1], 34, 17),
                                                      ([64, 128, 128, 1], 500, 250), ([64, 300, 96, 1], 256, 128),
                                                      ([64, 500, 497, 1], 66, 33), ([64, 4, 512, 1], 1040, 520)])
def test_fp32_steps_at_tile_edges(G, widths, n_pairs, minibatch):
    """hidden widths and minibatches around the tiles of the two-launch step: one to four 16-unit tiles per wavefront,
    remainders in units, reduction and rows.  After one step the moments are 0.1 g and 0.001 g^2, so they compare the
    gradient: a sum of n fp32 products is off by at most n 2^-24 of the sum of their magnitudes, the longest here is
    520, and the norms of sum and magnitudes differ by less than a factor of 30: 1e-3 (measured below 1e-6).  The second
    moment's factor 1 - beta2 is rounded to fp32, 5e-5 off."""
    F = widths[0]
    P = synth.param_count(widths)
    f32, _, _ = _pairs(n_pairs + (n_pairs & 1))
    f32 = np.ascontiguousarray(f32[:F])
    e = synth.measured_energy(f32[:, :n_pairs], 13)
    theta = synth.mlp_theta(widths, 3, bias_scale=0.1)
    model = G.make_model(widths, eck.F32, theta)
    st = _oracle_state(theta)
    feat = G.to_dev(f32)
    snr_g, loss_g = G.update_gpu(model, feat, e, 1, minibatch)
    snr_o, loss_o = oracle.update(widths, st, f32, e, 1, minibatch)
    assert abs(snr_g - snr_o) <= 1e-4 * snr_o and abs(loss_g - loss_o) <= 1e-4 * loss_o
    got = model.get_state().cpu().numpy().astype(np.float64)
    for lo, hi, tol in ((P, 2 * P, 1e-3), (2 * P, 3 * P, 3e-3)):
        off = np.linalg.norm(got[lo:hi] - st[lo:hi]) / np.linalg.norm(st[lo:hi])
        assert off <= tol, off
    assert got[3 * P] == 1.0
    # a parameter moves by lr against its gradient's sign; where the gradient vanishes, rounding decides
    d = np.abs(got[:P] - st[:P])
    clear = np.abs(st[P:2 * P]) > 1e-4 * np.abs(st[P:2 * P]).max()
    assert d[clear].max() <= 1e-5 and d.max() <= 2.001e-3
    # the minibatches after the first: the whole buffer once, the same bits every time
    again = G.make_model(widths, eck.F32, theta)
    steps = n_pairs // minibatch
    G.update_gpu(again, feat, e, steps, minibatch)
    assert np.isfinite(again.get_state().cpu().numpy()).all()
    twice = G.make_model(widths, eck.F32, theta)
    G.update_gpu(twice, feat, e, steps, minibatch)
    assert np.array_equal(twice.get_state().cpu().numpy(), again.get_state().cpu().numpy())


def test_bf16_refit_config4(G):
    cfg = synth.CONFIGS["c4"]
    widths = cfg["widths"]
    P = synth.param_count(widths)
    f32, b16, e = _pairs(cfg["n_pairs"], cfg["pair_seed"])
    theta = synth.mlp_theta(widths, cfg["weight_seeds"][0], bf16=True)
    model = G.make_model(widths, eck.BF16, theta)
    st = _oracle_state(theta)
    feat = G.bf16_dev(b16)
    feat_o = oracle.bf16_bits_to_f32(b16)
    # single step: forward scalars at the bf16 tolerance
    snr_g, loss_g = G.update_gpu(model, feat, e, 1, cfg["minibatch"], lr=cfg["lr"])
    snr_o, loss_o = oracle.update(widths, st, feat_o, e, 1, cfg["minibatch"], lr=cfg["lr"], bf16_weights=True)
    assert abs(snr_g - snr_o) <= 2e-2 * snr_o and abs(loss_g - loss_o) <= 2e-2 * loss_o
    got = model.get_state().cpu().numpy().astype(np.float64)
    d = np.abs(got[:P] - st[:P])
    assert d.max() <= 2.001 * cfg["lr"] and np.mean(d > 0.1 * cfg["lr"]) < 0.02
    # the remaining 99 steps
    snr_g, loss_g = G.update_gpu(model, feat, e, cfg["n_steps"] - 1, cfg["minibatch"], lr=cfg["lr"])
    snr_o, loss_o = oracle.update(widths, st, feat_o, e, cfg["n_steps"] - 1, cfg["minibatch"], lr=cfg["lr"],
                                  bf16_weights=True)
    assert abs(loss_g - loss_o) <= 0.05 * loss_o
    assert abs(snr_g - snr_o) <= 0.05 * snr_o
    # rescoring with the refitted model ranks candidates like the oracle's refitted model
    ref = oracle.Space(cfg["problem"], oracle.SPACE_SPLIT)
    genes = oracle.enumerate_candidates(ref, oracle.MODE_SAMPLE, 1 << 14, seed=2024)
    _, _, b16r, _ = oracle.features(ref, genes, 64)
    pred_g = G.score_gpu(model, G.bf16_dev(b16r), 1 << 14)
    eff = synth.round_to_bf16(st[:P].astype(np.float32))
    pred_o = oracle.score(widths, eff, oracle.bf16_bits_to_f32(b16r))
    assert spearmanr(pred_g, pred_o)[0] >= 0.99
    assert model.get_state().cpu().numpy()[3 * P] == 100.0


def test_bf16_single_steps_from_synchronised_states(G):
    """Weight for weight along config 4's trajectory.  Run freely, the two trajectories drift apart in single weights
    (the early Adam steps are lr * sign(g), so a rounding difference in a vanishing gradient moves a weight by up to
    2 lr) and are compared statistically above.  Here the library restarts from the oracle's state (weights, both
    moments, step count, rounded to the fp32 the library stores) after 1, 10, 50 and 99 steps and both take ONE
    step: once the moments have built up, every one of the 82 689 weights must land within a small fraction of lr
    of the oracle's (measured: 0.017 lr after 10 steps, 3e-4 lr after 50 and 99), and the second moments agree."""
    cfg = synth.CONFIGS["c4"]
    widths = cfg["widths"]
    P = synth.param_count(widths)
    lr = cfg["lr"]
    f32, b16, e = _pairs(cfg["n_pairs"], cfg["pair_seed"])
    theta = synth.mlp_theta(widths, cfg["weight_seeds"][0], bf16=True)
    st = _oracle_state(theta)
    feat = G.bf16_dev(b16)
    feat_o = oracle.bf16_bits_to_f32(b16)
    done = 0
    for upto, max_lr, q999_lr in ((1, 2.001, 0.05), (10, 0.06, 0.005), (50, 2e-3, 1e-3), (99, 2e-3, 1e-3)):
        oracle.update(widths, st, feat_o, e, upto - done, cfg["minibatch"], lr=lr, bf16_weights=True)
        done = upto
        st32 = st.astype(np.float32)
        model = eck.Model(widths, eck.BF16)
        model.set_state(G.to_dev(st32))
        so = st32.astype(np.float64)
        G.update_gpu(model, feat, e, 1, cfg["minibatch"], lr=lr)
        oracle.update(widths, so, feat_o, e, 1, cfg["minibatch"], lr=lr, bf16_weights=True)
        got = model.get_state().cpu().numpy().astype(np.float64)
        d = np.abs(got[:P] - so[:P]) / lr
        assert d.max() <= max_lr and np.quantile(d, 0.999) <= q999_lr, (upto, d.max(), np.quantile(d, 0.999))
        assert got[3 * P] == so[3 * P] == upto + 1
        if upto >= 10:  # second moments: sums of squares, no cancellation
            v_g, v_o = got[2 * P:3 * P], so[2 * P:3 * P]
            assert np.quantile(np.abs(v_g - v_o) / (v_o + 1e-20), 0.999) <= 5e-3


def test_resume_from_checkpoint_is_bit_identical(G):
    widths = [64, 256, 256, 1]
    f32, b16, e = _pairs(1024)
    theta = synth.mlp_theta(widths, 4, bf16=True)
    feat = G.bf16_dev(b16)
    a = G.make_model(widths, eck.BF16, theta)
    G.update_gpu(a, feat, e, 10, 256)
    once = a.get_state().cpu().numpy()
    b = G.make_model(widths, eck.BF16, theta)
    G.update_gpu(b, feat, e, 4, 256)
    blob = b.get_state()
    c = eck.Model(widths, eck.BF16)
    c.set_state(blob)
    G.update_gpu(c, feat, e, 0, 256)  # zero steps: state untouched
    assert np.array_equal(c.get_state().cpu().numpy(), blob.cpu().numpy())
    # minibatch order restarts with each call: 4 + 4 + 2 steps over whole passes of the 4-block buffer
    # equal 10 steps in one call
    d = G.make_model(widths, eck.BF16, theta)
    G.update_gpu(d, feat, e, 4, 256)
    G.update_gpu(d, feat, e, 4, 256)
    G.update_gpu(d, feat, e, 2, 256)
    assert np.array_equal(d.get_state().cpu().numpy(), once)


def test_data_error_leaves_the_model_alone(G):
    widths = [64, 256, 256, 1]
    f32, b16, e = _pairs(512)
    theta = synth.mlp_theta(widths, 4, bf16=True)
    model = G.make_model(widths, eck.BF16, theta)
    before = model.get_state().cpu().numpy()
    bad = e.copy()
    bad[17] = 0.0
    snr, loss = G.update_gpu(model, G.bf16_dev(b16), bad, 3, 256)
    assert math.isnan(snr) and math.isnan(loss)
    assert np.array_equal(model.get_state().cpu().numpy(), before)
    bad[17] = np.nan
    snr, loss = G.update_gpu(model, G.bf16_dev(b16), bad, 3, 256)
    assert math.isnan(snr) and np.array_equal(model.get_state().cpu().numpy(), before)


def test_zero_steps_reports_snr_only(G):
    widths = [32, 64, 64, 1]
    ref = oracle.Space(synth.CONFIGS["c1"]["problem"], oracle.SPACE_KNOB)
    genes = oracle.enumerate_candidates(ref, oracle.MODE_EXHAUSTIVE, 1024)
    _, f32, _, _ = oracle.features(ref, genes, 32)
    e = synth.measured_energy(f32, 5)
    theta = synth.mlp_theta(widths, 1)
    model = G.make_model(widths, eck.F32, theta)
    snr_g, loss_g = G.update_gpu(model, G.to_dev(f32), e, 0, 256)
    st = _oracle_state(theta)
    snr_o, _ = oracle.update(widths, st, f32, e, 0, 256)
    assert abs(snr_g - snr_o) <= 1e-4 * snr_o and math.isnan(loss_g)


@pytest.mark.parametrize("widths,mb", [([64, 512, 512, 1], 512), ([64, 128, 128, 1], 128), ([32, 64, 64, 1], 64),
                                       ([64, 256, 256, 1], 96)])
def test_bf16_refit_every_model_shape_and_both_step_paths(G, widths, mb):
    """BF16 models refit in two launches per step when the minibatch is a multiple of 64 (every shape the library
    builds), else product by product (minibatch 96 here); either way: one step against the oracle at the bf16
    tolerance, a 12-step run that lowers the loss as the oracle's does, fp32 features that hold bf16 values giving
    the bf16-feature result bit for bit, and the same call twice giving the same bits."""
    F = widths[0]
    n = 4 * mb
    if F == 64:
        f32, b16, e = _pairs(n + (n & 1))
    else:
        ref = oracle.Space(synth.CONFIGS["c1"]["problem"], oracle.SPACE_KNOB)
        genes = oracle.enumerate_candidates(ref, oracle.MODE_EXHAUSTIVE, n)
        _, f32, b16, _ = oracle.features(ref, genes, 32)
        e = synth.measured_energy(f32, 5)
    f32, b16, e = f32[:, :n], b16[:, :n], e[:n]
    P = synth.param_count(widths)
    theta = synth.mlp_theta(widths, 6, bf16=True, bias_scale=0.2)
    feat_o = oracle.bf16_bits_to_f32(b16)
    st = _oracle_state(theta)
    model = G.make_model(widths, eck.BF16, theta)
    feat = G.bf16_dev(np.ascontiguousarray(b16))
    snr_g, loss_g = G.update_gpu(model, feat, e, 1, mb)
    snr_o, loss_o = oracle.update(widths, st, feat_o, e, 1, mb, bf16_weights=True)
    assert abs(snr_g - snr_o) <= 2e-2 * snr_o and abs(loss_g - loss_o) <= 2e-2 * loss_o
    got = model.get_state().cpu().numpy().astype(np.float64)
    d = np.abs(got[:P] - st[:P])
    assert d.max() <= 2.001e-3 and np.mean(d > 1e-4) < 0.03      # Adam's first step is lr * sign(g)
    snr_g, loss_g = G.update_gpu(model, feat, e, 12, mb)
    snr_o, loss_o = oracle.update(widths, st, feat_o, e, 12, mb, bf16_weights=True)
    assert abs(loss_g - loss_o) <= 0.05 * loss_o and abs(snr_g - snr_o) <= 0.05 * snr_o
    assert model.get_state().cpu().numpy()[3 * P] == 13.0
    # fp32 features holding the same values; and a repeat
    a = G.make_model(widths, eck.BF16, theta)
    G.update_gpu(a, feat, e, 5, mb)
    b = G.make_model(widths, eck.BF16, theta)
    G.update_gpu(b, G.to_dev(np.ascontiguousarray(feat_o)), e, 5, mb)
    c = G.make_model(widths, eck.BF16, theta)
    G.update_gpu(c, feat, e, 5, mb)
    sa = a.get_state().cpu().numpy()
    assert np.array_equal(sa, b.get_state().cpu().numpy()) and np.array_equal(sa, c.get_state().cpu().numpy())


@pytest.mark.parametrize("widths,mb,ld_extra", [([64, 128, 128, 1], 576, 8), ([32, 64, 64, 1], 1088, 16), ([64, 256, 256, 1], 64, 24)])
def test_bf16_refit_rows_past_a_threads_32(G, widths, mb, ld_extra):
    """The output layer's blocks have up to 32 rows of a thread under way: 36, 68 (a remainder after one and two times 32) and 4
    of them, of features whose rows lie further apart than there are pairs; one step against the oracle at the bf16
    tolerance, and the output layer's and the biases' first moments, which are plain sums: their terms carry bfloat16's
    relative error of 2^-8 from h1 and the deltas, 2e-2 with the few activations that flip."""
    F, P, n = widths[0], synth.param_count(widths), 2 * mb
    _, b16, _ = _pairs(n + ld_extra)
    b16 = np.ascontiguousarray(b16[:F, :n + ld_extra])
    feat_o = oracle.bf16_bits_to_f32(b16)
    e = synth.measured_energy(feat_o[:, :n], 5)
    theta = synth.mlp_theta(widths, 6, bf16=True, bias_scale=0.2)
    st = _oracle_state(theta)
    model = G.make_model(widths, eck.BF16, theta)
    snr_g, loss_g = G.update_gpu(model, G.bf16_dev(b16), e, 1, mb)
    snr_o, loss_o = oracle.update(widths, st, feat_o, e, 1, mb, bf16_weights=True)
    assert abs(snr_g - snr_o) <= 2e-2 * snr_o and abs(loss_g - loss_o) <= 2e-2 * loss_o
    got = model.get_state().cpu().numpy().astype(np.float64)
    H1, H2 = widths[1], widths[2]
    b1, w2, b2, w3 = F * H1, F * H1 + H1, F * H1 + H1 + H1 * H2, F * H1 + H1 + H1 * H2 + H2
    for lo, hi in ((b1, w2), (b2, w3), (w3, P)):
        off = np.linalg.norm(got[P + lo:P + hi] - st[P + lo:P + hi]) / np.linalg.norm(st[P + lo:P + hi])
        assert off <= 2e-2, (lo, hi, off)


@pytest.mark.parametrize("widths,n_pairs,minibatch", [([64, 17, 48, 1], 45, 15), ([32, 33, 5, 1], 34, 17), ([64, 128, 128, 1], 500, 250),
                                                      ([64, 500, 497, 1], 66, 33), ([64, 300, 96, 1], 256, 128)])
def test_fp32_later_minibatches(G, widths, n_pairs, minibatch):
    """Every minibatch of the buffer and the first again, against the oracle: row offsets that are no multiple of a tile,
    padding rows left by the step before, bias corrections of the second step and later.  With lr = 1e-6 a weight whose
    vanishing gradient takes the other sign is 2e-6 off per step, 1e-4 of the weights' size at most, so the moments and
    the last minibatch's loss are bounded as after one step (n 2^-24 of the magnitudes summed, n <= 500: 1e-3, and 5e-5
    more in the second moment, whose factor 1 - beta2 is rounded to fp32)."""
    F, P = widths[0], synth.param_count(widths)
    f32, _, _ = _pairs(n_pairs + (n_pairs & 1))
    f32 = np.ascontiguousarray(f32[:F])
    e = synth.measured_energy(f32[:, :n_pairs], 13)
    theta = synth.mlp_theta(widths, 3, bias_scale=0.1)
    for steps in (2, n_pairs // minibatch + 1):
        model = G.make_model(widths, eck.F32, theta)
        st = _oracle_state(theta)
        snr_g, loss_g = G.update_gpu(model, G.to_dev(f32), e, steps, minibatch, lr=1e-6)
        snr_o, loss_o = oracle.update(widths, st, f32, e, steps, minibatch, lr=1e-6)
        assert abs(snr_g - snr_o) <= 1e-4 * snr_o and abs(loss_g - loss_o) <= 1e-3 * loss_o
        got = model.get_state().cpu().numpy().astype(np.float64)
        for lo, hi, tol in ((P, 2 * P, 1e-3), (2 * P, 3 * P, 3e-3)):
            off = np.linalg.norm(got[lo:hi] - st[lo:hi]) / np.linalg.norm(st[lo:hi])
            assert off <= tol, (steps, off)
        assert got[3 * P] == steps
        # each step moves a weight by lr times a ratio of corrected moments, equal on both sides where the gradient is clear
        clear = np.abs(st[P:2 * P]) > 1e-3 * np.abs(st[P:2 * P]).max()
        moved_g, moved_o = got[:P] - theta, st[:P] - theta
        assert np.abs(moved_g - moved_o)[clear].max() <= 1e-6 * 0.05 * steps + 2.0 ** -24 * steps * np.abs(theta).max()


@pytest.mark.parametrize("widths,minibatch", [([64, 17, 48, 1], 15), ([64, 256, 256, 1], 64)])
def test_data_error_leaves_an_fp32_model_alone(G, widths, minibatch):
    n = 4 * minibatch
    f32, _, e = _pairs(n + (n & 1))
    e = e[:n].copy()
    model = G.make_model(widths, eck.F32, synth.mlp_theta(widths, 4, bias_scale=0.1))
    feat = G.to_dev(f32)
    G.update_gpu(model, feat, e, 5, minibatch)                       # moments and a step count to leave alone
    before = model.get_state().cpu().numpy()
    for value in (0.0, -1.0, np.nan, np.inf):
        bad = e.copy()
        bad[n - 1] = value
        snr, loss = G.update_gpu(model, feat, bad, 3, minibatch)
        assert math.isnan(snr) and math.isnan(loss)
        assert np.array_equal(model.get_state().cpu().numpy().view(np.uint32), before.view(np.uint32))


@pytest.mark.parametrize("widths,mb,n_pairs,feat", [
    ([64, 256, 256, 1], 64, 64, "bf16"), ([64, 256, 256, 1], 1024, 1024, "f32"), ([64, 256, 256, 1], 192, 576, "bf16"),
    ([64, 128, 128, 1], 2048, 2048, "bf16"), ([64, 128, 128, 1], 448, 896, "f32"), ([32, 64, 64, 1], 320, 640, "bf16"),
    ([64, 256, 256, 1], 250, 500, "bf16"), ([64, 128, 128, 1], 333, 666, "f32"), ([32, 64, 64, 1], 201, 402, "bf16"),
    ([32, 64, 64, 1], 2048, 2048, "f32")])
def test_bf16_steps_of_a_crew_are_those_of_two_launches(G, widths, mb, n_pairs, feat):
    """Calls of a few steps launch each step by itself, longer ones of up to 1024 rows run all steps in one launch on one die: the same
    bits, and with minibatches that come round again.  (Several blocks of rows a member: small crews, below.)"""
    f32, b16, e = _pairs(n_pairs)
    F, epoch = widths[0], n_pairs // mb
    x = G.bf16_dev(b16[:F].copy()) if feat == "bf16" else G.to_dev(np.ascontiguousarray(f32[:F]))
    theta = synth.mlp_theta(widths, 4, bf16=True)
    a, b = G.make_model(widths, eck.BF16, theta), G.make_model(widths, eck.BF16, theta)
    steps = 6 if epoch < 3 else 9
    _, loss = G.update_gpu(a, x, e, steps, mb)
    for _ in range(steps // epoch):  # (a call starts with the first minibatch again)
        _, loss_b = G.update_gpu(b, x, e, epoch, mb)
    assert np.array_equal(a.get_state().cpu().numpy(), b.get_state().cpu().numpy())
    assert loss == loss_b


@pytest.mark.parametrize("widths,mb,ld_extra", [([64, 256, 256, 1], 250, 2), ([64, 128, 128, 1], 333, 4), ([32, 64, 64, 1], 201, 2),
                                                ([64, 512, 512, 1], 129, 0), ([64, 256, 256, 1], 65, 6), ([64, 128, 128, 1], 128, 2),
                                                ([64, 256, 256, 1], 20, 2)])
def test_bf16_refit_of_ragged_minibatches(G, widths, mb, ld_extra):
    """Minibatches that are no multiple of 64, and features that are not whole 16 bytes apart: rows past the minibatch count
    for nothing.  The last is so small that its steps run product by product."""
    test_bf16_refit_rows_past_a_threads_32(G, widths, mb, ld_extra)


def test_bf16_refits_on_two_streams_at_once(G):
    """Two crews may share the chip, and a die: each refit ends as it does alone."""
    import torch
    widths, n, mb, steps = [64, 256, 256, 1], 1024, 512, 24
    _, b16, e = _pairs(n)
    x, energy = G.bf16_dev(b16), G.to_dev(e.astype(np.float32))
    thetas = [synth.mlp_theta(widths, 4 + i, bf16=True) for i in range(4)]
    want = []
    for t in thetas:
        m = G.make_model(widths, eck.BF16, t)
        G.update_gpu(m, x, e, steps, mb)
        want.append(m.get_state().cpu().numpy())
    models = [G.make_model(widths, eck.BF16, t) for t in thetas]
    streams = [torch.cuda.Stream() for _ in thetas]
    ws = [torch.empty(eck.costmodel_update_workspace_bytes(m, n, mb), dtype=torch.uint8, device="cuda") for m in models]
    out = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    for i, s in enumerate(streams):
        with torch.cuda.stream(s):
            eck.costmodel_update(models[i], x, energy, steps, mb, out[2 * i:2 * i + 1], out[2 * i + 1:2 * i + 2], ws[i])
    torch.cuda.synchronize()
    for m, w in zip(models, want):
        assert np.array_equal(m.get_state().cpu().numpy(), w)


@pytest.mark.parametrize("widths,mb,epoch", [([64, 128, 128, 1], 250, 2), ([64, 128, 128, 1], 512, 1), ([64, 17, 48, 1], 15, 2), ([32, 1, 1, 1], 1, 2),
                                             ([32, 50, 30, 1], 497, 1), ([64, 113, 127, 1], 33, 2), ([32, 64, 64, 1], 16, 1)])
def test_fp32_steps_of_a_crew_are_those_of_two_launches(G, widths, mb, epoch):
    """The same for an fp32 model of up to 128 units: calls of one or two steps launch each by itself, longer ones run by a crew."""
    f32, _, e = _pairs(mb * epoch)
    x = G.to_dev(np.ascontiguousarray(f32[:widths[0]]))
    theta = synth.mlp_theta(widths, 4, bias_scale=0.1)
    a, b = G.make_model(widths, eck.F32, theta), G.make_model(widths, eck.F32, theta)
    _, loss = G.update_gpu(a, x, e, 6, mb)
    for _ in range(6 // epoch):
        _, loss_b = G.update_gpu(b, x, e, epoch, mb)
    assert np.array_equal(a.get_state().cpu().numpy(), b.get_state().cpu().numpy())
    assert loss == loss_b


@pytest.mark.parametrize("dtype,tol", [("bf16", 2e-2), ("f32", 1e-3)])
def test_steps_of_minibatches_past_4_gib(G, dtype, tol):
    """2.4 million rows of 512 units: a matrix of activations is 4.9 GB, and what lies behind 2^32 bytes of it counts most (the
    last 300 000 labels are a hundredth of the others, so their derivatives a hundred times theirs).  One step from zero moments
    leaves 0.1 g in the first one, compared layer by layer with the gradient in 64 bits; bfloat16's operands as in the tests
    above; in fp32 a part's chain of 2.4e6 / 8 terms, rounded at random, is off by sqrt(3e5) 2^-24 of it, 3e-5."""
    import torch
    widths, rows, late = [64, 512, 512, 1], 2400000, 300000
    P, F = synth.param_count(widths), widths[0]
    theta = synth.mlp_theta(widths, 6, bf16=True, bias_scale=0.2)
    model = G.make_model(widths, eck.BF16 if dtype == "bf16" else eck.F32, theta)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.rand((F, rows), generator=gen, device="cuda") * 4.0
    e = torch.rand(rows, generator=gen, device="cuda") + 1.0
    e[rows - late:] *= 0.01
    if dtype == "bf16":
        x = x.to(torch.bfloat16)
    out = torch.zeros(2, device="cuda")
    ws = torch.empty(eck.costmodel_update_workspace_bytes(model, rows, rows), dtype=torch.uint8, device="cuda")
    eck.costmodel_update(model, x, e, 1, rows, out[0:1], out[1:2], ws)
    del ws
    got = model.get_state()[P:2 * P].double() / (1.0 - float(np.float32(0.9)))
    y = (e / e.max()).double()
    layers, at = [], 0
    t = G.to_dev(theta).double()
    for fi, fo in zip(widths[:-1], widths[1:]):
        layers += [t[at:at + fi * fo].view(fi, fo), t[at + fi * fo:at + fi * fo + fo]]
        at += fi * fo + fo
    w1, b1, w2, b2, w3, b3 = layers
    want = [torch.zeros_like(v) for v in layers]
    for lo in range(0, rows, 1 << 17):
        xs, ys = x[:, lo:lo + (1 << 17)].double(), y[lo:lo + (1 << 17), None]
        h1 = torch.relu(xs.t() @ w1 + b1)
        h2 = torch.relu(h1 @ w2 + b2)
        dy = 2.0 * (h2 @ w3 + b3 - ys) / (ys * rows)
        d2 = (dy @ w3.t()) * (h2 > 0)
        d1 = (d2 @ w2.t()) * (h1 > 0)
        for g, v in zip(want, (xs @ d1, d1.sum(0), h1.t() @ d2, d2.sum(0), h2.t() @ dy, dy.sum(0))):
            g += v
    at = 0
    for g in want:
        part = got[at:at + g.numel()]
        at += g.numel()
        off = float((part - g.flatten()).norm() / g.norm())
        assert off <= tol, (tuple(g.shape), off)


@pytest.mark.parametrize("widths,dtype,mb,steps", [([64, 256, 256, 1], "bf16", 64, 1), ([64, 256, 256, 1], "bf16", 64, 4), ([64, 256, 256, 1], "bf16", 20, 2),
                                                   ([64, 128, 128, 1], "f32", 64, 2), ([64, 128, 128, 1], "f32", 64, 3)])
@pytest.mark.parametrize("done", [4294967040.0, 1e10])
def test_a_state_of_many_steps(G, widths, dtype, mb, steps, done):
    """A step count around 2^32 and past it, which a caller may set: Adam's corrections are 1.  With lr = 1e-6 the gradients stay what they
    are, and a weight moves by some 3 lr a step (0.1 g over sqrt(0.001) |g|, then more) whatever their size; bfloat16 rounds
    them by 2^-8 and flips a few activations, so that one weight in a hundred, whose gradient vanishes, may be further off than 0.1 lr a step
    and the weight's own rounding."""
    P = synth.param_count(widths)
    _, b16, e = _pairs(mb)
    x = oracle.bf16_bits_to_f32(b16)
    theta = synth.mlp_theta(widths, 4, bf16=True, bias_scale=0.1)
    st = _oracle_state(theta)
    st[3 * P] = done
    model = eck.Model(widths, eck.BF16 if dtype == "bf16" else eck.F32)
    model.set_state(G.to_dev(st.astype(np.float32)))
    G.update_gpu(model, G.bf16_dev(b16) if dtype == "bf16" else G.to_dev(x), e, steps, mb, lr=1e-6)
    oracle.update(widths, st, x, e, steps, mb, lr=1e-6, bf16_weights=dtype == "bf16")
    got = model.get_state().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    assert np.quantile(np.abs(got[:P] - st[:P]), 0.99) <= (1e-7 + 2.0 ** -24 * np.abs(theta).max()) * steps


@pytest.mark.parametrize("widths,dtype,mb,epoch", [([64, 256, 256, 1], "bf16", 512, 2), ([64, 128, 128, 1], "bf16", 250, 1), ([32, 64, 64, 1], "bf16", 64, 3),
                                                   ([64, 128, 128, 1], "f32", 250, 2), ([32, 50, 30, 1], "f32", 497, 1), ([64, 128, 128, 1], "f32", 16, 1)])
@pytest.mark.parametrize("candidates,at_once", [(1, 1), (3, 3), (7, 7), (32, 1), (32, 5)])
def test_steps_of_small_and_growing_crews(G, widths, dtype, mb, epoch, candidates, at_once):
    """Crews of fewer members than there are blocks of rows and tiles of weights, and such as take members on between steps, as
    beside other work on the chip: the bits of two launches a step."""
    import ctypes as C
    import torch
    f32, b16, e = _pairs(mb * epoch + (mb * epoch & 1))
    F, n, e = widths[0], mb * epoch, e[:mb * epoch]
    x = G.bf16_dev(b16[:F].copy()) if dtype == "bf16" else G.to_dev(np.ascontiguousarray(f32[:F]))
    kind = eck.BF16 if dtype == "bf16" else eck.F32
    theta = synth.mlp_theta(widths, 4, bf16=dtype == "bf16", bias_scale=0.1)
    a, b = G.make_model(widths, kind, theta), G.make_model(widths, kind, theta)
    steps = 12
    energy, out = G.to_dev(e.astype(np.float32)), torch.zeros(2, device="cuda")
    ws = torch.empty(eck.costmodel_update_workspace_bytes(a, n, mb), dtype=torch.uint8, device="cuda")
    update = eck.lib().eck_update_by_crew
    update.restype = C.c_int32
    update.argtypes = [C.c_void_p, C.c_void_p, C.c_int32, C.c_uint64, C.c_void_p, C.c_uint64, C.c_int32, C.c_int32] + [C.c_float] * 4 + \
        [C.c_void_p, C.c_void_p, C.c_void_p, C.c_uint64, C.c_uint32, C.c_uint32, C.c_void_p]
    assert update(a.h, x.data_ptr(), kind, x.shape[1], energy.data_ptr(), n, steps, mb, 1e-3, 0.9, 0.999, 1e-8, out.data_ptr(),
                  out.data_ptr() + 4, ws.data_ptr(), ws.numel(), candidates, at_once, torch.cuda.current_stream().cuda_stream) == eck.OK
    short = epoch if epoch > 1 else 2  # steps of a call that launches each: as many as bring the minibatches round, or the same one again
    for _ in range(steps // short):
        _, loss_b = G.update_gpu(b, x, e, short, mb)
    assert np.array_equal(a.get_state().cpu().numpy(), b.get_state().cpu().numpy())
    assert float(out[1]) == loss_b
