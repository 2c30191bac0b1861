"""The calls a program makes of this library, at the sizes it makes them, for timing and comparison.

A search for low-energy schedules generates candidates and computes their features, scores them with an energy and a
latency model, selects under the latency-then-energy objective, and refits the models on measured kernels.  Every case
is one of those steps through the Python entry points (one is a whole small round), on resident buffers that such a
program keeps: spaces, models, workspaces and result arrays are made in prepare(), new inputs come with the seed.

exact() restates the arithmetic in plain torch in 64 bits, without the library.  It has no value for the feature
matrices of the generation cases: they are fixed-point logarithms of integer counts and compared bit for bit.
"""
import math

import torch

from paper_2411_18873_amd import eck, synth

DEV = "cuda"
MASK64 = (1 << 64) - 1

# the operators of the configurations and of the paper's evaluation that the generation cases draw from
OPERATORS = {
    "conv": synth.CONFIGS["c2"]["problem"],
    "bgemm": synth.CONFIGS["c3"]["problem"],
    "MM2": synth.paper_operators()["MM2"],
    "MV4": synth.paper_operators()["MV4"],
    "CONV2": synth.paper_operators()["CONV2"],
}
MODES = {"sample": eck.MODE_SAMPLE, "mutate": eck.MODE_MUTATE, "crossover": eck.MODE_CROSSOVER}
KINDS = {"split": eck.SPACE_SPLIT, "xred": eck.SPACE_SPLIT_XRED}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
CODE = {"bf16": eck.BF16, "f32": eck.F32}
BF16_WIDTHS = ((64, 512, 512), (64, 256, 256), (64, 128, 128), (32, 64, 64))
F32_WIDTHS = ((64, 512, 512), (64, 256, 256), (64, 128, 128), (32, 64, 64), (64, 200, 96), (32, 50, 30))


def listed():
    return [
        # config 1 whole: every schedule of one small GEMM through the round; a chain of small dependent launches
        dict(name="round_knob_6400", do="round", M=512, N=512, K=512, first=0, n=6400, k=16, alpha=1.1),
        # the generation step of a whole-network sweep: 64 operator shapes side by side
        dict(name="sweep_generate_64x32768", do="sweep", spaces=64, n=1 << 15, feat="bf16"),
        # one generation bred from the survivors of the last, repeated children dropped; reduction split over threads
        dict(name="breed_mv_xred_f32", do="breed", op="MV4", kind="xred", mode="crossover", n=260001, parents=256,
             feat="f32", n_feat=64, dedup=True),
        # the sweep's latency model, with the least legal latency of every segment
        dict(name="score_bf16_512_min", do="score", F=64, H1=512, H2=512, model="bf16", feat="bf16", n=1 << 22,
             segments=64),
        # one operator's generation under the mid-sized model
        dict(name="score_bf16_256", do="score", F=64, H1=256, H2=256, model="bf16", feat="bf16", n=1 << 20, segments=0),
        # the same model kept in 32 bits, a ragged generation
        dict(name="score_f32_256", do="score", F=64, H1=256, H2=256, model="f32", feat="f32", n=100003, segments=0),
        # the sweep's selection, finding the least latencies itself
        dict(name="select_threshold_64x2e18", do="select", mode="threshold", n=1 << 18, segments=64, k=32, alpha=1.1, m=0),
        # Alg. 1's selection: the 128 fastest of a generation, of these the 64 of least energy
        dict(name="select_rank_2e20", do="select", mode="rank", n=1 << 20, segments=1, k=64, alpha=1.0, m=128),
        # the refit after a round of measurements: one pass over config 4's record
        dict(name="refit_bf16_256", do="refit", F=64, H1=256, H2=256, model="bf16", feat="bf16", pairs=4096, batch=512,
             steps=8),
        # an fp32 model refitted on a smaller record
        dict(name="refit_f32_128", do="refit", F=64, H1=128, H2=128, model="f32", feat="f32", pairs=1000, batch=250,
             steps=16),
        # the paper's model form over a generation: 100 trees of depth 6
        dict(name="trees_score_100x6", do="trees_score", n_feat=64, depth=6, trees=100, feat="bf16", n=1 << 20),
        # its refit after a round of measurements: 8 more trees on everything measured so far
        dict(name="trees_refit_1536", do="trees_refit", n_feat=64, depth=6, trees=40, rounds=8, pairs=1536, feat="bf16"),
    ]


def _between(rng, lo, hi):
    """a whole number between lo and hi, uniform over the logarithm"""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    do = rng.choice(["round", "sweep", "breed", "score", "score", "score", "select", "select", "refit", "refit",
                     "trees_score", "trees_refit"])
    if do == "round":
        n = _between(rng, 200, 6400)
        M, N, K = (_between(rng, 64, 4096) for _ in range(3))
        return dict(do=do, M=M, N=N, K=K, first=rng.randint(0, 6400 - n), n=n, k=_between(rng, 1, min(64, n)),
                    alpha=rng.choice([1.1, 1.5, math.inf]))
    if do == "sweep":
        spaces = _between(rng, 1, 64)
        return dict(do=do, spaces=spaces, n=_between(rng, 512, min(1 << 17, (1 << 22) // spaces)), feat=rng.choice(["bf16", "f32"]))
    if do == "breed":
        return dict(do=do, op=rng.choice(sorted(OPERATORS)), kind=rng.choice(sorted(KINDS)), mode=rng.choice(sorted(MODES)),
                    n=_between(rng, 1000, 1 << 20), parents=_between(rng, 8, 1024), feat=rng.choice(["bf16", "f32"]),
                    n_feat=rng.choice([32, 64]), dedup=rng.random() < 0.5)
    if do == "score":
        model = rng.choice(["bf16", "bf16", "f32"])
        F, H1, H2 = rng.choice(BF16_WIDTHS if model == "bf16" else F32_WIDTHS)
        feat = "f32" if model == "f32" else rng.choice(["bf16", "bf16", "f32"])
        most = (1 << 22) * (64 * 512 + 512 * 512) // (F * H1 + H1 * H2)  # no more arithmetic than the largest listed one
        n = _between(rng, 1000, min(1 << 22, most) if model == "bf16" else 1 << (15 if H2 > 256 else 17))
        segments = rng.choice([0, 0, 1, 16, 64])
        n = max(segments, n - n % segments) if segments else n
        return dict(do=do, F=F, H1=H1, H2=H2, model=model, feat=feat, n=n, segments=segments)
    if do == "select":
        mode = rng.choice(["threshold", "threshold", "rank", "known_min"])
        segments = rng.choice([1, 1, 8, 64])
        n = _between(rng, 4096, (1 << 24) // segments if segments > 1 else 1 << 21)
        return dict(do=do, mode=mode, n=n, segments=segments, k=_between(rng, 1, 1024),
                    alpha=rng.choice([1.1, 1.5, math.inf]) if mode == "threshold" else 1.1,
                    m=_between(rng, 16, 1024) if mode == "rank" else 0)
    if do == "refit":
        model = rng.choice(["bf16", "f32"])
        F, H1, H2 = rng.choice(BF16_WIDTHS if model == "bf16" else F32_WIDTHS)
        batch = rng.choice([64, 128, 250, 256, 512])
        # (more bf16 steps than these let a last-bit difference grow to the size of the weights' own changes)
        return dict(do=do, F=F, H1=H1, H2=H2, model=model, feat="f32" if model == "f32" else rng.choice(["bf16", "f32"]),
                    pairs=batch * rng.randint(1, 8), batch=batch, steps=_between(rng, 1, 16 if model == "f32" else 8))
    if do == "trees_score":
        return dict(do=do, n_feat=rng.choice([32, 64]), depth=rng.randint(3, 8), trees=_between(rng, 8, 150),
                    feat=rng.choice(["bf16", "bf16", "f32"]), n=_between(rng, 1000, 1 << 21))
    return dict(do=do, n_feat=rng.choice([32, 64]), depth=rng.randint(3, 8), trees=rng.choice([0, 40, 100]),
                rounds=_between(rng, 1, 12), pairs=_between(rng, 64, 8192), feat=rng.choice(["bf16", "bf16", "f32"]))


# ------------------------------------------------------------------------------------------------- inputs


def _generator(case, seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + salt * 7919) & 0x7FFFFFFF)
    return g


def _even(n):
    return n + (n & 1)


def _features(n_feat, n, dtype, g):
    """Fixed-point logarithms as candidates of one space have them: a level and a spread per feature, every tenth
    feature the same for all candidates, ten bits behind the point; [n_feat][ld], ld even."""
    ld = _even(n)
    level = 2.0 + 22.0 * torch.rand(n_feat, 1, generator=g, device=DEV)
    spread = 0.5 + 2.5 * torch.rand(n_feat, 1, generator=g, device=DEV)
    spread[::10] = 0.0
    out = torch.empty(n_feat, ld, dtype=dtype, device=DEV)
    for f in range(0, n_feat, 8):  # a few rows at a time: little scratch memory beside the matrix
        x = level[f:f + 8] + spread[f:f + 8] * torch.randn(min(8, n_feat - f), ld, generator=g, device=DEV)
        out[f:f + 8] = (x.clamp_(0.0, 47.0).mul_(1024.0).floor_().div_(1024.0)).to(dtype)
    return out


def _theta(F, H1, H2, bf16, g):
    """W ~ N(0, 1/fan_in), small biases, output weights shifted so that scores are mostly positive, as those of a
    fitted model are (it predicts energies normalised to (0, 1]); values that bf16 holds for a bf16 model."""
    parts = []
    for fi, fo in ((F, H1), (H1, H2), (H2, 1)):
        w = torch.randn(fi, fo, generator=g, device=DEV) / math.sqrt(fi)
        if fi == F:
            w /= 12.0  # features are around 12: hidden units of order one
        if fo == 1:
            w = w + 1.0 / math.sqrt(fi)
        parts += [w.flatten(), 0.05 * torch.randn(fo, generator=g, device=DEV)]
    theta = torch.cat(parts)
    return theta.to(torch.bfloat16).float() if bf16 else theta


def _energies(feat, n, g):
    """measured energies: a positive-weight linear form of the features times lognormal(0, 0.1) noise"""
    u = torch.rand(feat.shape[0], 1, generator=g, device=DEV, dtype=torch.float64)
    z = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    return ((u / u.sum() * feat[:, :n].double()).sum(0) * torch.exp(0.1 * z)).float()


def _scores(case, seed):
    """energies, latencies and legality flags of a generation (positive, a third of the candidates legal)"""
    g = _generator(case, seed)
    n = case["n"] * case["segments"]
    energy = 2.0 + 0.4 * torch.randn(n, generator=g, device=DEV)
    latency = 2.0 + 0.4 * torch.randn(n, generator=g, device=DEV)
    legal = (torch.rand(n, generator=g, device=DEV) < 0.3).to(torch.uint8)
    return energy, latency, legal


def _ensemble(n_feat, depth, trees, g):
    """trees as boosting leaves them: thresholds on the quarter grid, one node in sixteen without a split, small leaves"""
    nodes = (1 << depth) - 1
    node_feat = torch.randint(0, n_feat, (trees, nodes), generator=g, device=DEV).to(torch.uint8)
    node_thr = torch.randint(8, 96, (trees, nodes), generator=g, device=DEV).float() / 4.0
    still = torch.rand(trees, nodes, generator=g, device=DEV) < 1.0 / 16.0
    node_thr[still] = math.inf
    node_feat[still] = 0
    leaf = 0.02 * torch.randn(trees, nodes + 1, generator=g, device=DEV)
    return node_feat.contiguous(), node_thr.contiguous(), leaf.contiguous()


def _knob_space(case):
    return synth.gemm(case["M"], case["N"], case["K"])


def _sweep_problems(case):
    return [synth.gemm(*s) for s in synth.sweep_shapes()[:case["spaces"]]]


def _empty(shape, dtype):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def _select_buffers(n, segments, k, m=0):
    return dict(idx=_empty((segments, k), torch.int32), energy_out=_empty((segments, k), torch.float32),
                count=_empty(segments, torch.int32),
                ws=torch.empty(eck.topk_select_workspace_bytes(n, segments, k, m_latency=m), dtype=torch.uint8, device=DEV))


def prepare(case, seed):
    do, g = case["do"], _generator(case, seed)
    s = dict(case=case, do=do)
    if do == "round":
        n, ld = case["n"], _even(case["n"])
        s["space"] = eck.Space(_knob_space(case), eck.SPACE_KNOB).upload()
        s["models"] = []
        for _ in range(2):
            m = eck.Model([32, 64, 64, 1], eck.F32)
            m.set_state(_theta(32, 64, 64, False, g))
            s["models"].append(m)
        s.update(genes=_empty((6, ld), torch.int16), feat=_empty((32, ld), torch.float32), legal=_empty(n, torch.uint8),
                 energy=_empty(n, torch.float32), latency=_empty(n, torch.float32), **_select_buffers(n, 1, case["k"]))
    elif do == "sweep":
        s["spaces"] = [eck.Space(p, eck.SPACE_SPLIT).upload() for p in _sweep_problems(case)]
        s["seeds"] = [seed * 1000 + i for i in range(case["spaces"])]
        total = case["spaces"] * case["n"]
        s.update(genes=_empty((s["spaces"][0].n_genes, _even(total)), torch.int16),
                 feat=_empty((64, _even(total)), TORCH[case["feat"]]), legal=_empty(total, torch.uint8))
    elif do == "breed":
        n = case["n"]
        s["space"] = eck.Space(OPERATORS[case["op"]], KINDS[case["kind"]]).upload()
        s["seed"] = seed & MASK64
        radix = torch.tensor(s["space"].radix, device=DEV).view(-1, 1)
        unit = torch.rand(len(s["space"].radix), case["parents"], generator=g, device=DEV)
        s["parents"] = (unit * radix).long().clamp_(max=radix - 1).to(torch.int16).contiguous()
        s.update(genes=_empty((s["space"].n_genes, _even(n)), torch.int16),
                 feat=_empty((case["n_feat"], _even(n)), TORCH[case["feat"]]), legal=_empty(n, torch.uint8))
        if case["dedup"]:
            s["ws"] = torch.empty(eck.candidates_dedup_workspace_bytes(n), dtype=torch.uint8, device=DEV)
    elif do == "score":
        F, H1, H2, n = case["F"], case["H1"], case["H2"], case["n"]
        s["model"] = eck.Model([F, H1, H2, 1], CODE[case["model"]])
        s["model"].set_state(_theta(F, H1, H2, case["model"] == "bf16", g))
        s["feat"] = _features(F, n, TORCH[case["feat"]], g)
        s["score"] = _empty(n, torch.float32)
        if case["segments"]:
            s["legal"] = (torch.rand(n, generator=g, device=DEV) < 0.3).to(torch.uint8)
            s["key"] = _empty(case["segments"], torch.int32)
    elif do == "select":
        n = case["n"] * case["segments"]
        s["energy"], s["latency"], s["legal"] = _scores(case, seed)
        s.update(_select_buffers(n, case["segments"], case["k"], case["m"]))
        if case["mode"] == "known_min":
            least = torch.where(s["legal"].bool(), s["latency"], math.inf).view(case["segments"], -1).amin(1)
            s["key"] = least.view(torch.int32) ^ -(1 << 31)  # the order key of a positive float
    elif do == "refit":
        F, H1, H2 = case["F"], case["H1"], case["H2"]
        s["model"] = eck.Model([F, H1, H2, 1], CODE[case["model"]])
        s["theta"] = _theta(F, H1, H2, case["model"] == "bf16", g)
        s["feat"] = _features(F, case["pairs"], TORCH[case["feat"]], g)
        s["energy"] = _energies(s["feat"], case["pairs"], g)
        s.update(snr=_empty(1, torch.float32), loss=_empty(1, torch.float32),
                 ws=torch.empty(eck.costmodel_update_workspace_bytes(s["model"], case["pairs"], case["batch"]),
                                dtype=torch.uint8, device=DEV))
    elif do == "trees_score":
        s["trees"] = eck.Trees(case["n_feat"], case["depth"], case["trees"], 0.5)
        s["trees"].set(*_ensemble(case["n_feat"], case["depth"], case["trees"], g))
        s["feat"] = _features(case["n_feat"], case["n"], TORCH[case["feat"]], g)
        s["score"] = _empty(case["n"], torch.float32)
    else:
        s["trees"] = eck.Trees(case["n_feat"], case["depth"], case["trees"] + case["rounds"], 0.5)
        s["ensemble"] = _ensemble(case["n_feat"], case["depth"], case["trees"], g)
        s["feat"] = _features(case["n_feat"], case["pairs"], TORCH[case["feat"]], g)
        s["energy"] = _energies(s["feat"], case["pairs"], g)
        s.update(snr=_empty(1, torch.float32), loss=_empty(1, torch.float32),
                 ws=torch.empty(eck.treemodel_update_workspace_bytes(s["trees"], case["pairs"]), dtype=torch.uint8, device=DEV))
    return s


# --------------------------------------------------------------------------------------------------- runs


def run(s):
    case, do = s["case"], s["do"]
    if do == "round":
        n = case["n"]
        eck.candidate_enumerate(s["space"], eck.MODE_EXHAUSTIVE, n, s["genes"], first_index=case["first"])
        eck.features_compute(s["space"], s["genes"], n, 32, eck.F32, feat_out=s["feat"], legal_out=s["legal"])
        eck.costmodel_score(s["models"][0], s["feat"], n, s["energy"])
        eck.costmodel_score(s["models"][1], s["feat"], n, s["latency"])
        eck.topk_select(s["energy"], s["latency"], s["legal"], 1, case["k"], s["idx"], s["energy_out"], s["count"], s["ws"],
                        alpha=case["alpha"])
        return {k: s[k] for k in ("genes", "feat", "legal", "energy", "latency", "idx", "energy_out", "count")}
    if do == "sweep":
        eck.candidate_enumerate_batch(s["spaces"], eck.MODE_SAMPLE, case["n"], s["genes"], s["seeds"])
        eck.features_compute_batch(s["spaces"], s["genes"], case["n"], 64, CODE[case["feat"]], feat_out=s["feat"],
                                   legal_out=s["legal"])
        return {k: s[k] for k in ("genes", "feat", "legal")}
    if do == "breed":
        n = case["n"]
        eck.candidate_enumerate(s["space"], MODES[case["mode"]], n, s["genes"], seed=s["seed"], round=3,
                                parents=None if case["mode"] == "sample" else s["parents"], p_mut_q32=synth.P_MUT_Q32)
        eck.features_compute(s["space"], s["genes"], n, case["n_feat"], CODE[case["feat"]], feat_out=s["feat"],
                             legal_out=s["legal"])
        if case["dedup"]:
            eck.candidates_dedup(s["genes"], n, s["legal"], ws=s["ws"])
        return {k: s[k] for k in ("genes", "feat", "legal")}
    if do == "score":
        if not case["segments"]:
            eck.costmodel_score(s["model"], s["feat"], case["n"], s["score"])
            return {"score": s["score"]}
        eck.costmodel_score_min(s["model"], s["feat"], case["n"], s["score"], s["legal"], case["segments"], s["key"])
        # the keys as the numbers they order (every score that counts here is a number)
        return {"score": s["score"], "least": _numbers(s["key"])}
    if do == "select":
        args = (s["energy"], s["latency"], s["legal"], case["segments"], case["k"])
        out = (s["idx"], s["energy_out"], s["count"], s["ws"])
        if case["mode"] == "known_min":
            eck.topk_select_known_min(*args, s["key"], *out, alpha=case["alpha"])
        elif case["mode"] == "threshold":
            eck.topk_select(*args, *out, alpha=case["alpha"])
        else:
            eck.topk_select(*args, *out, mode=eck.SELECT_RANK, m_latency=case["m"])
        return {k: s[k] for k in ("idx", "energy_out", "count")}
    if do == "refit":
        s["model"].set_state(s["theta"])
        eck.costmodel_update(s["model"], s["feat"], s["energy"], case["steps"], case["batch"], s["snr"], s["loss"], s["ws"])
        state = s["model"].get_state()
        P = s["model"].n_params
        return {"theta": state[:P], "m": state[P:2 * P], "v": state[2 * P:3 * P], "t": state[3 * P:], "snr": s["snr"],
                "loss": s["loss"]}
    if do == "trees_score":
        eck.treemodel_score(s["trees"], s["feat"], case["n"], s["score"])
        return {"score": s["score"]}
    s["trees"].set(*s["ensemble"])
    eck.treemodel_update(s["trees"], s["feat"], s["energy"], case["rounds"], s["snr"], s["loss"], s["ws"])
    node_feat, node_thr, leaf = s["trees"].get()
    return {"node_feat": node_feat, "node_thr": node_thr, "leaf": leaf, "snr": s["snr"], "loss": s["loss"]}


def _numbers(key):
    """the floats whose order keys these are"""
    positive = key < 0  # the top bit of a key is set for positive numbers
    return torch.where(positive, key ^ -(1 << 31), ~key).view(torch.float32)


# --------------------------------------------------------------------------------------- work and tolerance


def work(case):
    do = case["do"]
    if do == "round":
        n = case["n"]
        return {"bytes": n * (2 * 6 + 4 * 32 + 1 + 8), "flops": 2 * n * 2 * (32 * 64 + 64 * 64 + 64)}
    if do == "sweep":
        total = case["spaces"] * case["n"]
        return {"bytes": total * (2 * 5 + 64 * (2 if case["feat"] == "bf16" else 4) + 1), "flops": 0}
    if do == "breed":
        genes = 2 * eck.Space(OPERATORS[case["op"]], KINDS[case["kind"]]).n_genes
        return {"bytes": case["n"] * (genes + case["n_feat"] * (2 if case["feat"] == "bf16" else 4) + 1), "flops": 0}
    if do == "score":
        F, H1, H2 = case["F"], case["H1"], case["H2"]
        per = F * (2 if case["feat"] == "bf16" else 4) + 4 + (1 if case["segments"] else 0)
        return {"bytes": case["n"] * per, "flops": case["n"] * 2 * (F * H1 + H1 * H2 + H2)}
    if do == "select":
        return {"bytes": case["n"] * case["segments"] * 9, "flops": 0}
    if do == "refit":
        F, H1, H2 = case["F"], case["H1"], case["H2"]
        P = F * H1 + H1 + H1 * H2 + H2 + H2 + 1
        rows = case["steps"] * case["batch"]
        # forward and both weight gradients, the second layer's way back; state in and out once
        return {"bytes": 6 * 4 * P + case["pairs"] * (F * (2 if case["feat"] == "bf16" else 4) + 4),
                "flops": case["pairs"] * 2 * (F * H1 + H1 * H2 + H2) + rows * 2 * (2 * F * H1 + 3 * H1 * H2 + 3 * H2)}
    if do == "trees_score":
        # one comparison per level and tree
        return {"bytes": case["n"] * (case["n_feat"] * (2 if case["feat"] == "bf16" else 4) + 4),
                "flops": case["n"] * case["trees"] * case["depth"]}
    # one pass over the bins per level and round
    return {"bytes": case["pairs"] * case["n_feat"] * (2 if case["feat"] == "bf16" else 4) + case["pairs"] * 4,
            "flops": case["rounds"] * case["depth"] * case["pairs"] * case["n_feat"] * 3 +
            case["pairs"] * case["trees"] * case["depth"]}


def tolerance(case):
    """four times what the library's results and exact()'s differ by, as measured over the declared ranges"""
    do = case["do"]
    if do in ("sweep", "breed", "select", "trees_score"):
        return "exact"  # integers, their fixed-point logarithms, copies of inputs, sums in a stated order
    if do == "round":
        return {"rel": 1e-6, "max": 1e-5}
    if do == "score":
        return {"rel": 1e-6, "max": 1e-5} if case["model"] == "f32" else {"rel": 3e-3, "max": 3e-2}
    if do == "refit":
        return {"rel": 1e-4, "max": 2e-3} if case["model"] == "f32" else {"rel": 3e-3, "max": 0.03}
    return {"rel": 1e-6, "max": 1e-5}  # splits are integer decisions; leaves, SNR and loss are rounded once


# ---------------------------------------------------------------------------------------- 64-bit restatement


def _layers(theta, F, H1, H2):
    out, at = [], 0
    for fi, fo in ((F, H1), (H1, H2), (H2, 1)):
        w = theta[at:at + fi * fo].view(fi, fo)
        out += [w, theta[at + fi * fo:at + fi * fo + fo]]
        at += fi * fo + fo
    return out


def _forward(theta, F, H1, H2, x):
    """scores of the columns of x in 64 bits, in slices that fit"""
    w1, b1, w2, b2, w3, b3 = (t.double() for t in _layers(theta, F, H1, H2))
    parts = []
    for c in range(0, x.shape[1], 1 << 18):
        h = torch.relu(x[:, c:c + (1 << 18)].t().double() @ w1 + b1)
        parts.append((torch.relu(h @ w2 + b2) @ w3 + b3).flatten())
    return torch.cat(parts)


def _select(energy, latency, legal, case, gate=None):
    """idx, energies and counts by sorting; gate: admitted candidates beside the legal ones, or by the case's mode"""
    S, k = case["segments"], case["k"]
    energy, latency, legal = energy.view(S, -1), latency.view(S, -1), legal.view(S, -1).bool()
    if gate is None and case["mode"] == "rank":
        least = torch.where(legal, latency, math.inf).sort(dim=1, stable=True).indices[:, :case["m"]]
        gate = torch.zeros_like(legal).scatter_(1, least, True)
    elif gate is None:
        low = torch.where(legal, latency, math.inf).amin(1, keepdim=True)
        slack = torch.tensor(case["alpha"], dtype=torch.float32, device=DEV) - 1.0
        gate = latency <= (low + slack * low.abs() if math.isfinite(case["alpha"]) else torch.full_like(low, math.inf))
    fine = gate & legal
    order = torch.where(fine, energy, math.inf).sort(dim=1, stable=True)
    count = fine.sum(1).clamp(max=k)
    empty = torch.arange(k, device=DEV).view(1, -1) >= count.view(-1, 1)
    idx = torch.where(empty, -1, order.indices[:, :k]).to(torch.int32)
    return {"idx": idx, "energy_out": torch.where(empty, math.inf, order.values[:, :k].double()), "count": count.to(torch.int32)}


def _knob_round(case, g):
    """the 32 features of knob schedules first .. first + n - 1 of a GEMM, restated over 64-bit integers"""
    n, M, N, K = case["n"], case["M"], case["N"], case["K"]
    cus, wave, lds, max_threads, max_blocks = synth.HW_MI355X
    rest = torch.arange(case["first"], case["first"] + n, device=DEV)
    genes = []
    for radix in (4, 4, 4, 4, 5, 5):
        genes.append(rest % radix)
        rest = rest // radix
    genes = torch.stack(genes[::-1])
    up = lambda a, b: (a + b - 1) // b  # noqa: E731
    tm, tn, tk, T = 16 << genes[0], 16 << genes[1], 8 << genes[2], 64 << genes[3]
    U, V = 1 << genes[4], 1 << genes[5]
    on_n = torch.minimum(T, tn)
    on_m = T // on_n
    fits = on_m <= tm
    rm, rn = torch.where(fits, tm // on_m, 1), tn // on_n
    one = torch.ones_like(tm)
    grid, threads, outs = up(M, tm) * up(N, tn), on_m * on_n, rm * rn
    stages, all_threads = up(K, tk), grid * threads
    tile_m, tile_n = on_m * rm, on_n * rn
    fp, b = (tile_m + tile_n) * tk, 2
    red, padded = stages * tk, all_threads * outs
    lts = up(up(fp, threads), V)
    smem, bytes_in = fp * b, grid * stages * fp * b
    blocks = torch.minimum(max_threads // threads, lds // smem).clamp(max=max_blocks)
    blocks = torch.where(smem > lds, 0, blocks)
    slots = cus * blocks.clamp(min=1)
    waves, tail, active = grid // slots, grid % slots, grid.clamp(max=cus)
    in_sec, out_sec = up(bytes_in, 32), up(padded * b, 32)
    flop = 2 * padded * red
    depth = sum((x > 1).long() for x in (up(M, tm), on_m, rm, up(N, tn), on_n, rn, stages, tk))
    low = torch.minimum(rn & -rn, V)
    must_in = (M * K + K * N) * b
    raw = [one * (2 * M * N * K), flop, outs * red, all_threads * (stages * (4 * lts + 2) + 2 * up(red, U)), outs,
           outs + rm + rn, grid, threads, up(threads, wave), blocks, active, cus - active, waves + (tail > 0).long(), tail,
           all_threads * stages * lts, in_sec, out_sec, all_threads * up(outs, V), smem, up(bytes_in, 128),
           all_threads * (rm + rn) * red, flop * 8 // (in_sec + out_sec), one * (must_in + M * N * b),
           bytes_in * 256 // must_in, stages, tk, tk, U, torch.minimum(U, tk) * outs, depth, V, low]
    v = torch.stack(raw) + 1
    e = torch.frexp(v.double()).exponent.long() - 1  # v is below 2^53
    tenth = torch.where(e >= 10, (v - (one << e)) >> (e - 10).clamp(min=0), (v - (one << e)) << (10 - e).clamp(min=0))
    legal = (threads >= 32) & (threads <= 1024) & fits & (smem <= lds) & (V * b <= 16) & (rn % V == 0)
    return genes, e.double() + tenth.double() / 1024.0, legal


def _refit(case, seed):
    """Adam on Eq. (1) in 64 bits; for a bf16 model on weights, first activations and deltas rounded as it defines them"""
    F, H1, H2 = case["F"], case["H1"], case["H2"]
    g = _generator(case, seed)
    bf16 = case["model"] == "bf16"
    theta = _theta(F, H1, H2, bf16, g).double()
    feat = _features(F, case["pairs"], TORCH[case["feat"]], g)
    energy = _energies(feat, case["pairs"], g).double()
    r = (lambda t: t.to(torch.bfloat16).double()) if bf16 else (lambda t: t)
    x, y = r(feat[:, :case["pairs"]].t().double()), energy / energy.max()

    def forward(rows):
        w1, b1, w2, b2, w3, b3 = _layers(r(theta), F, H1, H2)
        h1 = r(torch.relu(rows @ w1 + b1))
        h2 = torch.relu(h1 @ w2 + b2)
        return h1, h2, (h2 @ w3 + b3).flatten(), w2, w3

    pred = forward(x)[2]
    snr = (y * y).sum() / ((pred - y) ** 2).sum()
    m, v, B, lr, beta1, beta2, loss = torch.zeros_like(theta), torch.zeros_like(theta), case["batch"], 1e-3, 0.9, 0.999, snr
    for t in range(case["steps"]):
        rows = slice(t % (case["pairs"] // B) * B, t % (case["pairs"] // B) * B + B)
        h1, h2, p, w2, w3 = forward(x[rows])
        loss = ((p - y[rows]) ** 2 / y[rows]).mean()
        dy = (2.0 * (p - y[rows]) / (y[rows] * B)).view(-1, 1)
        d2 = r(dy * w3.t() * (h2 > 0))
        d1 = r((d2 @ w2.t()) * (h1 > 0))
        grad = torch.cat([(x[rows].t() @ d1).flatten(), d1.sum(0), (h1.t() @ d2).flatten(), d2.sum(0), (h2.t() @ dy).flatten(),
                          dy.sum(0)])
        m, v = beta1 * m + (1 - beta1) * grad, beta2 * v + (1 - beta2) * grad * grad
        theta = theta - lr * (m / (1 - beta1 ** (t + 1))) / ((v / (1 - beta2 ** (t + 1))).sqrt() + 1e-8)
    return {"theta": theta, "m": m, "v": v, "t": torch.full((1,), float(case["steps"]), dtype=torch.float64, device=DEV),
            "snr": snr.view(1), "loss": loss.view(1)}


def _walk(node_feat, node_thr, leaf, depth, x, n):
    """the leaf values of every tree for the candidates, tree by tree"""
    nodes = (1 << depth) - 1
    col = torch.arange(n, device=DEV)
    for f, t, w in zip(node_feat.long(), node_thr, leaf):
        at = torch.zeros(n, dtype=torch.long, device=DEV)
        for _ in range(depth):
            at = 2 * at + torch.where(x[f[at], col].float() < t[at], 1, 2)
        yield w[at - nodes]


def _boost(case, seed):
    """the boosting rounds restated: integer histograms by scattered sums, gains in 64 bits"""
    F, depth, n, rounds = case["n_feat"], case["depth"], case["pairs"], case["rounds"]
    g = _generator(case, seed)
    node_feat, node_thr, leaf = _ensemble(F, depth, case["trees"], g)
    feat = _features(F, n, TORCH[case["feat"]], g)
    energy = _energies(feat, n, g)
    eta, unit = float(torch.tensor(0.3, dtype=torch.float32)), 1048576.0
    lam, nodes = 1.0 * unit, (1 << depth) - 1
    y = energy / energy.max()  # labels and predictions are 32-bit by definition: they feed integer decisions
    p = torch.full((n,), 0.5, device=DEV)
    for w in _walk(node_feat, node_thr, leaf, depth, feat, n):
        p = p + w
    snr = (y.double() ** 2).sum() / ((p.double() - y.double()) ** 2).sum()
    x = feat[:, :n].float()
    bins = (x * 4.0).floor().clamp(0, 255).long()
    out_f, out_t, out_w = [], [], []
    for _ in range(rounds):
        yd, d = y.double(), p.double() - y.double()
        gh = [((2.0 * d / yd).clamp(-unit, unit) * unit).round().long(), ((2.0 / yd).clamp(-unit, unit) * unit).round().long(),
              torch.ones(n, dtype=torch.long, device=DEV)]
        tf = torch.zeros(nodes, dtype=torch.long, device=DEV)
        tt = torch.full((nodes,), math.inf, device=DEV)
        at = torch.zeros(n, dtype=torch.long, device=DEV)  # node within the level
        for level in range(depth):
            L = 1 << level
            cell = ((at.view(1, -1) * F + torch.arange(F, device=DEV).view(-1, 1)) * 256 + bins).flatten()
            left = [torch.zeros(L * F * 256, dtype=torch.long, device=DEV).index_add_(0, cell, q.expand(F, n).flatten())
                    .view(L, F, 256).cumsum(2) for q in gh]
            GL, HL, NL = left
            G, H, N = (q[:, :, 255:] for q in left)
            sq = lambda a, b: a.double() * a.double() / (b.double() + lam)  # noqa: E731
            gain = sq(GL, HL) + sq(G - GL, H - HL) - sq(G, H)
            gain = torch.where((NL > 0) & (NL < N), gain, -math.inf)
            gain[:, :, 255] = -math.inf
            best, rank = gain.view(L, -1).max(1).values, gain.view(L, -1).argmax(1)
            rank = torch.where(gain.view(L, -1) == best.view(-1, 1), torch.arange(F * 256, device=DEV).view(1, -1), F * 256).amin(1)
            split = best > 0.0
            f, t = torch.where(split, rank // 256, 0), torch.where(split, (rank % 256 + 1).float() * 0.25, math.inf)
            tf[L - 1:2 * L - 1], tt[L - 1:2 * L - 1] = f, t
            at = 2 * at + torch.where(x[f[at], torch.arange(n, device=DEV)] < t[at], 0, 1)
        # a node that no pair stands on does not split
        sums = [torch.zeros(nodes + 1, dtype=torch.long, device=DEV).index_add_(0, at, q) for q in gh]
        w = torch.where(sums[2] > 0, -eta * sums[0].double() / (sums[1].double() + lam), 0.0)
        p = p + w.float()[at]
        out_f.append(tf), out_t.append(tt), out_w.append(w)
    loss = ((p.double() - y.double()) ** 2 / y.double()).mean()
    return {"node_feat": torch.cat([node_feat, torch.stack(out_f).to(torch.uint8)]),
            "node_thr": torch.cat([node_thr, torch.stack(out_t)]).double(),
            "leaf": torch.cat([leaf.double(), torch.stack(out_w)]), "snr": snr.view(1), "loss": loss.view(1)}


def exact(case, seed):
    do, g = case["do"], _generator(case, seed)
    if do == "round":
        thetas = [_theta(32, 64, 64, False, g) for _ in range(2)]
        genes, x, legal = _knob_round(case, g)
        ld = _even(case["n"])
        energy, latency = (_forward(t, 32, 64, 64, x) for t in thetas)
        picked = _select(energy, latency, legal, dict(case, segments=1, mode="threshold"))
        wide = lambda t: torch.nn.functional.pad(t, (0, ld - case["n"]))  # noqa: E731
        return dict(genes=wide(genes).to(torch.int16), feat=wide(x), legal=legal.to(torch.uint8), energy=energy, latency=latency, **picked)
    if do == "score":
        F, H1, H2, n = case["F"], case["H1"], case["H2"], case["n"]
        theta = _theta(F, H1, H2, case["model"] == "bf16", g)
        feat = _features(F, n, TORCH[case["feat"]], g)
        if case["model"] == "bf16":
            feat = feat.to(torch.bfloat16)
        score = _forward(theta, F, H1, H2, feat[:, :n])
        if not case["segments"]:
            return {"score": score}
        legal = torch.rand(n, generator=g, device=DEV) < 0.3
        return {"score": score, "least": torch.where(legal, score, math.inf).view(case["segments"], -1).amin(1)}
    if do == "select":
        return _select(*_scores(case, seed), case)
    if do == "refit":
        return _refit(case, seed)
    if do == "trees_score":
        ensemble = _ensemble(case["n_feat"], case["depth"], case["trees"], g)
        feat = _features(case["n_feat"], case["n"], TORCH[case["feat"]], g)
        score = torch.full((case["n"],), 0.5, dtype=torch.float64, device=DEV)
        for w in _walk(*ensemble, case["depth"], feat, case["n"]):
            score += w.double()
        return {"score": score}
    if do == "trees_refit":
        return _boost(case, seed)
    return None
