"""Performance cases of the auto-tuner: the calls a tuning session makes, over their ranges.

A session (Falch & Elster, Sections 5 and 6) samples training configurations, trains a bagged
ensemble on their measured times, sweeps the whole space with it and keeps the candidates with
the lowest predictions; it checks the model on held-out configurations and, for spaces too large
for one call, streams the sweep chunk by chunk.  Every case goes through `api.Sweep` and
`api.Tuner`, as a tuning program does.

A case is a dict of plain values:
  call      topk | all | stream | indices | train | sample
  radices   lengths of the parameters' value lists, "8x8x2"; 4 and 8 are powers of two and 16 is
            1..16 (both enter the networks as logarithms), 2 is a flag, any other r is 1..r
  rule      validity rules: none | group (work-group size, the first two parameters) |
            group+order (also third <= fourth) | product (three rules over the first ten)
  members, hidden ("30", "64x64"), precision (fp32 | bf16), algo (auto | split16 | valu)
  begin, count  range of configurations; k  candidates kept; prepared  weights packed once
  grouped   the candidates' indices in ascending order, in which a program measures them when
            neighbours share compiled kernels (spaces of a million and more, two-layer networks:
            their best predictions lie so close that fp32 rounding decides the order of some)
  mask      predict_all also writes the validity bytes; chunks  calls of a streamed sweep
  n         list length (indices), samples (train, sample); epochs
"""
import math

import numpy as np
import torch

from paper_1506_00842_amd import (TUNER_ALGO_AUTO, TUNER_ALGO_SPLIT16, TUNER_ALGO_VALU,
                                  TUNER_BF16_MFMA, TUNER_FP32)
from paper_1506_00842_amd.api import Sweep, Tuner

DEVICE = "cuda:0"
LARGE = "8x8x8x8x4x4x4x4x4x2x2x2x2x2"                       # 2**27 configurations
STREAMED = "16x16x16x4x4x4x" + "x".join(["2"] * 14)         # 2**32 configurations


def _sweep_case(call, radices, rule, members, hidden, **more):
    case = {"call": call, "radices": radices, "rule": rule, "members": members, "hidden": hidden,
            "precision": "fp32", "algo": "auto", "begin": 0, "count": _size(radices), "k": 0,
            "prepared": False, "grouped": False, "mask": False, "chunks": 1, "n": 0, "epochs": 0}
    case.update(more)
    return case


def listed():
    return [
        # a first try-out of the tuner on a handful of parameters: nothing but call latency
        {"name": "tiny_topk", **_sweep_case("topk", "4x4x2x8", "none", 1, "16", k=10)},
        # second stage of the tuner on the convolution space, one call per trained model
        {"name": "convolution_topk",
         **_sweep_case("topk", "8x8x8x8x2x2x2x2x2", "group", 11, "30", k=200)},
        # raycasting space (a list of five values), swept again and again with one model
        {"name": "raycasting_topk",
         **_sweep_case("topk", "8x8x8x8x2x2x2x2x2x5", "group", 11, "30", k=300, prepared=True)},
        # every prediction of the stereo space (lists of three), to study the model
        {"name": "stereo_all",
         **_sweep_case("all", "8x8x8x8x2x2x2x2x4x3x3", "group", 11, "30", mask=True)},
        # part of a space with odd list lengths, odd layer widths, a range that starts anywhere
        {"name": "ragged_topk",
         **_sweep_case("topk", "7x6x8x5x3x5x4x3x3x2", "group+order", 5, "48x24", begin=12_345,
                       count=1_500_001, k=77, grouped=True)},
        # the large space in one call: the headline sweep
        {"name": "large_topk", **_sweep_case("topk", LARGE, "group+order", 4, "64x64", k=1000, grouped=True)},
        # a part of the large space written out by a wide ensemble, from an odd position on
        {"name": "wide_all",
         **_sweep_case("all", LARGE, "group+order", 16, "128x128", begin=40_000_001, count=1 << 23)},
        # the wide ensemble over the whole space where 1e-2 is enough
        {"name": "wide_bf16_all",
         **_sweep_case("all", LARGE, "group+order", 16, "128x128", precision="bf16", prepared=True)},
        # a space too large for one call: chunks with a running result
        {"name": "streamed_topk",
         **_sweep_case("stream", STREAMED, "product", 8, "64x64", begin=3 << 27, count=3 << 26,
                       chunks=3, k=1000, prepared=True, grouped=True)},
        # accuracy of a model on held-out configurations of the stereo space
        {"name": "heldout_indices",
         **_sweep_case("indices", "8x8x8x8x2x2x2x2x4x3x3", "group", 11, "30", n=100_003, mask=True)},
        # training of the ensemble on the convolution space's samples
        {"name": "convolution_train",
         **_sweep_case("train", "8x8x8x8x2x2x2x2x2", "group", 11, "30", n=2000, epochs=1000)},
        # choice of the training configurations
        {"name": "stereo_sample",
         **_sweep_case("sample", "8x8x8x8x2x2x2x2x4x3x3", "group", 1, "1", n=3000)},
    ]


def draw(rng):
    """A case of the ranges above: the paper's kind of space (four lists, then flags and short
    lists), 256 to 2**27 configurations, ensembles of 1 to 16 networks with one hidden layer of 8 to
    64 or two of 8 to 128 units, 1 to 500 candidates."""
    call = rng.choice(["topk"] * 4 + ["all"] * 3 + ["stream", "indices", "indices", "train", "sample"])
    while True:
        target = 2.0 ** rng.uniform(8, 27)
        radices = [rng.choice([8, 8, 7, 6, 5, 4]) for _ in range(4)]
        n = math.prod(radices)
        while n < target and len(radices) < 20:
            radices.append(rng.choice([2, 2, 2, 2, 3, 4, 5]))
            n *= radices[-1]
        while n > target and len(radices) > 3:
            n //= radices.pop(0)
        if n > 1 << 27 or n < 256:
            continue
        if rng.random() < 0.6:
            radices.sort(reverse=True)          # long lists first, flags last: the usual order
        text = "x".join(map(str, radices))
        rule = rng.choice(["none", "group", "group", "group+order"])
        two = rng.random() < 0.5
        hidden = "%dx%d" % (rng.randint(8, 128), rng.randint(8, 128)) if two else str(rng.randint(8, 64))
        case = _sweep_case(call, text, rule, rng.randint(1, 16), hidden)
        if call in ("topk", "all", "stream"):
            case["begin"] = rng.randrange(n // 4) if rng.random() < 0.5 else 0
            case["count"] = n - case["begin"] - (rng.randrange(n // 8) if rng.random() < 0.5 else 0)
            # (the order of candidates is only comparable at full precision)
            case["precision"] = rng.choice(["fp32", "fp32", "bf16"]) if call == "all" else "fp32"
            case["algo"] = rng.choice(["auto"] * 6 + ["split16", "valu"]) if case["precision"] == "fp32" else "auto"
            case["prepared"] = rng.random() < 0.5
        if call in ("topk", "stream"):
            # a few candidates, or the paper's 200 and more; a small share of the space (at most
            # 1.7 % there)
            few, many = int(2.0 ** rng.uniform(0, 5.3)), rng.randint(200, 500)
            case["grouped"] = case["count"] >= 1 << 20 or two
            case["k"] = many if case["count"] // 128 > many and rng.random() < 0.6 else max(1, min(few, case["count"] // 64))
        if call == "stream":
            case["chunks"] = rng.randint(2, 5)
        if call == "all":
            case["mask"] = rng.random() < 0.5
        if call == "indices":
            case["n"], case["mask"] = int(2.0 ** rng.uniform(9, 20)), True
        if call == "train":
            case["hidden"] = str(rng.randint(8, 64))
            case["members"] = rng.randint(2, 16)
            case["n"], case["epochs"] = int(2.0 ** rng.uniform(8, 12)), rng.randint(100, 1000)
        if call == "sample":
            case["n"] = max(1, min(int(2.0 ** rng.uniform(6, 12)), n // 64))
        if call == "train" and n < 4 * case["n"]:
            continue
        if work(case)["flops"] > 2e12 * (0.2 if case["algo"] == "valu" else 1.0):
            continue
        return case


# ---- the space and the inputs -----------------------------------------------------------------

def _radices(text):
    return [int(r) for r in text.split("x")]


def _size(text):
    return math.prod(_radices(text))


def _hidden(case):
    return [int(h) for h in case["hidden"].split("x")]


class _Space:
    """Value lists, scales and rules in the form api.Sweep and api.Tuner take."""

    def __init__(self, text, rule):
        self.radices = np.array(_radices(text), np.int32)
        lists, scales = [], []
        for r in self.radices:
            if r in (4, 8):
                lists.append([float(1 << j) for j in range(r)]); scales.append(1)
            elif r == 16:
                lists.append([float(j + 1) for j in range(r)]); scales.append(1)
            elif r == 2:
                lists.append([0.0, 1.0]); scales.append(0)
            else:
                lists.append([float(j + 1) for j in range(r)]); scales.append(0)
        self.lists, self.scales = lists, scales
        self.flat_values = np.array([v for l in lists for v in l], np.float64)
        rules, bounds = [], []
        r = [int(x) for x in self.radices]
        if "group" in rule:
            rules.append({0: range(r[0]), 1: range(r[1])})
            bounds.append(math.ceil(0.7 * (r[0] + r[1] - 2)))
        if "order" in rule and len(r) > 3:
            rules.append({2: range(r[2]), 3: [-j for j in range(r[3])]})
            bounds.append(0)
        if rule == "product":
            rules.append({p: [round((1 << 20) * math.log2(v)) for v in lists[p]] for p in (0, 1, 2)})
            rules.append({p: range(r[p]) for p in (3, 4, 5)})
            rules.append({p: range(r[p]) for p in (6, 7, 8, 9)})
            bounds += [10 << 20, 7, 3]
        self.rules = rules
        self.constraint_terms = np.zeros((len(rules), int(self.radices.sum())), np.int32)
        first = np.concatenate([[0], np.cumsum(self.radices)[:-1]])
        for c, terms in enumerate(rules):
            for p, t in terms.items():
                self.constraint_terms[c, first[p]:first[p] + r[p]] = list(t)
        self.constraint_bounds = np.array(bounds, np.int64)

    def valid_share(self):
        """Share of the space's configurations that satisfy the rules (each parameter is in one)."""
        share = 1.0
        for terms, bound in zip(self.rules, self.constraint_bounds):
            sums = np.zeros(1, np.int64)
            for t in terms.values():
                sums = (sums[:, None] + np.array(list(t), np.int64)[None, :]).ravel()
            share *= float(np.mean(sums <= bound))
        return share

    def features(self):
        """Per parameter the min-max normalised list, rounded once to fp32."""
        out = []
        for v, s in zip(self.lists, self.scales):
            x = np.log2(np.array(v)) if s else np.array(v)
            span = x.max() - x.min()
            out.append(((x - x.min()) / span if span else x * 0).astype(np.float32))
        return out

    def digits(self, index):
        """Digits of int64 configuration indices, last parameter fastest."""
        out = [None] * len(self.radices)
        for p in range(len(self.radices) - 1, -1, -1):
            out[p] = index % int(self.radices[p])
            index = torch.div(index, int(self.radices[p]), rounding_mode="floor")
        return out

    def valid(self, digits):
        ok = torch.ones_like(digits[0], dtype=torch.bool)
        for terms, bound in zip(self.rules, self.constraint_bounds):
            total = torch.zeros_like(digits[0])
            for p, t in terms.items():
                total += torch.tensor(list(t), dtype=torch.int64, device=digits[p].device)[digits[p]]
            ok &= total <= int(bound)
        return ok


class _Model:
    def __init__(self, n_members, widths, weights):
        self.n_members, self.widths, self.weights = n_members, widths, weights


def _widths(case):
    return [len(_radices(case["radices"]))] + _hidden(case) + [1]


def _start_weights(case, rng):
    """Where training starts: W ~ N(0, 1 / fan_in), b ~ U(-0.1, 0.1), member by member."""
    w, parts = _widths(case), []
    for _ in range(case["members"]):
        for a, b in zip(w[:-1], w[1:]):
            parts.append(rng.standard_normal(a * b) / math.sqrt(a))
            parts.append(rng.uniform(-0.1, 0.1, b))
    return np.concatenate(parts).astype(np.float32)


def _trained_weights(case, rng):
    """An ensemble as training leaves it.  Ensembles of 11 networks with 30 units trained for 1000
    epochs have input weights 1.5 times, biases 7 times and output weights 4.3 to 5.4 times as large
    as at the start; the members, trained on nearly the same samples, resemble one another and
    predict log-times about a common mean (here -2)."""
    w = _widths(case)
    grow = [1.5] + [1.5] * (len(w) - 3) + [4.5]
    shared = [rng.standard_normal(a * b) for a, b in zip(w[:-1], w[1:])]
    parts = []
    for _ in range(case["members"]):
        for g, base, a, b in zip(grow, shared, w[:-1], w[1:]):
            parts.append(g * (0.9 * base + 0.436 * rng.standard_normal(a * b)) / math.sqrt(a))
            parts.append(rng.uniform(-0.7, 0.7, b))
        parts[-1] += -2.0 - 0.5 * parts[-2].sum()
    return np.concatenate(parts).astype(np.float32)


def _indices(case, space, rng, only_valid):
    """case["n"] distinct-enough configuration indices, as int64 numpy."""
    size, n = _size(case["radices"]), case["n"]
    found = np.zeros(0, np.int64)
    while len(found) < n:
        i = torch.from_numpy(rng.integers(0, size, 4 * n))
        if only_valid:
            i = i[space.valid(space.digits(i))]
        found = np.concatenate([found, i.numpy()])
    return found[:n]


def _times(case, space, index, rng):
    """Measured times: a smooth surface of the parameters, 3 % noise, 3 % failed runs (-1)."""
    x = np.stack([f[d.numpy()] for f, d in zip(space.features(), space.digits(torch.from_numpy(index)))], 1)
    best, curve = rng.uniform(0.2, 0.8, x.shape[1]), rng.uniform(0.3, 2.0, x.shape[1])
    log_t = -3.0 + ((x - best) ** 2) @ curve + 0.5 * np.sin(3.0 * x[:, 0] + 2.0 * x[:, 1])
    t = np.exp(log_t + 0.03 * rng.standard_normal(len(index)))
    t[rng.random(len(index)) < 0.03] = -1.0
    return t.astype(np.float32)


def _inputs(case, seed):
    """Host inputs of a case, from the seed alone."""
    rng = np.random.default_rng([seed & 0xFFFFFFFF, 1506])
    space = _Space(case["radices"], case["rule"])
    inp = {"space": space, "weights": (_start_weights if case["call"] == "train" else _trained_weights)(case, rng)}
    if case["call"] == "indices":
        inp["index"] = _indices(case, space, rng, only_valid=False)
        inp["times"] = _times(case, space, inp["index"], rng)
    if case["call"] == "train":
        inp["index"] = _indices(case, space, rng, only_valid=True)
        inp["times"] = _times(case, space, inp["index"], rng)
        inp["parts"] = (np.arange(case["n"]) % case["members"]).astype(np.int32)
    if case["call"] == "sample":
        inp["draw_seed"] = int(rng.integers(0, 1 << 62))
    return inp


def _u32(index):
    return torch.from_numpy(index.astype(np.uint32).view(np.int32)).to(DEVICE)


# ---- what a tuning program holds, and what it calls -------------------------------------------

def prepare(case, seed):
    inp = _inputs(case, seed)
    state = {"case": case, "space": inp["space"]}
    if case["call"] in ("train", "sample"):
        state["tuner"] = Tuner(inp["space"], DEVICE)
        if case["call"] == "train":
            state["index"], state["times"] = _u32(inp["index"]), torch.from_numpy(inp["times"]).to(DEVICE)
            state["parts"] = torch.from_numpy(inp["parts"]).to(DEVICE)
            state["weights"] = torch.from_numpy(inp["weights"]).to(DEVICE)
        else:
            state["draw_seed"] = inp["draw_seed"]
        return state
    model = _Model(case["members"], _widths(case), inp["weights"])
    algo = {"auto": TUNER_ALGO_AUTO, "split16": TUNER_ALGO_SPLIT16, "valu": TUNER_ALGO_VALU}[case["algo"]]
    sweep = Sweep(inp["space"], model, case["k"], DEVICE,
                  TUNER_BF16_MFMA if case["precision"] == "bf16" else TUNER_FP32, algo)
    if case["prepared"]:
        sweep.prepare()
    state["sweep"] = sweep
    if case["call"] == "all":
        state["out"] = torch.empty(case["count"], dtype=torch.float32, device=DEVICE)
        state["mask"] = torch.empty(case["count"], dtype=torch.uint8, device=DEVICE) if case["mask"] else None
    if case["call"] == "indices":
        state["tuner"] = Tuner(inp["space"], DEVICE)
        state["index"], state["times"] = _u32(inp["index"]), torch.from_numpy(inp["times"]).to(DEVICE)
    return state


def _chunks(case):
    """(begin, count) of the calls of a streamed sweep."""
    step = -(-case["count"] // case["chunks"])
    end = case["begin"] + case["count"]
    return [(b, min(step, end - b)) for b in range(case["begin"], end, step)]


def _candidates(sweep, grouped):
    if not grouped:
        return sweep.values, sweep.indices, sweep.n_found
    return sweep.values, (sweep.indices.long() & 0xFFFFFFFF).sort().values, sweep.n_found


def run(state):
    case, call = state["case"], state["case"]["call"]
    if call == "topk":
        sweep = state["sweep"]
        sweep.topk(case["begin"], case["count"])
        return _candidates(sweep, case["grouped"])
    if call == "stream":
        sweep = state["sweep"]
        for i, (begin, count) in enumerate(_chunks(case)):
            sweep.topk(begin, count, merge=i > 0)
        return _candidates(sweep, case["grouped"])
    if call == "all":
        out, mask = state["sweep"].predict_all(case["begin"], case["count"], case["mask"],
                                               state["out"], state["mask"])
        return (out, mask) if case["mask"] else (out,)
    if call == "indices":
        pred, mask = state["sweep"].predict_indices(state["index"], case["mask"])
        error, used = state["tuner"].mean_relative_error(pred, state["times"])
        return pred, mask, error, used
    if call == "train":
        return state["tuner"].train(case["members"], _hidden(case)[0], state["index"], state["times"],
                                    state["parts"], state["weights"], case["epochs"], 0.125, 0.875)
    return state["tuner"].sample_valid(state["draw_seed"], case["n"], 64 * case["n"])


def work(case):
    """One pass: every valid configuration through every network (2 flop a multiply-add), weights
    and lists read once, outputs written once.  Training: forward and backward pass a sample
    (4 P H + 9 H, as counted for one hidden layer) and epoch for every network but the one it is
    left out of.  Sampling: about twenty integer operations a draw."""
    widths, call = _widths(case), case["call"]
    macs = case["members"] * sum(a * b for a, b in zip(widths[:-1], widths[1:]))
    weights = 4 * case["members"] * sum(a * b + b for a, b in zip(widths[:-1], widths[1:]))
    if call == "train":
        p, h = widths[0], widths[1]
        return {"bytes": 2 * weights + 12 * case["n"] + 4 * case["members"] * (case["epochs"] + 1),
                "flops": float(case["epochs"]) * case["n"] * (case["members"] - 1) * (4 * p * h + 9 * h)}
    if call == "sample":
        return {"bytes": 4 * case["n"], "flops": 20.0 * 64 * case["n"]}
    n = case["n"] if call == "indices" else case["count"]
    flops = 2.0 * macs * n * _Space(case["radices"], case["rule"]).valid_share()
    out = 8 * case["k"] + 4
    if call == "all":
        out = n * (5 if case["mask"] else 4)
    if call == "indices":
        out = n * (4 + 4 + 1 + 4)                 # indices and times in, predictions and mask out
    return {"bytes": weights + out, "flops": flops}


def tolerance(case):
    """About four times what the paths show against 64 bits.  fp32: 0.5e-7 to 4e-7 of the
    predictions' norm, single ones 2e-6, with the order of near-equal candidates decided by such
    differences.  bf16: 2e-4 to 3e-3, the more the fewer members.  Training: 1.2e-6, single weights 8e-6,
    after 1000 epochs."""
    if case["call"] == "sample":
        return "exact"
    if case["call"] == "train":
        return {"rel": 5e-6, "max": 5e-5}
    if case["precision"] == "bf16":
        return {"rel": 1e-2, "max": 4e-2}
    return {"rel": 2e-6, "max": 1e-5, "differ": 0.01}


# ---- the same in 64 bits ----------------------------------------------------------------------

def _layers(case, weights):
    """Per member [(W, b), ...] in float64 on the GPU."""
    w, at, out = _widths(case), 0, []
    flat = torch.from_numpy(weights).to(DEVICE).double()
    for _ in range(case["members"]):
        member = []
        for a, b in zip(w[:-1], w[1:]):
            member.append((flat[at:at + a * b].view(b, a), flat[at + a * b:at + a * b + b]))
            at += a * b + b
        out.append(member)
    return out


def _predict(case, space, layers, index):
    """(predictions, +inf where invalid; validity) in float64 at int64 indices on the GPU."""
    digits = space.digits(index)
    ok = space.valid(digits)
    rows = ok.nonzero().squeeze(1)
    tables = [torch.from_numpy(f).to(DEVICE).double() for f in space.features()]
    x = torch.stack([t[d[rows]] for t, d in zip(tables, digits)], 1)
    total = torch.zeros(len(rows), dtype=torch.float64, device=DEVICE)
    for member in layers:
        a = x
        for w, b in member[:-1]:
            a = torch.sigmoid(torch.addmm(b, a, w.t()))
        w, b = member[-1]
        total += torch.addmm(b, a, w.t()).squeeze(1)
    out = torch.full((len(index),), math.inf, dtype=torch.float64, device=DEVICE)
    out[rows] = total / case["members"]
    return out, ok


def _in_blocks(case, space, layers, begin, count):
    step = 1 << 20
    for b in range(begin, begin + count, step):
        index = torch.arange(b, min(b + step, begin + count), device=DEVICE)
        yield index, _predict(case, space, layers, index)


def _train64(case, inp):
    """Full-batch gradient descent with momentum, all networks side by side in float64."""
    space, e, h, p = inp["space"], case["members"], _hidden(case)[0], len(_radices(case["radices"]))
    digits = space.digits(torch.from_numpy(inp["index"]))
    x = torch.stack([torch.from_numpy(f).double()[d] for f, d in zip(space.features(), digits)], 1).to(DEVICE)
    t = torch.from_numpy(inp["times"]).to(DEVICE).double()
    use = (t > 0)[None, :] & (torch.from_numpy(inp["parts"]).to(DEVICE)[None, :] != torch.arange(e, device=DEVICE)[:, None])
    use = use.double()
    n_e = use.sum(1)
    target = torch.where(t > 0, t, torch.ones_like(t)).log()
    layers = _layers(case, inp["weights"])
    w1, b1 = torch.stack([m[0][0] for m in layers]), torch.stack([m[0][1] for m in layers])
    wo, bo = torch.stack([m[1][0][0] for m in layers]), torch.stack([m[1][1] for m in layers])
    params = [w1.clone(), b1.clone(), wo.clone(), bo.clone()]
    moves = [torch.zeros_like(q) for q in params]
    loss = torch.zeros(e, case["epochs"] + 1, dtype=torch.float64, device=DEVICE)
    for epoch in range(case["epochs"] + 1):
        w1, b1, wo, bo = params
        hid = torch.sigmoid(torch.matmul(w1.reshape(e * h, p), x.t()).view(e, h, -1) + b1[:, :, None])
        err = ((wo[:, :, None] * hid).sum(1) + bo - target[None, :]) * use
        loss[:, epoch] = (err * err).sum(1) / n_e
        if epoch == case["epochs"]:
            break
        dz = err[:, None, :] * wo[:, :, None] * hid * (1 - hid)
        grads = [torch.matmul(dz.view(e * h, -1), x).view(e, h, p), dz.sum(2),
                 (err[:, None, :] * hid).sum(2), err.sum(1, keepdim=True)]
        for q, v, g in zip(params, moves, grads):
            v.mul_(0.875).sub_(0.125 * 2 * g / n_e.view([e] + [1] * (g.dim() - 1)))
            q.add_(v)
    return torch.cat([q.reshape(e, -1) for q in params], 1).reshape(-1), loss


def exact(case, seed):
    """What run() returns, in float64; None for whole numbers, whose order near-ties decide."""
    if case["call"] == "sample":
        return None
    # about 20 s of float64 work on the GPU
    if work(case)["flops"] > 5e13:
        return None
    inp = _inputs(case, seed)
    space = inp["space"]
    if case["call"] == "train":
        return _train64(case, inp)
    layers = _layers(case, inp["weights"])
    if case["call"] == "indices":
        index = torch.from_numpy(inp["index"]).to(DEVICE)
        pred, ok = _predict(case, space, layers, index)
        t = torch.from_numpy(inp["times"]).to(DEVICE).double()
        used = ok & (t > 0)
        error = ((pred[used].exp() - t[used]).abs() / t[used]).mean().reshape(1)
        return pred, None, error, None
    if case["call"] == "all":
        out = torch.cat([p for _, (p, _) in _in_blocks(case, space, layers, case["begin"], case["count"])])
        return (out, None) if case["mask"] else (out,)
    best = torch.zeros(0, dtype=torch.float64, device=DEVICE)
    for _, (p, _) in _in_blocks(case, space, layers, case["begin"], case["count"]):
        both = torch.cat([best, p])
        best = torch.topk(both, min(case["k"], len(both)), largest=False, sorted=True).values
    values = torch.full((case["k"],), math.inf, dtype=torch.float64, device=DEVICE)
    values[:len(best)] = best
    return values, None, None
