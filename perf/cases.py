"""Workloads of the parameter-server aggregation path, for timing on a GPU.

Every case is one call (or the two calls that belong together) a parameter server makes per
training step on gradients that already sit in HBM: the whole path (majority vote, then median or
trimmed mean of the winners), the vote for honest copies that agree only up to rounding, and the
aggregators that can take the median's place on f gradient vectors.  Shapes are the clusters of
synth/configs.py (MOLS and Ramanujan-bigraph assignments), gradient lengths run from a small
layer to ResNet-50, with rows padded to 64 words as bench.py lays them out and with odd pitches.

    listed()  draw(rng)  prepare(case, seed)  run(state)  work(case)  tolerance(case)
    exact(case, seed)
"""
import math

import torch

import paper_2010_04902_amd as B

DEV = "cuda:0"
RESNET18, RESNET50 = 11173962, 25557032

# (scheme, a, b, q): the clusters of synth/configs.py with the Byzantine workers they are run with
CLUSTERS = {
    "mols5x3": (B.BYZ_SCHEME_MOLS, 5, 3, 4),          # f =  25, r = 3
    "mols7x3": (B.BYZ_SCHEME_MOLS, 7, 3, 5),          # f =  49, r = 3
    "mols7x5": (B.BYZ_SCHEME_MOLS, 7, 5, 5),          # f =  49, r = 5
    "mols9x3": (B.BYZ_SCHEME_MOLS, 9, 3, 4),          # f =  81, r = 3
    "mols11x3": (B.BYZ_SCHEME_MOLS, 11, 3, 3),        # f = 121, r = 3
    "mols13x3": (B.BYZ_SCHEME_MOLS, 13, 3, 3),        # f = 169, r = 3
    "ram5x5": (B.BYZ_SCHEME_RAMANUJAN, 5, 5, 5),      # f =  25, r = 5
    "ram5x7": (B.BYZ_SCHEME_RAMANUJAN, 5, 7, 5),      # f =  35, r = 5
    "ram7x7": (B.BYZ_SCHEME_RAMANUJAN, 7, 7, 4),      # f =  49, r = 7
    "ram7x9": (B.BYZ_SCHEME_RAMANUJAN, 7, 9, 4),      # f =  63, r = 7
    "ram5x13": (B.BYZ_SCHEME_RAMANUJAN, 5, 13, 5),    # f =  65, r = 5
    "ram3x85": (B.BYZ_SCHEME_RAMANUJAN, 3, 85, 2),    # f = 255, r = 3 (no single pass)
}
SHAPES = {"mols5x3": (25, 3), "mols7x3": (49, 3), "mols7x5": (49, 5), "mols9x3": (81, 3),
          "mols11x3": (121, 3), "mols13x3": (169, 3), "ram5x5": (25, 5), "ram5x7": (35, 5),
          "ram7x7": (49, 7), "ram7x9": (63, 7), "ram5x13": (65, 5), "ram3x85": (255, 3)}


def padded(d):
    return (d + 63) // 64 * 64


def listed():
    return [
        # the smallest model a server aggregates (a linear layer); launches and latency count
        {"name": "aggregate_mols5x3_1k", "op": "aggregate", "cluster": "mols5x3", "agg": "median",
         "early": False, "attack": "alie", "d": 1003, "ld": 1003},
        # a small network, the size the package's smoke run uses
        {"name": "aggregate_mols5x3_100k", "op": "aggregate", "cluster": "mols5x3", "agg": "median",
         "early": False, "attack": "alie", "d": 100003, "ld": padded(100003)},
        # workload 1 of synth/configs.py: one million coordinates, reversed gradients
        {"name": "aggregate_mols5x3_1m", "op": "aggregate", "cluster": "mols5x3", "agg": "median",
         "early": False, "attack": "reversed", "d": 1 << 20, "ld": 1 << 20},
        # workload 2, bench.py's headline: ResNet-18 gradients, ALIE
        {"name": "aggregate_mols5x3_resnet18", "op": "aggregate", "cluster": "mols5x3",
         "agg": "median", "early": False, "attack": "alie", "d": RESNET18, "ld": padded(RESNET18)},
        # workload 5, the largest: ResNet-50 gradients on 21 workers, 15 GB of returns
        {"name": "aggregate_mols7x3_resnet50", "op": "aggregate", "cluster": "mols7x3",
         "agg": "median", "early": False, "attack": "alie", "d": RESNET50, "ld": padded(RESNET50)},
        # trimmed mean of the winners behind five-fold replication, odd row pitch
        {"name": "aggregate_trim_ram5x5_2m", "op": "aggregate", "cluster": "ram5x5", "agg": "trim",
         "b": 4, "early": False, "attack": "constant", "d": 2000003, "ld": 2000003},
        # workload 14's cluster: the widest file count, vote and median one after the other
        {"name": "aggregate_ram3x85_1m", "op": "aggregate", "cluster": "ram3x85", "agg": "median",
         "early": False, "attack": "alie", "d": 1 << 20, "ld": 1 << 20},
        # honest copies that agree up to rounding: tolerant vote, then the median of its winners
        {"name": "tolerant_vote_median_mols7x5_1m", "op": "tolerant", "cluster": "mols7x5",
         "attack": "alie", "d": 1000001, "ld": padded(1000001)},
        # median over the winners' rows of a wide cluster (MOLS over F_13), vote done elsewhere
        {"name": "median_169_4m", "op": "median", "f": 169, "d": 4000000, "ld": 4000000},
        # trimmed mean over 81 gradient vectors of ResNet-18
        {"name": "trimmed_mean_81_resnet18", "op": "trimmed_mean", "f": 81, "b": 8, "d": RESNET18,
         "ld": padded(RESNET18)},
        # Multi-Krum over 25 gradient vectors of ResNet-18
        {"name": "multi_krum_25_resnet18", "op": "multi_krum", "f": 25, "c": 5, "m": 20,
         "d": RESNET18, "ld": padded(RESNET18)},
        # Bulyan over 49 gradient vectors of ResNet-18
        {"name": "bulyan_49_resnet18", "op": "bulyan", "f": 49, "c": 8, "d": RESNET18,
         "ld": padded(RESNET18)},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["aggregate"] * 6 + ["tolerant", "median", "trimmed_mean", "multi_krum",
                                         "bulyan", "mean_around_median"])
    case = {"op": op}
    if op in ("aggregate", "tolerant"):
        cluster = rng.choice(sorted(CLUSTERS))
        f, r = SHAPES[cluster]
        rows = f * r
        case.update(cluster=cluster, attack=rng.choice(["alie", "reversed", "constant"]))
        if op == "aggregate":
            case["agg"] = rng.choice(["median", "median", "trim"])
            if case["agg"] == "trim":
                case["b"] = rng.randint(1, (f - 1) // 3)
            case["early"] = rng.random() < 0.2
            if rng.random() < 0.15:
                case["attack"] = "split"
        budget = (6 << 30) if op == "aggregate" else (2 << 30)
    else:
        if op == "median":
            f = 2 * rng.randint(4, 127) + 1
        elif op == "trimmed_mean":
            f = rng.randint(9, 256)
            case["b"] = rng.randint(1, (f - 1) // 3)
        elif op == "multi_krum":
            f = rng.randint(9, 128)
            case["c"] = rng.randint(1, (f - 3) // 2)
            case["m"] = rng.randint(1, f - case["c"])
        else:
            f = 2 * rng.randint(5, 63) + 1
            if op == "bulyan":
                case["c"] = rng.randint(1, (f - 3) // 4)
            else:
                case["beta"] = rng.randint(1, f)
        case["f"] = f
        rows = f
        budget = 2 << 30
    d = _log_uniform(rng, 1000, min(RESNET50, budget // (4 * rows)))
    case["d"] = d
    case["ld"] = rng.choice([d, padded(d)])
    return case


# ---------------------------------------------------------------------------- inputs


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _honest(f, d, ld, gen):
    """[f, ld] gradients of f files: N(0, 0.01^2) with a scale of its own, U(0.5, 2), per file, on
    a common signal (the files' gradients point the same way), as mini-batch gradients have."""
    G = torch.empty((f, ld), dtype=torch.float32, device=DEV)
    signal = torch.randn(ld, generator=gen, device=DEV) * 0.002
    scale = (torch.rand(f, generator=gen, device=DEV) * 1.5 + 0.5) * 0.01
    for j in range(f):
        G[j].normal_(generator=gen)
        G[j].mul_(scale[j]).add_(signal)
    return G


def _attacked(G, d, attack):
    """The vector(s) Byzantine workers send: -> function of the file."""
    if attack in ("alie", "split"):
        std, mean = torch.std_mean(G, dim=0, correction=0)
        v = mean - 1.0 * std
        return lambda j: v
    if attack == "reversed":
        return lambda j: G[j] * -100.0
    return lambda j: torch.full_like(G[j], 1e3)


def _copies(case, seed):
    """(stacked returns [K*l, ld], file -> rows table [f, r], r)."""
    scheme, a, b, q = CLUSTERS[case["cluster"]]
    asg = B.byz_build_assignment(scheme, a, b)
    byz = set(B.byz_worst_case(asg, q)[0])
    gen = _generator(seed)
    d, ld = case["d"], case["ld"]
    G = _honest(asg.f, d, ld, gen)
    sent = _attacked(G, d, case["attack"])
    files = asg.worker_files()
    X = torch.empty((asg.K * asg.l, ld), dtype=torch.float32, device=DEV)
    for w in range(asg.K):
        for t in range(asg.l):
            j = int(files[w, t])
            row = X[w * asg.l + t]
            if w in byz:
                row.copy_(sent(j))
                if case["attack"] == "split":  # false copies of a file told apart by one word
                    row[(37 * w + t) % d] += 1.0
            else:
                row.copy_(G[j])
                if case["op"] == "tolerant" and t % 2:  # another order of summation: one rounding
                    row.mul_(1.0 + 2.0 ** -23)
    del G
    return X, asg.file_rows(), asg.r


def _rows(case, seed):
    """(f gradient vectors [f, ld]): honest ones and, from the end, a tenth that are reversed."""
    gen = _generator(seed)
    f = case["f"]
    G = _honest(f, case["d"], case["ld"], gen)
    for j in range(f - f // 10, f):
        G[j].mul_(-3.0)
    return G


def prepare(case, seed):
    op, d = case["op"], case["d"]
    out = torch.empty(d, dtype=torch.float32, device=DEV)
    if op in ("aggregate", "tolerant"):
        X, rows, r = _copies(case, seed)
        f = rows.shape[0]
        state = dict(case, X=X, f=f, r=r, out=out,
                     rows=torch.tensor(rows.reshape(-1), dtype=torch.int32, device=DEV))
        if op == "aggregate":
            state["winner"] = torch.empty(f, dtype=torch.int32, device=DEV)
            state["ws"] = torch.empty(B.byz_aggregate_workspace_bytes(f, r), dtype=torch.uint8,
                                      device=DEV)
            flags = B.BYZ_AGG_TRIM(case["b"]) if case["agg"] == "trim" else 0
            state["flags"] = flags | (B.BYZ_AGG_EARLY_MAJORITY if case["early"] else 0)
        return state
    f = case["f"]
    state = dict(case, X=_rows(case, seed), out=out,
                 index=torch.arange(f, dtype=torch.int32, device=DEV))
    if op == "multi_krum":
        state["ws"] = torch.empty(B.byz_multi_krum_workspace_bytes(f), dtype=torch.uint8, device=DEV)
    elif op == "bulyan":
        state["ws"] = torch.empty(B.byz_bulyan_workspace_bytes(f), dtype=torch.uint8, device=DEV)
    return state


def run(s):
    op, d, X = s["op"], s["d"], s["X"]
    if op == "aggregate":
        out, winner, _ = B.byz_aggregate_opts(X, d, s["rows"], s["f"], s["r"], s["flags"],
                                              out=s["out"], winner_replica=s["winner"],
                                              workspace=s["ws"])
        return out, winner
    if op == "tolerant":
        replica, row, far = B.byz_vote_tolerant(X, d, s["rows"], s["f"], s["r"], ATOL, RTOL)
        return B.byz_median(X, d, row, out=s["out"]), replica, row, far
    if op == "median":
        return B.byz_median(X, d, s["index"], out=s["out"])
    if op == "trimmed_mean":
        return B.byz_trimmed_mean(X, d, s["index"], s["b"], out=s["out"])
    if op == "mean_around_median":
        return B.byz_mean_around_median(X, d, s["index"], s["beta"], out=s["out"])
    if op == "multi_krum":
        return B.byz_multi_krum(X, d, s["index"], s["c"], s["m"], out=s["out"], workspace=s["ws"])
    return B.byz_bulyan(X, d, s["index"], s["c"], out=s["out"], workspace=s["ws"])


ATOL, RTOL = 1e-6, 1e-5  # tolerant vote: what one rounding more or less can do, with room


def work(case):
    op, d = case["op"], case["d"]
    if op in ("aggregate", "tolerant"):
        f, r = SHAPES[case["cluster"]]
        return {"bytes": 4.0 * (f * r + 1) * d, "flops": 0.0}
    f = case["f"]
    if op == "multi_krum" or op == "bulyan":
        return {"bytes": 4.0 * (f + 1) * d, "flops": float(f * (f + 1)) * d}
    return {"bytes": 4.0 * (f + 1) * d, "flops": 0.0}


def tolerance(case):
    op = case["op"]
    if op in ("median", "tolerant") or (op == "aggregate" and case["agg"] == "median"):
        return "exact"  # selection: the result is one of the inputs
    # sums of up to 256 fp32 values and Gram entries summed in fp32 slices: up to 6e-7 (rel) and
    # 2.4e-6 (max) away from the 64-bit results over the drawn ranges
    return {"rel": 3e-6, "max": 1.2e-5}


# ---------------------------------------------------------------------- 64-bit results


def _winners(X, rows, d, close):
    """Per file: copy with the most equal (close) copies, lowest replica first; -> (replica, row,
    mask of unequal pairs)."""
    f, r = rows.shape
    replica, row, masks = [], [], []
    for j in range(f):
        c = [X[int(rows[j, k]), :d] for k in range(r)]
        like = [[True] * r for _ in range(r)]
        mask, bit = 0, 0
        for a in range(r):
            for b in range(a + 1, r):
                same = close(c[a], c[b])
                like[a][b] = like[b][a] = same
                mask |= 0 if same else 1 << bit
                bit += 1
        votes = [sum(x) for x in like]
        k = votes.index(max(votes))
        replica.append(k)
        row.append(int(rows[j, k]))
        masks.append(mask)
    return replica, row, masks


def _close(a, b):
    bound = torch.maximum(a.abs(), b.abs()).mul_(RTOL).add_(ATOL)
    return bool(((a - b).abs() <= bound).all())


def _columns(X, index, d, fn):
    """fn([f, n] values of n coordinates, ascending) -> [n], over all coordinates, in 64 bits."""
    out = torch.empty(d, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // len(index))
    index = torch.as_tensor(index, dtype=torch.int64, device=DEV)
    for c0 in range(0, d, step):
        c1 = min(d, c0 + step)
        out[c0:c1] = fn(torch.sort(X[:, c0:c1].index_select(0, index), dim=0).values)
    return out


def _mean_around(v, beta):
    """Mean of the beta values of each (ascending) column closest to its median: the window grows
    from the median, the lower neighbour first on ties (differences in fp32)."""
    n = v.shape[0]
    h = (n - 1) // 2
    start = torch.full((v.shape[1],), max(0, h - beta + 1), dtype=torch.int64, device=v.device)
    for s in range(max(0, h - beta + 1), h):
        if s + beta <= n - 1:
            start += ((v[h] - v[s]) > (v[s + beta] - v[h])).to(torch.int64)
    total = torch.zeros(v.shape[1], dtype=torch.float64, device=v.device)
    for t in range(beta):
        total += v.gather(0, (start + t).unsqueeze(0))[0].to(torch.float64)
    return total / beta


def _distances(X, d, f):
    gram = torch.zeros((f, f), dtype=torch.float64, device=DEV)
    for c0 in range(0, d, 1 << 20):
        W = X[:f, c0:min(d, c0 + (1 << 20))].to(torch.float64)
        gram += W @ W.T.contiguous()
    g = gram.diagonal()
    dist = (g[:, None] + g[None, :] - 2.0 * gram).clamp_(min=0.0)
    dist.fill_diagonal_(0.0)
    return dist


def _krum_score(dist, left, i, n_terms):
    others = sorted(float(dist[i, j]) for j in left if j != i)
    return sum(others[:max(0, n_terms)])


def exact(case, seed):
    op, d = case["op"], case["d"]
    f64 = torch.float64
    if op in ("aggregate", "tolerant"):
        X, rows, r = _copies(case, seed)
        same = torch.equal if op == "aggregate" else _close
        replica, row, masks = _winners(X, rows, d, same)
        f = len(row)
        if op == "aggregate" and case["agg"] == "trim":
            b = case["b"]
            out = _columns(X, row, d, lambda v: v[b:f - b].to(f64).mean(dim=0))
        else:
            out = _columns(X, row, d, lambda v: v[(f - 1) // 2].to(f64))
        ints = [torch.tensor(t, dtype=torch.int32, device=DEV) for t in (replica, row, masks)]
        return (out, ints[0]) if op == "aggregate" else (out, ints[0], ints[1], ints[2])
    X, f = _rows(case, seed), case["f"]
    every = list(range(f))
    if op == "median":
        return _columns(X, every, d, lambda v: v[(f - 1) // 2].to(f64))
    if op == "trimmed_mean":
        b = case["b"]
        return _columns(X, every, d, lambda v: v[b:f - b].to(f64).mean(dim=0))
    if op == "mean_around_median":
        return _columns(X, every, d, lambda v: _mean_around(v, case["beta"]))
    dist = _distances(X, d, f)
    host = dist.cpu()
    c = case["c"]
    selected = torch.zeros(f, dtype=torch.int32, device=DEV)
    if op == "multi_krum":
        scores = [_krum_score(host, every, i, f - c - 2) for i in every]
        chosen = sorted(sorted(every, key=lambda i: (scores[i], i))[:case["m"]])
        selected[chosen] = 1
        out = torch.zeros(d, dtype=f64, device=DEV)
        for i in chosen:
            out += X[i, :d].to(f64)
        return out / len(chosen), selected, torch.tensor(scores, dtype=f64, device=DEV), dist
    left, order = list(every), []
    for _ in range(f - 2 * c):
        scores = [(_krum_score(host, left, i, len(left) - c - 2), i) for i in left]
        best = min(scores)[1]
        order.append(best)
        left.remove(best)
    selected[order] = 1
    beta = f - 4 * c
    out = _columns(X, order, d, lambda v: _mean_around(v, beta))
    return out, selected, torch.tensor(order, dtype=torch.int32, device=DEV), dist
