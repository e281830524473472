"""The work that users of this library have it do, as a list of cases that a timing program can run.

Every case goes through the public entry points of ``paper_1903_00757_amd`` the way a training program does: graph,
alias table and embeddings are in place (``prepare``), then one pool is trained, one pool of walks is produced, or one
evaluation is made (``run``).  Graphs, pools and embeddings are synthetic and made on the GPU from the seed alone.

Fields of a case
  path      pool           one pool that lies in device memory, asynchronous mode      gv_train_device_pool
            static         the same through the entry point that allocates nothing     gv_train_device_pool_static
            push           one pool in host memory, pushed and trained                 gv_push_pool, gv_train_pool
            deterministic  one pool, batches without shared rows                       gv_train_device_pool
            walks          one pool written by the producer on the device              gv_augment_device
            loss           mean loss of an evaluation pool                             gv_eval_loss
            auc            link prediction                                             gv_link_prediction_auc
  nodes, edges, gamma   the graph: power law of that exponent, or (gamma 0) communities without hubs
  samples               pool length; node pairs of an evaluation
  dim, negatives        row length d and K
  track                 the running training loss is summed as well
  weighted, length, window, shuffle   of the walks
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1903_00757_amd as gv

WALK_LENGTH, WINDOW = 40, 5  # of the walks that pools are cut from
# a run of 10^10 samples near its end: an order of the same samples that is as good as another leaves rows that differ
# in proportion to the learning rate, and the time of a pass does not depend on it
LR0, LR_FLOOR, TOTAL, START = 0.025, 0.01, 10_000_000_000, 9_750_000_000
TRAINING_SEED, EVAL_SEED = 1234, 4711
EDGE_WEIGHTS = (0.25, 1.0, 4.0, 9.0)
TRAINING = ("pool", "static", "push", "deterministic")


def _train(name, path, nodes, edges, gamma, samples, dim, negatives, track=False):
    return dict(name=name, path=path, nodes=nodes, edges=edges, gamma=gamma, samples=samples, dim=dim,
                negatives=negatives, track=track)


def _walks(name, nodes, edges, gamma, samples, weighted, length, window, shuffle):
    return dict(name=name, path="walks", nodes=nodes, edges=edges, gamma=gamma, samples=samples, weighted=weighted,
                length=length, window=window, shuffle=shuffle)


def _evaluate(name, path, nodes, edges, gamma, samples, dim, negatives):
    return dict(name=name, path=path, nodes=nodes, edges=edges, gamma=gamma, samples=samples, dim=dim,
                negatives=negatives)


def listed():
    return [
        # the headline workload: a social graph of a million nodes with hubs, pools of 2^24 samples
        _train("million nodes, d128 k1", "pool", 1_000_000, 5_000_000, 2.1, 1 << 24, 128, 1),
        # the same graph with long rows and five negatives
        _train("million nodes, d512 k5", "pool", 1_000_000, 5_000_000, 2.1, 1 << 22, 512, 5),
        # community graph without hubs: the pool-order schedule
        _train("communities, d128 k1", "pool", 4_000_000, 40_000_000, 0.0, 1 << 22, 128, 1),
        # a graph whose matrices fit the last-level cache, 200 samples per node
        _train("ten thousand nodes, d128 k1", "pool", 10_000, 50_000, 3.0, 2_000_000, 128, 1),
        # odd sizes, rows that do not fill their lanes, and the running loss that a training program prints
        _train("tracked, d96 k3", "pool", 200_003, 1_000_000, 2.5, 1_000_003, 96, 3, track=True),
        # small steps of a loop that must not allocate
        _train("small static steps", "static", 100_000, 500_000, 2.5, 4096, 128, 1),
        # pools that a producer elsewhere in the program hands over in host memory
        _train("pushed from the host", "push", 1_000_000, 5_000_000, 2.1, 1 << 20, 64, 2),
        # reproducible training
        _train("deterministic", "deterministic", 10_000, 50_000, 3.0, 200_000, 128, 1),
        # the producer on the device: the pools of the headline workload
        _walks("walks", 1_000_000, 5_000_000, 2.1, 1 << 24, False, 40, 5, True),
        # edge weights, short-sighted window, pool in order of the walks
        _walks("weighted walks", 300_000, 1_500_000, 2.1, 3_000_001, True, 40, 2, False),
        # evaluation between pools: 2^18 samples
        _evaluate("evaluation loss", "loss", 1_000_000, 5_000_000, 2.1, 1 << 18, 128, 1),
        # five per cent of the edges held out against as many random pairs
        _evaluate("link prediction", "auc", 1_000_000, 5_000_000, 2.1, 250_000, 128, 1),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even on the logarithm's scale."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["pool", "pool", "pool", "static", "push", "deterministic", "walks", "walks", "loss", "auc"])
    if path in ("static", "deterministic"):
        nodes = _spread(rng, 5_000, 200_000)
    elif path == "walks":
        nodes = _spread(rng, 5_000, 1_000_000)
    else:
        nodes = _spread(rng, 10_000, 2_000_000)
    edges = nodes * rng.randint(4, 10) + rng.randint(0, 999)
    gamma = rng.choice([0.0, 2.1, 2.3, 2.5, 3.0])
    # of short rows with one negative, as trained most, up to the longest
    dim = rng.choice([32, 64, 96, 128, 128, 128, 160, 256, 352, 512])
    negatives = rng.choice([1, 1, 1, 2, 3, 5])
    if path == "walks":
        return {k: v for k, v in _walks("", nodes, edges, gamma, _spread(rng, 20_000, 1 << 24), rng.random() < 0.4,
                                        rng.choice([5, 10, 20, 40, 40, 64]), rng.choice([1, 2, 5, 5, 10]),
                                        rng.random() < 0.7).items() if k != "name"}
    if path == "loss":
        case = _evaluate("", path, nodes, edges, gamma, _spread(rng, 1_000, 1 << 20), dim, negatives)
    elif path == "auc":
        case = _evaluate("", path, nodes, edges, gamma, _spread(rng, 1_000, 500_000), dim, 1)
    else:
        most = {"pool": 1 << 23, "static": 100_000, "push": 1 << 21, "deterministic": 150_000}[path]
        most = min(most, 200 * nodes, (1 << 31) // (dim * (2 + negatives)))
        samples = _spread(rng, {"pool": 50_000, "static": 1_000, "push": 50_000, "deterministic": 1_000}[path], most)
        case = _train("", path, nodes, edges, gamma, samples, dim, negatives,
                      track=path in ("pool", "push") and rng.random() < 0.25)
    del case["name"]
    return case


# ---------------------------------------------------------------------------------------------------- inputs


def _graph(case, gen):
    """CSR adjacency (offsets int64[n + 1], adj int64[2m]) on the GPU, both directions of every edge."""
    n, m, gamma = case["nodes"], case["edges"], case["gamma"]

    def uniform(count):
        return torch.rand(count, dtype=torch.float64, device="cuda", generator=gen)

    names = torch.randperm(n, device="cuda", generator=gen)  # hubs lie anywhere in the matrices
    if gamma:
        b = 1.0 - 1.0 / (gamma - 1.0)  # node of rank r is drawn with weight r^(b - 1)

        def ends(count):
            r = (1.0 + uniform(count) * (float(n + 1) ** b - 1.0)) ** (1.0 / b)
            return names[(r.long() - 1).clamp_(0, n - 1)]
    else:
        groups = max(1, n // 10_000)

    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < m:
        count = int((m - keys.numel()) * 1.3) + 1024
        if gamma:
            x, y = ends(count), ends(count)
        else:  # one edge in nine stays inside its community
            x = (uniform(count) * n).long().clamp_(max=n - 1)
            y = (uniform(count) * n).long().clamp_(max=n - 1)
            inside = uniform(count) < 1.0 / 9.0
            y = torch.where(inside, (y - y % groups + x % groups).clamp_(max=n - 1), y)
        lo, hi = torch.minimum(x, y), torch.maximum(x, y)
        keys = torch.unique(torch.cat([keys, (lo * n + hi)[lo != hi]]))
    keys = keys[torch.sort(torch.randperm(keys.numel(), device="cuda", generator=gen)[:m]).values]
    lo, hi = keys // n, keys % n
    both = torch.sort(torch.cat([keys, hi * n + lo])).values
    offsets = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(both // n, minlength=n), 0, out=offsets[1:])
    return offsets, both % n


def _edge_weights(offsets, adj):
    """A weight from EDGE_WEIGHTS for every adjacency entry, the same in both directions."""
    n = offsets.numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), offsets[1:] - offsets[:-1])
    lo, hi = torch.minimum(row, adj), torch.maximum(row, adj)
    pick = ((lo * 2654435761 + hi * 40503) >> 7) & 3
    return torch.tensor(EDGE_WEIGHTS, dtype=torch.float32, device="cuda")[pick]


def _pool(offsets, adj, count, gen):
    """int32[count, 2] on the GPU: pairs within WINDOW steps of random walks, in the producer's shuffled order."""
    ij = [(i, j) for i in range(WALK_LENGTH + 1) for j in range(i + 1, min(i + WINDOW, WALK_LENGTH) + 1)]
    walks = -(-count // len(ij))

    def below(limit):
        u = torch.rand(walks, dtype=torch.float64, device="cuda", generator=gen)
        return torch.minimum((u * limit).long(), limit - 1)

    start = below(torch.full((walks,), adj.numel(), dtype=torch.int64, device="cuda"))
    at = torch.searchsorted(offsets, start, right=True) - 1
    path = torch.empty((walks, WALK_LENGTH + 1), dtype=torch.int32, device="cuda")
    path[:, 0] = at
    for t in range(1, WALK_LENGTH + 1):
        at = adj[offsets[at] + below(offsets[at + 1] - offsets[at])]
        path[:, t] = at
    i, j = (torch.tensor(x, device="cuda") for x in zip(*ij))
    pairs = torch.stack([path[:, i], path[:, j]], dim=2).reshape(-1, 2)[:count]
    return torch.cat([pairs[b::WINDOW] for b in range(WINDOW)]).contiguous()


def _rows(n, dim, gen):
    """Embedding rows as a run has them after its first part: of length about one and a half."""
    return torch.randn((n, dim), dtype=torch.float32, device="cuda", generator=gen).mul_(1.5 / math.sqrt(dim))


def _inputs(case, seed):
    """Everything that the seed decides: adjacency, and what the path needs beside it."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    offsets, adj = _graph(case, gen)
    made = {"offsets": offsets, "adj": adj}
    path, n = case["path"], case["nodes"]
    if path == "walks":
        made["first_walk"] = int(torch.randint(1 << 40, (1,), device="cuda", generator=gen))
        if case["weighted"]:
            made["weights"] = _edge_weights(offsets, adj)
        return made
    if path == "auc":
        count = case["samples"]
        at = torch.randint(adj.numel(), (count,), device="cuda", generator=gen)
        made["edges"] = torch.stack([torch.searchsorted(offsets, at, right=True) - 1, adj[at]])
        first = torch.randint(n, (count,), device="cuda", generator=gen)
        step = torch.randint(1, n, (count,), device="cuda", generator=gen)
        made["others"] = torch.stack([first, (first + step) % n])
    else:
        made["pairs"] = _pool(offsets, adj, case["samples"], gen)
    made["vertex"], made["context"] = _rows(n, case["dim"], gen), _rows(n, case["dim"], gen)
    if path == "auc":
        # rows that a run has taught something: a node is a little like one of its neighbours
        friend = adj[offsets[:-1].clamp(max=adj.numel() - 1)]
        made["vertex"] += 0.5 * made["context"][torch.minimum(friend, torch.arange(n, device="cuda"))]
    return made


class _Trainer:
    """A context that is given back when nothing refers to it any more."""

    def __init__(self, **config):
        self.ctx = gv.gv_create(**config)

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            gv.gv_destroy(self.ctx)
            self.ctx = None


class _Matrix:
    """One of a context's matrices, for torch.as_tensor: the tensor keeps the context."""

    def __init__(self, trainer, which, shape):
        self.trainer = trainer
        self.__cuda_array_interface__ = {"shape": shape, "typestr": "<f4", "version": 3, "strides": None,
                                         "data": (gv.gv_device_embeddings(trainer.ctx, which), False)}


def _host(x, dtype):
    return np.ascontiguousarray(x.cpu().numpy().astype(dtype))


def prepare(case, seed):
    made = _inputs(case, seed)
    path, n, count = case["path"], case["nodes"], case["samples"]
    offsets, adj = made["offsets"], made["adj"]
    degree = _host(offsets[1:] - offsets[:-1], np.uint32)
    trainer = _Trainer(dim=case.get("dim", 32), num_neg=case.get("negatives", 1), lr0=LR0, lr_min_ratio=LR_FLOOR,
                       total_samples=TOTAL, seed=TRAINING_SEED, pool_capacity=count if path == "push" else 8,
                       mode=gv.GV_MODE_DETERMINISTIC if path == "deterministic" else gv.GV_MODE_HOGWILD,
                       track_loss=1 if case.get("track") else 0)
    ctx = trainer.ctx
    state = {"case": case, "trainer": trainer}
    if path == "walks":
        if case["weighted"]:
            gv.gv_set_weighted_graph(ctx, _host(offsets, np.uint64), _host(adj, np.uint32),
                                     _host(made["weights"], np.float32))
        else:
            gv.gv_set_degrees(ctx, degree)
            gv.gv_set_adjacency(ctx, _host(offsets, np.uint64), _host(adj, np.uint32))
        state["first_walk"] = made["first_walk"]
        state["out"] = torch.empty((count, 2), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        return state
    gv.gv_set_degrees(ctx, degree)
    gv.gv_build_alias(ctx, 0.75)
    gv.gv_set_position(ctx, START)
    rows = [torch.as_tensor(_Matrix(trainer, which, (n, case["dim"])), device="cuda")
            for which in (gv.GV_VERTEX, gv.GV_CONTEXT)]
    rows[0].copy_(made["vertex"])
    rows[1].copy_(made["context"])
    state["rows"] = rows
    if path in ("push", "loss"):
        state["pairs"] = _host(made["pairs"], np.uint32)
    elif path == "auc":
        state["ends"] = [_host(x, np.uint32) for x in (*made["edges"], *made["others"])]
    else:
        state["pairs"] = made["pairs"]
    torch.cuda.synchronize()  # the context works on streams of its own
    return state


def run(state):
    case, ctx = state["case"], state["trainer"].ctx
    path, count = case["path"], case["samples"]
    if path in ("pool", "deterministic"):
        gv.gv_train_device_pool(ctx, state["pairs"].data_ptr(), count)
    elif path == "static":
        gv.gv_train_device_pool_static(ctx, state["pairs"].data_ptr(), count)
    elif path == "push":
        gv.gv_push_pool(ctx, state["pairs"], count)
        gv.gv_train_pool(ctx)
    elif path == "walks":
        gv.gv_augment_device(ctx, state["out"].data_ptr(), seed=TRAINING_SEED, walk_length=case["length"],
                             window=case["window"], first_walk=state["first_walk"], count=count,
                             shuffle=gv.GV_SHUFFLE_PSEUDO if case["shuffle"] else gv.GV_SHUFFLE_NONE)
        return state["out"]
    elif path == "loss":
        return gv.gv_eval_loss(ctx, state["pairs"], EVAL_SEED)
    else:
        return gv.gv_link_prediction_auc(ctx, *state["ends"])
    return {"vertex": state["rows"][0], "context": state["rows"][1]}


def work(case):
    """Every row that is named is read once and, in training, written once; so are pools and walk pairs."""
    path, n, count = case["path"], case["nodes"], case["samples"]
    if path == "walks":
        per_walk = sum(case["length"] + 1 - d for d in range(1, min(case["window"], case["length"]) + 1))
        steps = -(-count // per_walk) * (case["length"] + 1)
        entry = 4 + (8 if case["weighted"] else 0)  # a neighbour, and the alias entry that chose it
        graph = 8.0 * (n + 1) + 2.0 * case["edges"] * entry
        return {"bytes": 8.0 * count + min(graph, steps * (16.0 + entry)), "flops": 0.0}
    row = 4.0 * case["dim"]
    if path == "auc":
        return {"bytes": 16.0 * count + row * min(n, 4 * count), "flops": 2.0 * count * 6 * case["dim"]}
    K = case["negatives"]
    rows = min(2 * n, (2 + K) * count)
    table = min(16.0 * n, 16.0 * K * count)
    if path == "loss":
        return {"bytes": 8.0 * count + table + rows * row, "flops": 2.0 * (1 + K) * case["dim"] * count}
    return {"bytes": 8.0 * count + table + 2 * rows * row, "flops": 6.0 * (1 + K) * case["dim"] * count}


def tolerance(case):
    path = case["path"]
    if path == "walks":
        return "exact"
    if path in ("loss", "auc"):
        return {"rel": 1e-6, "max": 1e-6}
    if path == "deterministic":
        return {"rel": 1e-6, "max": 4e-5}
    # asynchronous: concurrent samples that share rows meet in another order each time.  Between the schedules that
    # keep contended updates (and from one of them to itself, and to sequential training) up to 0.0011 was measured
    # where rows are named often, with single values 0.46 apart, and up to 0.0004 and 0.064 elsewhere; a schedule that
    # loses such updates (device-scope stores everywhere) is 0.003 to 0.008 off, with single values over 1 apart.
    if case["samples"] > 8 * case["nodes"]:
        return {"rel": 0.004, "max": 0.99}
    return {"rel": 0.0015, "max": 0.25}


# ------------------------------------------------------------------------- the same in 64 bits, in plain numpy and torch


def _philox(index, sub, stream, seed):
    """Philox4x32-10 (Salmon et al.): four words for every pair of index and sub-index."""
    index = np.asarray(index, dtype=np.uint64)
    low = np.uint64(0xFFFFFFFF)
    c = [index & low, index >> np.uint64(32), np.full_like(index, sub), np.full_like(index, stream)]
    k = [seed & 0xFFFFFFFF, seed >> 32]
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k[0]), b & low, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k[1]), a & low]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    return c


def _alias_table(degree):
    """Vose's construction over degree^(3/4), with the stacks and roundings that the header states."""
    root = np.sqrt(degree.astype(np.float64))
    q = root * np.sqrt(root)
    n = q.size
    p = (q * float(n) / float(np.cumsum(q)[-1])).tolist()
    keep, alias = [1.0] * n, list(range(n))
    below = [i for i in range(n) if p[i] < 1.0]
    above = [i for i in range(n) if not p[i] < 1.0]
    while below and above:
        poor, rich = below.pop(), above.pop()
        keep[poor], alias[poor] = p[poor], rich
        p[rich] = (p[rich] + p[poor]) - 1.0
        (below if p[rich] < 1.0 else above).append(rich)
    thresh = np.minimum(np.floor(np.array(keep) * 4294967296.0), 4294967295.0).astype(np.uint64)
    return thresh, np.array(alias, dtype=np.int64)


def _negatives(degree, first, count, K, stream, seed):
    """int64[count, K]: the alias table's draws."""
    n = degree.size
    thresh, alias = _alias_table(degree)
    out = np.empty((count, K), dtype=np.int64)
    for k in range(K):
        w = _philox(np.arange(first, first + count, dtype=np.uint64), k, stream, seed)
        # floor(R n / 2^64) of the 64-bit R = w0 2^32 + w1, for n below 2^32
        at = ((w[0] * np.uint64(n) + ((w[1] * np.uint64(n)) >> np.uint64(32))) >> np.uint64(32)).astype(np.int64)
        out[:, k] = np.where(w[2] < thresh[at], at, alias[at])
    return out


def _exact_training(case, made):
    n, K, count = case["nodes"], case["negatives"], case["samples"]
    degree = (made["offsets"][1:] - made["offsets"][:-1]).cpu().numpy()
    pairs = made["pairs"].cpu().numpy().astype(np.int64)
    neg = _negatives(degree, START, count, K, 0, TRAINING_SEED)
    # samples in order, cut into levels: a sample comes one level after the last one that shares a row with it, so
    # those of one level share none and may be taken together
    level_u, level_c = [0] * n, [0] * n
    level = np.empty(count, dtype=np.int64)
    for i, (u, v, ks) in enumerate(zip(pairs[:, 0].tolist(), pairs[:, 1].tolist(), neg.tolist())):
        at = max(level_u[u], level_c[v])
        for k in ks:
            if level_c[k] > at:
                at = level_c[k]
        level[i] = at
        level_u[u] = level_c[v] = at + 1
        for k in ks:
            level_c[k] = at + 1
    order = np.argsort(level, kind="stable")
    ends = np.cumsum(np.bincount(level)).tolist()
    x, c = made["vertex"].double(), made["context"].double()
    u = torch.from_numpy(pairs[order, 0]).cuda()
    rows = torch.from_numpy(np.concatenate([pairs[order, 1:2], neg[order]], axis=1)).cuda()
    g = START + order.astype(np.float64)
    lr0, floor = float(np.float32(LR0)), float(np.float32(LR_FLOOR))
    lr = torch.from_numpy((lr0 * np.maximum(1.0 - g / TOTAL, floor)).astype(np.float32).astype(np.float64)).cuda()
    label = torch.zeros(K + 1, dtype=torch.float64, device="cuda")
    label[0] = 1.0
    weight = torch.full((K + 1,), float(np.float32(5.0) / np.float32(K)), dtype=torch.float64, device="cuda")
    weight[0] = 1.0
    lo = 0
    for hi in ends:
        uu, rr = u[lo:hi], rows[lo:hi]
        xs, cs = x[uu], c[rr]  # [s, d], [s, K + 1, d]
        coef = (label - torch.sigmoid((cs * xs[:, None]).sum(2))) * weight * lr[lo:hi, None]
        x.index_copy_(0, uu, xs + (coef[:, :, None] * cs).sum(1))
        c.index_add_(0, rr.reshape(-1), (coef[:, :, None] * xs[:, None]).reshape(-1, x.shape[1]))
        lo = hi
    return {"vertex": x, "context": c}


def _exact_loss(case, made):
    K, count = case["negatives"], case["samples"]
    degree = (made["offsets"][1:] - made["offsets"][:-1]).cpu().numpy()
    rows = torch.from_numpy(_negatives(degree, 0, count, K, 2, EVAL_SEED)).cuda()
    pairs = made["pairs"].long()
    total, w = 0.0, float(np.float32(5.0) / np.float32(K))
    for at in range(0, count, 1 << 14):
        x = made["vertex"][pairs[at:at + (1 << 14), 0]].double()
        s = (x * made["context"][pairs[at:at + (1 << 14), 1]].double()).sum(1)
        total -= float(torch.nn.functional.logsigmoid(s).sum())
        for k in range(K):
            s = (x * made["context"][rows[at:at + (1 << 14), k]].double()).sum(1)
            total -= w * float(torch.nn.functional.logsigmoid(-s).sum())
    return total / count


def _exact_auc(case, made):
    def cosines(ends):
        a, b = (made["vertex"][e].double() for e in ends)
        return (a * b).sum(1) / (a.norm(dim=1) * b.norm(dim=1))

    pos, neg = cosines(made["edges"]), torch.sort(cosines(made["others"])).values
    under = torch.searchsorted(neg, pos) + torch.searchsorted(neg, pos, right=True)  # equal scores count half
    return float(under.double().sum()) / 2.0 / (pos.numel() * neg.numel())


def exact(case, seed):
    path = case["path"]
    if path == "walks":
        return None  # whole numbers
    if path in TRAINING and (case["samples"] * (2 + case["negatives"]) > 7_000_000 or case["nodes"] * case["dim"] > 300_000_000):
        return None  # sample after sample: takes too long
    made = _inputs(case, seed)
    return {"loss": _exact_loss, "auc": _exact_auc}.get(path, _exact_training)(case, made)
