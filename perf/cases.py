"""Performance cases of the library: the calls a serving loop makes, through
the Python binding, over the range of sizes, families and activation types
the library is used with.

A case is a dict of plain values.  ``listed`` gives the fixed cases, ``draw``
one more of the same ranges, ``prepare`` the device tensors of one case,
``run`` one pass, ``work`` the bytes and operations a pass cannot do without,
``tolerance`` how far two correct implementations may differ and ``exact`` the
same outputs in fp64 from the definition, in plain torch.

Kinds of case (``op``):
  verify  one speculative round of ``layers`` layers: per layer one
          sla_verify with the previous round's accepted paths pending (fused
          commit-and-verify), or with ``fused`` false the draft alone;
  step    the same with the layer's short convolution in front of each;
  commit  the standalone accepted-path commit of one layer;
  conv    one layer's short convolution, with the accepted rows pending;
  prune   draft pruning and packing ahead of a round.
With ``graph`` the pass is the replay of a HIP graph of the whole round, as a
serving loop captures it; else every call is made eagerly.

Values: state ~ N(0, 0.02^2); q, k unit vectors and v ~ N(0, 1) in the
activation type; alpha = sigmoid(U(2, 5)), beta = sigmoid(N(0, 1)); GLA gates
sigmoid(N(0, 1))^(1/16); random trees within depth and branch limits (or
chains); accepted path: the root path of a uniformly drawn node (a uniform
prefix of a chain).  Pending records: keys and gates alike, corrected values
beta v.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_16673_amd import binding as B

CONV_K = 4


def _verify(name, batch, heads, dk, dv, n, *, family="gdn", dtype="bf16", chain=False, depth=5, branch=3, layers=1,
            graph=False, fused=True, n_prev=None, op="verify"):
    case = dict(op=op, family=family, dtype=dtype, batch=batch, heads=heads, dk=dk, dv=dv, n=n,
                n_prev=n if n_prev is None else n_prev, chain=chain, depth=depth, branch=branch, layers=layers,
                graph=graph, fused=fused)
    return dict(name=name, **case) if name else case


def _conv(name, batch, channels, n, *, kernel=CONV_K, dtype="bf16", bias=False, depth=5, branch=3):
    case = dict(op="conv", dtype=dtype, batch=batch, channels=channels, n=n, n_prev=n, kernel=kernel, bias=bias,
                chain=False, depth=depth, branch=branch)
    return dict(name=name, **case) if name else case


def _prune(name, batch, n, tau, budget):
    case = dict(op="prune", batch=batch, n=n, tau=tau, budget=budget)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # one interactive sequence, chain drafts, one layer called eagerly: the
        # smallest call, latency and host cost only
        _verify("chain8_call", 1, 16, 128, 128, 8, chain=True, depth=8, branch=1),
        # one interactive sequence, 32-node trees, every layer of a 24-layer
        # model (convolution, then recurrent core) from one HIP graph: the
        # latency of many small dependent launches, at head size 256
        _verify("batch1_step", 1, 8, 256, 256, 32, depth=12, branch=2, layers=24, graph=True, op="step"),
        # batched serving: 64 sequences, 16-node trees, 24 layers from one HIP
        # graph; the ordinary load
        _verify("tree_serving_step", 64, 16, 128, 128, 16, layers=24, graph=True),
        # the same layer with fp32 activations, called eagerly
        _verify("tree_serving_f32", 64, 16, 128, 128, 16, dtype="f32"),
        # per-key gates, sizes that fit no tile: 40 sequences, 12 heads, 144
        # value columns, 23 nodes
        _verify("gla_ragged", 40, 12, 128, 144, 23, family="gla", depth=6, branch=4),
        # throughput serving with the largest drafts
        _verify("large_tree64", 256, 16, 128, 256, 64, depth=8, branch=4),
        # plain decoding of a large batch: one node per sequence
        _verify("decode_chain1", 256, 16, 128, 256, 1, chain=True, depth=1, branch=1),
        # a moderate batch at head size 256, trees of 32 nodes
        _verify("d256_tree32", 16, 8, 256, 256, 32, depth=8, branch=4),
        # a few sequences at head size 256 with fp32 activations and the
        # largest trees
        _verify("d256_f32_tree64", 8, 8, 256, 256, 64, dtype="f32", depth=8, branch=4),
        # immediate commit of accepted paths (verification not fused with it)
        _verify("commit_trees", 64, 16, 128, 128, 16, op="commit"),
        # the short convolution of one batched serving layer: the q, k and v
        # channels of 16 heads
        _conv("conv_serving", 64, 16 * 3 * 128, 16),
        # 64-candidate rollouts of a batch cut to 16-node trees
        _prune("prune_batch", 64, 64, 3.0, 16),
    ]


# ------------------------------------------------------------------- draws
MAX_DRAW_BYTES = 1.2e9


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _limits(rng, n):
    """Depth and branch limits that hold n nodes."""
    branch = rng.randint(2, 4)
    depth = rng.randint(3, 8)
    while (branch ** depth - 1) // (branch - 1) < n:
        depth += 1
    return depth, branch


def _fits(case):
    return work(case)["bytes"] <= MAX_DRAW_BYTES


def draw(rng):
    op = rng.choices(["verify", "decode", "commit", "conv", "prune"], [12, 2, 2, 3, 1])[0]
    batch = _log_int(rng, 1, 256)
    n = _log_int(rng, 2, 64)
    dtype = rng.choices(["bf16", "f32"], [7, 3])[0]
    depth, branch = _limits(rng, 64)
    if op == "prune":
        n = rng.randint(8, 64)
        return _prune(None, batch, n, round(rng.uniform(0.5, 4.0), 2), rng.choice([0, rng.randint(1, n)]))
    if op == "conv":
        channels = rng.choice([rng.choice([4, 8, 16]) * 3 * rng.choice([64, 128, 256]), 8 * rng.randint(32, 1024)])
        case = _conv(None, batch, channels, rng.choice([1, n, n]), kernel=rng.choice([4, 4, 3, 2]), dtype=dtype,
                     bias=rng.random() < 0.3, depth=depth, branch=branch)
    else:
        heads = rng.choice([4, 8, 12, 16, 24, 32])
        dk = rng.choice([64, 128, 128, 256])
        dv = rng.choice([64, 128, 128, 256, 16 * rng.randint(2, 20)])
        family = rng.choices(["gdn", "deltanet", "decay", "gla"], [6, 1, 1, 2])[0]
        if op == "decode":
            case = _verify(None, batch, heads, dk, dv, 1, family=family, dtype=dtype, chain=True, depth=1, branch=1)
        else:
            if dk == 256 and (family == "gla" or dtype == "f32") and n > 32:  # the largest on-chip stage: small batches
                n, batch = min(n, 48 if family == "gla" else 64), min(batch, 64 // heads)
            chain = rng.random() < 0.25
            case = _verify(None, batch, heads, dk, dv, n, family=family, dtype=dtype, chain=chain,
                           depth=n if chain else depth, branch=1 if chain else branch,
                           fused=op == "commit" or rng.random() < 0.85,
                           n_prev=rng.choice([n, n, _log_int(rng, 1, 32)]) if op == "verify" else n,
                           op="commit" if op == "commit" else "verify")
    while not _fits(case) and case["batch"] > 1:
        case["batch"] = (case["batch"] + 1) // 2
    return case


# -------------------------------------------------------------- topologies
def _trees(rng, batch, n, depth, branch):
    """Random parent arrays [batch][n]; node 0 is the root."""
    parent = np.full((batch, n), -1, np.int32)
    level = np.full((batch, n), 1 << 20, np.int64)
    kids = np.zeros((batch, n), np.int64)
    level[:, 0] = 1
    rows = np.arange(batch)
    for i in range(1, n):
        free = (level[:, :i] < depth) & (kids[:, :i] < branch)
        pick = np.where(free, rng.random((batch, i)), -1.0).argmax(1)
        parent[:, i] = pick
        level[:, i] = level[rows, pick] + 1
        kids[rows, pick] += 1
    return parent


def _topology(rng, case, n):
    """(parent, path, length) of one round: int32 arrays."""
    batch = case["batch"]
    parent = np.tile(np.arange(-1, n - 1, dtype=np.int32), (batch, 1)) if case["chain"] else \
        _trees(rng, batch, n, case["depth"], case["branch"])
    path = np.full((batch, n), -1, np.int32)
    length = np.zeros(batch, np.int32)
    last = rng.integers(0, n, batch)
    if case["chain"] and n > 1:
        last = rng.integers(-1, n, batch)  # any prefix, the empty one too
    for b in range(batch):
        p, a = [], int(last[b])
        while a >= 0:
            p.append(a)
            a = int(parent[b, a])
        path[b, : len(p)] = p[::-1]
        length[b] = len(p)
    return parent, path, length


def _rng(seed):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([int(seed), 17])))


def _topologies(case, seed):
    """The draft of this round and the one before it, each (parent, path, length)."""
    rng = _rng(seed)
    cur = _topology(rng, case, case["n"])
    prev = _topology(rng, case, case.get("n_prev", case["n"]))
    return cur, prev


# ------------------------------------------------------------------ inputs
class _Gen:
    def __init__(self, seed, device):
        self.g = torch.Generator(device=device)
        self.g.manual_seed(int(seed))
        self.device = device

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device=self.device, dtype=torch.float32)

    def uniform(self, lo, hi, *shape):
        return torch.rand(shape, generator=self.g, device=self.device, dtype=torch.float32) * (hi - lo) + lo

    def unit(self, dtype, *shape):
        x = self.normal(*shape)
        return x.div_(x.norm(dim=-1, keepdim=True)).to(dtype)


def _act(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _gates(g, case, n):
    """(alpha, beta) of one round, each with the layers in front; None where the family reads none."""
    L, Bn, H, fam = case["layers"], case["batch"], case["heads"], case["family"]
    alpha = beta = None
    if fam in ("gdn", "decay"):
        alpha = torch.sigmoid(g.uniform(2.0, 5.0, L, Bn, n, H))
    elif fam == "gla":
        alpha = torch.sigmoid(g.normal(L, Bn, n, H, case["dk"])).pow_(1.0 / 16.0)
    if fam in ("gdn", "deltanet"):
        beta = torch.sigmoid(g.normal(L, Bn, n, H))
    return alpha, beta


def _core_inputs(case, seed, device):
    """Everything one round of the recurrent core takes, layers in front."""
    g = _Gen(seed, device)
    L, Bn, H, dk, dv, n, m = (case[x] for x in ("layers", "batch", "heads", "dk", "dv", "n", "n_prev"))
    dt = _act(case)
    cur, prev = _topologies(case, seed)
    s = {"state": g.normal(L, Bn, H, dk, dv).mul_(0.02)}
    s["q"], s["k"] = g.unit(dt, L, Bn, n, H, dk), g.unit(dt, L, Bn, n, H, dk)
    s["v"] = g.normal(L, Bn, n, H, dv).to(dt)
    s["alpha"], s["beta"] = _gates(g, case, n)
    pk = g.unit(dt, L, Bn, m, H, dk)
    pa, pb = _gates(g, case, m)
    pu = g.normal(L, Bn, m, H, dv)
    if pb is not None:
        pu.mul_(pb[..., None])
    if pa is None:
        pa = torch.ones(L, Bn, m, H, device=device)
    s["parent"], s["prev_parent"], s["path"], s["length"] = (torch.from_numpy(x).to(device)
                                                             for x in (cur[0], prev[0], prev[1], prev[2]))
    s["prev"] = dict(k=pk, u=pu, alpha=pa)
    return s


def _conv_inputs(case, seed, device, layers=1):
    g = _Gen(seed + 1000003, device)
    Bn, D, n, m, K = case["batch"], case["channels"], case["n"], case["n_prev"], case["kernel"]
    dt = _act(case)
    cur, prev = _topologies(case, seed)
    lim = 1.0 / math.sqrt(K)
    s = {"x": g.normal(layers, Bn, n, D).to(dt), "px": g.normal(layers, Bn, m, D).to(dt),
         "conv": g.normal(layers, Bn, K - 1, D).to(dt).float(), "weight": g.uniform(-lim, lim, layers, D, K),
         "bias": g.uniform(-lim, lim, layers, D) if case["bias"] else None}
    s["parent"], s["prev_parent"], s["path"], s["length"] = (torch.from_numpy(x).to(device)
                                                             for x in (cur[0], prev[0], prev[1], prev[2]))
    return s


def _step_conv(case):
    """The convolution case of one layer of a whole step."""
    return dict(batch=case["batch"], channels=case["heads"] * (2 * case["dk"] + case["dv"]), n=case["n"],
                n_prev=case["n_prev"], kernel=CONV_K, dtype=case["dtype"], bias=False, chain=case["chain"],
                depth=case["depth"], branch=case["branch"])


def _rollouts(case, seed):
    """Beam rollouts of the drafter: parents, log-probabilities [batch][n]."""
    rng = _rng(seed)
    Bn, n, k = case["batch"], case["n"], 4
    parent = np.full((Bn, n), -1, np.int32)
    logp = np.zeros((Bn, n), np.float32)
    for b in range(Bn):
        score, frontier, made = np.zeros(n), [-1], 0
        while made < n:
            nxt = []
            for f in sorted(frontier, key=lambda a: -score[a] if a >= 0 else 0.0)[:k]:
                z = 2.0 * rng.standard_normal(32)
                lp = np.sort(z - np.log(np.exp(z).sum()))[::-1][:k]
                for x in lp[: n - made]:
                    parent[b, made], logp[b, made] = f, x
                    score[made] = x + (score[f] if f >= 0 else 0.0)
                    nxt.append(made)
                    made += 1
            frontier = nxt
    return parent, logp


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    op = case["op"]
    if op == "prune":
        parent, logp = _rollouts(case, seed)
        return dict(case=case, parent=torch.from_numpy(parent).to(dev), logp=torch.from_numpy(logp).to(dev))
    if op == "conv":
        s = _conv_inputs(case, seed, dev)
        s.update(case=case, y=torch.empty_like(s["x"]),
                 status=torch.zeros(1, case["batch"], dtype=torch.int32, device=dev))
        return s
    s = _core_inputs(case, seed, dev)
    L, Bn, H, dk, dv, n, m = (case[x] for x in ("layers", "batch", "heads", "dk", "dv", "n", "n_prev"))
    dt = _act(case)
    s.update(case=case, status=torch.zeros(L, Bn, dtype=torch.int32, device=dev))
    prev = s["prev"]
    s["prev"] = [B.Factors(prev["k"][l], prev["u"][l], prev["alpha"][l], s["prev_parent"]) for l in range(L)]
    if op == "commit":
        return s
    gate = (L,) + B.gate_shape(Bn, n, H, dk, case["family"])
    s["out"] = torch.empty(L, Bn, n, H, dv, device=dev)
    s["records"] = dict(k=torch.empty(L, Bn, n, H, dk, dtype=dt, device=dev), u=torch.empty(L, Bn, n, H, dv, device=dev),
                        alpha=torch.empty(gate, device=dev),
                        parent=torch.empty(L, Bn, n, dtype=torch.int32, device=dev))
    r = s["records"]
    s["cur"] = [B.Factors(r["k"][l], r["u"][l], r["alpha"][l], r["parent"][l]) for l in range(L)]
    if op == "step":
        c = _conv_inputs(_step_conv(case), seed, dev, L)
        s["c"] = dict(c, y=torch.empty_like(c["x"]), status=torch.zeros(L, Bn, dtype=torch.int32, device=dev))
    if case["graph"]:
        # the kernels are loaded by one call on copies of a layer's states, then the round is captured
        t = dict(s, state=s["state"][:1].clone())
        if op == "step":
            t["c"] = dict(s["c"], conv=s["c"]["conv"][:1].clone())
        _layer(t, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        stream = torch.cuda.Stream(dev)
        stream.wait_stream(torch.cuda.current_stream(dev))
        with torch.cuda.stream(stream), torch.cuda.graph(graph, stream=stream):
            for l in range(L):
                _layer(s, l)
        torch.cuda.current_stream(dev).wait_stream(stream)
        s["graph"] = graph
    return s


# -------------------------------------------------------------------- pass
def _conv_layer(c, l):
    B.sla_conv_verify(c["conv"][l], c["x"][l], c["weight"][l], c["parent"], c["y"][l],
                      bias=None if c["bias"] is None else c["bias"][l],
                      pending=(c["px"][l], c["prev_parent"], c["path"], c["length"]), status=c["status"][l])


def _layer(s, l):
    case = s["case"]
    if case["op"] == "step":
        _conv_layer(s["c"], l)
    a, b = s["alpha"], s["beta"]
    B.sla_verify(s["state"][l], s["q"][l], s["k"][l], s["v"][l], None if a is None else a[l],
                 None if b is None else b[l], s["parent"], s["out"][l], s["cur"][l],
                 pending=(s["prev"][l], s["path"], s["length"]) if case["fused"] else None, status=s["status"][l],
                 topology="chain" if case["chain"] else "tree", family=case["family"])


def run(state):
    s = state
    case = s["case"]
    op = case["op"]
    if op == "prune":
        return B.sla_prune(s["parent"], s["logp"], case["tau"], case["budget"], with_scores=True)
    if op == "conv":
        _conv_layer(s, 0)
        return dict(y=s["y"], conv=s["conv"], status=s["status"])
    if op == "commit":
        B.sla_commit(s["state"][0], s["prev"][0], s["path"], s["length"], status=s["status"][0],
                     family=case["family"])
        return dict(state=s["state"], status=s["status"])
    if case["graph"]:
        s["graph"].replay()
    else:
        for l in range(case["layers"]):
            _layer(s, l)
    res = dict(state=s["state"], out=s["out"], records=s["records"], status=s["status"])
    if op == "step":
        res.update(y=s["c"]["y"], conv=s["c"]["conv"])
    return res


# -------------------------------------------------------------------- work
def _conv_work(c, length):
    Bn, D, n, m, K = c["batch"], c["channels"], c["n"], c["n_prev"], c["kernel"]
    w = 2 if c["dtype"] == "bf16" else 4
    rows = float(np.minimum(length, K - 1).sum())
    return (2 * Bn * n * D * w + 2 * Bn * (K - 1) * D * 4 + D * K * 4 + (D * 4 if c["bias"] else 0) + Bn * n * 4
            + rows * D * w + 2 * Bn * m * 4 + Bn * 8), 2.0 * Bn * n * D * K


def work(case):
    """Bytes: every input read once, every output written once (of the pending records those the accepted paths of
    one draw name; no state write-back without a pending path).  Operations: the contractions with the state, the
    Grams of each root path, the triangular solve and readout, and the rank-one updates of the accepted paths."""
    op = case["op"]
    if op == "prune":
        return {"bytes": case["batch"] * (case["n"] * 20 + 8), "flops": 10.0 * case["batch"] * case["n"]}
    (parent, _, _), (_, _, length) = _topologies(case, 0)
    if op == "conv":
        by, fl = _conv_work(case, length)
        return {"bytes": float(by), "flops": fl}
    L, Bn, H, dk, dv, n, m = (case[x] for x in ("layers", "batch", "heads", "dk", "dv", "n", "n_prev"))
    fam = case["family"]
    w = 2 if case["dtype"] == "bf16" else 4
    gate = dk * 4 if fam == "gla" else 4
    acc = float(length.sum())
    state = Bn * H * dk * dv * 4
    commit = acc * H * (dk * w + dv * 4 + gate) + acc * 4 + Bn * m * 4 + Bn * 8
    upd = 3.0 * acc * H * dk * dv
    if op == "commit":
        return {"bytes": 2.0 * state + commit, "flops": upd}
    reads = {"gdn": 8, "deltanet": 4, "decay": 4, "gla": dk * 4}[fam]
    by = state * (2 if case["fused"] else 1) + (commit if case["fused"] else 0)
    by += Bn * n * H * (2 * dk * w + dv * w + reads) + Bn * n * 4 + Bn * 4         # draft in, status out
    by += Bn * n * H * (dv * 4 + dk * w + dv * 4 + gate) + Bn * n * 4              # outputs, records
    pairs = 0.0  # (node, ancestor or itself) pairs of the drafts
    depth = np.zeros(parent.shape, np.int64)
    for j in range(n):
        up = np.take_along_axis(depth, np.maximum(parent[:, j:j + 1], 0), 1)[:, 0]
        depth[:, j] = np.where(parent[:, j] >= 0, up, 0) + 1
        pairs += float(depth[:, j].sum())
    delta = fam in ("gdn", "deltanet")
    fl = (2 if delta else 1) * (2.0 * Bn * H * n * dk * dv + 2.0 * pairs * H * dk + 2.0 * pairs * H * dv)
    fl += upd if case["fused"] else 0.0
    if op == "step":
        cb, cf = _conv_work(_step_conv(case), length)
        by, fl = by + cb, fl + cf
    return {"bytes": float(L * by), "flops": float(L * fl)}


def tolerance(case):
    """About four times the error measured against ``exact`` (2-norm), where rounding is not all of it."""
    if case["op"] == "prune":
        return "exact"  # whole numbers, and scores that the definition sums in fp32 in a stated order
    if case["op"] in ("conv", "step") and case["dtype"] == "bf16":
        # y rounded to bf16 (1.7e-3 from fp64): sums that differ in the last fp32 bits fall on the other side of a
        # rounding now and then, and are then one bf16 step apart
        return {"rel": 1e-3, "max": 1e-2}
    if case["op"] == "verify" and case["dtype"] == "bf16":
        # bf16 q, k, v against an fp32 state whose products take the state in two bf16 parts (measured 4e-6)
        return {"rel": 2e-5, "max": 1e-3}
    return {"rel": 2e-6, "max": 1e-4}  # fp32 products and sums (measured 2e-7)


# ------------------------------------------------------------------- exact
def _commit64(S, rec, path, length, fam):
    """State [B][H][dk][dv] (fp64) advanced along each accepted path, root first."""
    Bn = S.shape[0]
    rows = torch.arange(Bn, device=S.device)
    for t in range(int(length.max()) if Bn else 0):
        on = (length > t).view(Bn, 1, 1, 1)
        a = path[:, t].clamp(min=0).long()
        k, u, g = (rec[x][rows, a].double() for x in ("k", "u", "alpha"))  # [B][H][..]
        g = g[..., None] if fam == "gla" else g[..., None, None]
        S = torch.where(on, S * g + k[..., None] * u[:, :, None, :], S)
    return S


def _verify64(S, q, k, v, alpha, beta, parent, fam):
    """(out, u) of every node by the step's definition: the parent's state read through the committed state and the
    rank-one updates of the root path."""
    Bn, n, H, dk = q.shape
    q, k, v = q.double(), k.double(), v.double()
    one = torch.ones(Bn, n, H, 1, dtype=torch.float64, device=q.device)
    g = {"gla": lambda: alpha.double(), "deltanet": lambda: one}.get(fam, lambda: alpha.double()[..., None])()
    b = beta.double()[..., None] if fam in ("gdn", "deltanet") else None
    out, u = torch.empty_like(v), torch.empty_like(v)
    rows = torch.arange(Bn, device=q.device)
    par = parent.long()
    # what the committed state gives node j, through the gates of its root path (per key dimension for GLA)
    G = torch.empty(Bn, n, H, g.shape[-1], dtype=torch.float64, device=q.device)
    for j in range(n):
        up = torch.where((par[:, j] >= 0).view(Bn, 1, 1), G[rows, par[:, j].clamp(min=0)], one[:, 0])
        G[:, j] = up * g[:, j]

    def state_read(x):  # [B][n][H][dk] -> [B][n][H][dv]
        return torch.matmul((x * G).permute(0, 2, 1, 3).contiguous(), S).permute(0, 2, 1, 3)

    o0 = state_read(q)
    a0 = state_read(k) if b is not None else None
    for j in range(n):
        ak = torch.zeros(Bn, H, v.shape[-1], dtype=torch.float64, device=q.device)
        aq = torch.zeros_like(ak)
        D, x = g[:, j], par[:, j]  # D: the gates of the root path strictly below the ancestor x
        while bool((x >= 0).any()):
            on = (x >= 0).view(Bn, 1, 1)
            xc = x.clamp(min=0)
            ka, ua = k[rows, xc], u[rows, xc]
            wq = (q[:, j] * D * ka).sum(-1, keepdim=True)
            aq += torch.where(on, wq * ua, torch.zeros_like(aq))
            if b is not None:
                wk = (k[:, j] * D * ka).sum(-1, keepdim=True)
                ak += torch.where(on, wk * ua, torch.zeros_like(ak))
            D = torch.where(on, D * g[rows, xc], D)
            x = torch.where(x >= 0, par[rows, xc], x)
        # the parent's state read by k_j, times the node's own gate (alpha_j S_par k_j)
        u[:, j] = b[:, j] * (v[:, j] - (a0[:, j] + ak)) if b is not None else v[:, j]
        out[:, j] = o0[:, j] + aq + (q[:, j] * k[:, j]).sum(-1, keepdim=True) * u[:, j]
    return out, u


def _conv64(s, c, l):
    """(y, new conv state) of one layer, rows gathered by ancestor."""
    K, n = c["kernel"], c["n"]
    x, px, C, w = s["x"][l].double(), s["px"][l].double(), s["conv"][l].double(), s["weight"][l].double()
    Bn = x.shape[0]
    rows = torch.arange(Bn, device=x.device)
    new = C.clone()
    length, path = s["length"].long(), s["path"].long()
    for r in range(K - 1):
        z = length + r  # position in [C rows, accepted rows]
        old = C[rows, z.clamp(max=K - 2)]
        t = (z - (K - 1)).clamp(min=0, max=path.shape[1] - 1)
        acc = px[rows, path[rows, t].clamp(min=0)]
        new[:, r] = torch.where((z < K - 1)[:, None], old, acc)
    y = torch.empty_like(x)
    par = s["parent"].long()
    for j in range(n):
        acc = s["bias"][l].double().expand(Bn, -1).clone() if s["bias"] is not None else torch.zeros_like(x[:, 0])
        a = torch.full((Bn,), j, device=x.device, dtype=torch.long)
        past = torch.zeros(Bn, dtype=torch.long, device=x.device)  # committed rows used so far
        for lag in range(K):
            on = a >= 0
            z = torch.where(on[:, None], x[rows, a.clamp(min=0)], new[rows, (K - 2 - past).clamp(min=0)])
            acc += w[:, K - 1 - lag] * z
            past = torch.where(on, past, past + 1)
            a = torch.where(on, par[rows, a.clamp(min=0)], a)
        y[:, j] = acc * torch.sigmoid(acc)
    return y, new


def exact(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")
    op = case["op"]
    if op == "prune":
        return None  # whole numbers, and fp32 scores summed in a stated order
    if op == "conv":
        s = _conv_inputs(case, seed, dev)
        y, new = _conv64(s, case, 0)
        return dict(y=y[None], conv=new[None], status=None)
    s = _core_inputs(case, seed, dev)
    L, fam = case["layers"], case["family"]
    state, outs, us = [], [], []
    for l in range(L):
        S = s["state"][l].double()
        if case["fused"] or op == "commit":
            S = _commit64(S, {x: s["prev"][x][l] for x in ("k", "u", "alpha")}, s["path"], s["length"], fam)
        state.append(S)
        if op == "commit":
            break
        o, u = _verify64(S, s["q"][l], s["k"][l], s["v"][l], None if s["alpha"] is None else s["alpha"][l],
                         None if s["beta"] is None else s["beta"][l], s["parent"], fam)
        outs.append(o)
        us.append(u)
    if op == "commit":
        return dict(state=torch.stack(state), status=None)
    res = dict(state=torch.stack(state), out=torch.stack(outs), status=None,
               records=dict(k=None, u=torch.stack(us), alpha=None, parent=None))
    if op == "step":
        c = _step_conv(case)
        sc = _conv_inputs(c, seed, dev, L)
        got = [_conv64(sc, c, l) for l in range(L)]
        res.update(y=torch.stack([x[0] for x in got]), conv=torch.stack([x[1] for x in got]))
    return res
