"""The work that a serving program gives this library, as cases that can be timed and checked.

A case is a dict of plain values. `prepare` makes the device inputs of one serving
iteration from a seed (trees, plans, operands, state banks, the previous iteration's
accepted path), `run` takes ONE pass through the package's public calls, `exact` gives the
same results in 64-bit torch arithmetic without the package, `work` the bytes and
operations one pass cannot do without.

Kinds of cases:
  step       one serving iteration of the GDN layers. `flow` says how it is called:
               deferred   conv, verification that publishes the previous path first, commit
                          that only derives the path (`hist` names the call that publishes
                          the conv history: the conv or the commit)
               fused      conv inside the verification, operands prepared in the kernels
               per_layer  one conv and one verification launch per layer, each layer with
                          its own buffers, one commit for all
               eager      conv, verification, commit with the replay (the form of fp32
                          operands, long paths and the sequential schedules)
  attention  one attention layer's verification of the same trees
  select     the drafter's fused argmax and top-k of full-vocabulary logits
"""
import math

import numpy as np
import torch

import paper_2609_23900_amd as L

DEV = "cuda"


# ------------------------------------------------------------------------------ cases
def _step(name, flow, n_req, layers, nodes, depth, accept, **kw):
    c = dict(name=name, kind="step", flow=flow, n_req=n_req, layers=layers, nodes=nodes, depth=depth,
             accept=accept, tree="uniform", chains=0, ragged=0, pad=0, h_k=16, h_v=32, d=128,
             dtype="bf16", policy="wy", hist="conv", bias=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one interactive request, one layer, the evaluated draft
        # geometry (28 nodes in 32 rows, 12 levels); latency and launches
        _step("one_request", "deferred", 1, 1, 28, 12, 12, tree="paper", pad=4, hist="commit"),
        # the way a model calls the step, layer by layer (eight of its layers), a batch of 8
        _step("per_layer", "per_layer", 8, 8, 64, 8, 8),
        # the headline: a batch of 8 requests, 48 GDN layers stacked in each call
        _step("stacked", "deferred", 8, 48, 64, 8, 8),
        # the same iteration from raw conv inputs: conv, normalisation and gates fused in
        _step("fused_prepared", "fused", 8, 12, 64, 8, 8, bias=True),
        # many requests with large deep trees, one layer
        _step("wide_deep", "deferred", 32, 1, 256, 16, 16, tree="skewed", hist="commit"),
        # a busy mixed batch: plain chains beside trees of odd sizes, padded rows
        _step("chains_and_trees", "deferred", 64, 1, 128, 16, 16, chains=32, ragged=9, pad=3, hist="commit"),
        # fp32 operands and outputs
        _step("fp32", "eager", 8, 12, 64, 8, 8, dtype="f32"),
        # paths beyond the matrix-core form's depth: long chain drafts inside trees
        _step("long_paths", "eager", 16, 4, 96, 32, 20, tree="spine", ragged=7),
        # the default policy of a plan, the paper's path scans, state bits equal to the commit's
        _step("sequential", "eager", 8, 6, 64, 8, 8, policy="paths"),
        # attention layer, one long-context request with the evaluated draft geometry
        dict(name="attention_long", kind="attention", n_req=1, nodes=28, depth=12, tree="paper", ragged=0, pad=4,
             h_q=16, h_kv=8, ctx=131072, ctx_step=0),
        # attention layer, a batch of 64-node trees over ragged contexts, eight query heads a key head
        dict(name="attention_batch", kind="attention", n_req=8, nodes=64, depth=8, tree="uniform", ragged=5, pad=0,
             h_q=32, h_kv=4, ctx=16384, ctx_step=1237),
        # the drafter's selection, one logits row per request at one drafting depth
        dict(name="draft_select", kind="select", rows=8, vocab=248320, dtype="f32", k=3, ties=1),
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["attention"] * 2 + ["select"])
    if kind == "select":
        return dict(kind="select", rows=_logint(rng, 1, 64), vocab=_logint(rng, 2000, 248320),
                    dtype=rng.choice(["f32", "bf16"]), k=rng.randint(1, 8), ties=rng.randint(0, 1))
    if kind == "attention":
        n_req, ctx = _logint(rng, 1, 16), _logint(rng, 64, 131072)
        ctx = min(ctx, 262144 // n_req)
        h_kv = rng.choice([2, 4, 8])
        return dict(kind="attention", n_req=n_req, nodes=_logint(rng, 1, 128), depth=rng.randint(8, 16),
                    tree="uniform", ragged=rng.randint(0, 8), pad=rng.randint(0, 4),
                    h_q=h_kv * rng.choice([1, 2, 4, 8]), h_kv=h_kv, ctx=ctx, ctx_step=rng.randint(0, ctx // (2 * n_req)))
    flow = rng.choice(["deferred", "deferred", "fused", "per_layer", "eager", "eager", "eager"])
    h_k, h_v = rng.choice([(16, 32), (16, 32), (16, 48), (8, 16), (2, 4), (8, 8)])
    d, dtype, policy, most = 128, "bf16", "wy", 24576
    n_req, nodes, depth = _logint(rng, 1, 64), _logint(rng, 8, 256), rng.randint(8, 17)
    if flow == "eager":
        form = rng.choice(["fp32", "long", "paths", "paths", "two_level", "recompute"])
        depth = rng.randint(18, 32) if form == "long" else depth
        dtype = "f32" if form == "fp32" or rng.random() < 0.2 else "bf16"
        d = rng.choice([64, 128, 128, 128])
        if form in ("fp32", "long"):
            most = 6144
        else:
            policy, most = form, 3072 if form == "paths" else 1024
    elif flow == "fused":
        h_k, h_v = rng.choice([(16, 32), (8, 16), (2, 4)])
    units = max(1, most * 32 // h_v)
    n_req = min(n_req, max(1, units // nodes))
    tiles = (6144 if flow == "eager" else 12288) // h_v  # state matrices of the batch
    layers = min(_logint(rng, 1, 48), max(1, units // (n_req * nodes)), max(1, tiles // n_req))
    if flow == "per_layer":
        layers = min(layers, 12)
    return dict(kind="step", flow=flow, n_req=n_req, layers=layers, nodes=nodes, depth=depth,
                accept=rng.randint(1, min(depth, 20)), tree=rng.choice(["uniform", "skewed", "spine"]),
                chains=rng.choice([0, 0, n_req // 2]), ragged=rng.randint(0, min(7, nodes - 1)),
                pad=rng.randint(0, 3), h_k=h_k, h_v=h_v, d=d, dtype=dtype, policy=policy,
                hist=rng.choice(["conv", "commit"]), bias=rng.random() < 0.3)


# ------------------------------------------------------------------------------ trees
def _grow(rng, n, depth, tree):
    """Parent array of an n-node candidate tree with at most `depth` nodes per path."""
    if tree == "chain":
        return list(range(-1, n - 1))
    if tree == "paper":  # 5 levels of three candidates, a six-token tail, two rescue branches
        par, spine = [-1], [0]
        for _ in range(5):
            par += [spine[-1]] * 3
            spine.append(len(par) - 3)
        for _ in range(6):
            par.append(spine[-1])
            spine.append(len(par) - 1)
        for at, length in ((2, 4), (4, 2)):
            p = spine[at]
            for _ in range(length):
                par.append(p)
                p = len(par) - 1
        return par
    par, dep = [-1], [0]
    if tree == "spine":  # one chain as deep as allowed, branches grown around it
        while len(par) < min(n, depth):
            par.append(len(par) - 1)
            dep.append(len(dep))
    front = [i for i in range(len(par)) if dep[i] < depth - 1]
    while len(par) < n:
        if not front:
            front.append(int(rng.choice([i for i in range(len(par)) if dep[i] < depth - 1])))
        p = front.pop(int(rng.integers(len(front))))
        most = max(1, 6 - dep[p] // 3) if tree == "skewed" else 4
        for _ in range(min(int(rng.integers(1, most + 1)), n - len(par))):
            par.append(p)
            dep.append(dep[p] + 1)
            if dep[-1] < depth - 1:
                front.append(len(par) - 1)
    return par


def _sizes(c):
    """Nodes of every request (a fixed rule of the case)."""
    if c["tree"] == "paper":
        return [28] * c["n_req"]
    n = []
    for r in range(c["n_req"]):
        if r < c.get("chains", 0):
            n.append(min(c["nodes"], c["depth"]))
        else:
            n.append(max(1, c["nodes"] - (3 * r) % (c["ragged"] + 1)))
    return n


def _accept_len(c, r, n):
    return min(1 + (5 * r + 2) % c["accept"], n, c["depth"])


class Batch:
    """Trees of a batch and where their rows are (host data, written out from the layout rule)."""

    def __init__(self, c, rng):
        self.sizes = _sizes(c)
        self.parents = [_grow(rng, n, c["depth"], "chain" if r < c.get("chains", 0) else c["tree"])
                        for r, n in enumerate(self.sizes)]
        self.n_rows = [n + c["pad"] for n in self.sizes]
        self.row_off = np.concatenate([[0], np.cumsum(self.n_rows)]).astype(np.int64)
        self.node_off = np.concatenate([[0], np.cumsum(self.sizes)]).astype(np.int32)
        self.rows_total = int(self.row_off[-1])
        self.depth, self.row, self.req, self.flat_parent = [], [], [], []
        for r, par in enumerate(self.parents):
            dep = [0] * len(par)
            first = {}
            for i in range(1, len(par)):
                dep[i] = dep[par[i]] + 1
                first.setdefault(par[i], i)
            slot, node = {}, 0
            while node is not None:  # the spine first, then the other nodes in order
                slot[node] = len(slot)
                node = first.get(node)
            for i in range(len(par)):
                if i not in slot:
                    slot[i] = len(slot)
            self.depth += dep
            self.row += [int(self.row_off[r]) + slot[i] for i in range(len(par))]
            self.req += [r] * len(par)
            self.flat_parent += [-1] + [int(self.node_off[r]) + p for p in par[1:]]

    def desc(self, policy):
        return L.TreeDesc.build(self.node_off, np.concatenate([np.asarray(p, np.int32) for p in self.parents]),
                                np.asarray(self.n_rows, np.int32), policy, DEV)

    def accepted(self, c, rng):
        """Per request a node at the depth of its accepted length (or the deepest there is)."""
        got = []
        for r in range(c["n_req"]):
            lo = int(self.node_off[r])
            dep = np.asarray(self.depth[lo:lo + self.sizes[r]])
            want = min(_accept_len(c, r, self.sizes[r]) - 1, int(dep.max()))
            got.append(int(rng.choice(np.nonzero(dep == want)[0])))
        return got

    def path(self, r, node):
        """Flat node ids from the root to `node` of request r."""
        out, i = [], int(self.node_off[r]) + node
        while i >= 0:
            out.append(i)
            i = self.flat_parent[i]
        return out[::-1]


# ------------------------------------------------------------------------------ inputs
def _paths(c, batch, accepted, width):
    out = np.full((c["n_req"], width), -1, np.int32)
    length = np.zeros(c["n_req"], np.int32)
    for r, node in enumerate(accepted):
        p = batch.path(r, node)
        length[r] = len(p)
        out[r, :len(p)] = np.asarray(p) - int(batch.node_off[r])
    return out, length


class Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, shape, dtype=torch.float32, scale=1.0):
        x = torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, scale, generator=self.g)
        return x.to(dtype)

    def uniform(self, shape, lo, hi):
        return torch.empty(shape, dtype=torch.float32, device=DEV).uniform_(lo, hi, generator=self.g)


def _rows_of(c, rnd, rows, dt, raw):
    """Recorded operands of one iteration: unit key rows, gates (or raw gate inputs)."""
    n, hk, hv, d = c["layers"], c["h_k"], c["h_v"], c["d"]
    t = dict(g=rnd.normal((n, rows, hv)), beta=rnd.normal((n, rows, hv)))
    if not raw:
        t["g"] = -torch.nn.functional.softplus(t["g"])
        t["beta"] = torch.sigmoid(t["beta"])
        t["q"] = rnd.normal((n, rows, hk, d), dt)
        t["k"] = torch.nn.functional.normalize(rnd.normal((n, rows, hk, d)), dim=-1).to(dt)
        t["v"] = rnd.normal((n, rows, hv, d), dt)
    return t


def _step_inputs(c, seed):
    rng, rnd = np.random.default_rng([int(seed), 1]), Rand(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    n, hk, hv, d, R = c["layers"], c["h_k"], c["h_v"], c["d"], c["n_req"]
    ch = 2 * hk * d + hv * d
    b = Batch(c, rng)
    s = dict(batch=b, dt=dt, channels=ch, accepted=b.accepted(c, rng), width=max(c["accept"], 1))
    s["now"] = _rows_of(c, rnd, b.rows_total, dt, c["flow"] == "fused")
    s["state"] = rnd.normal((R, n, hv, d, d), scale=0.1)
    s["x"] = rnd.normal((n, b.rows_total, ch), dt)
    s["hist"] = rnd.normal((R, n, 3, ch), dt)
    s["w"] = rnd.uniform((n, ch, 4), -0.5, 0.5)
    s["bias"] = rnd.normal((n, ch), scale=0.2) if c["bias"] else None
    if c["flow"] == "fused":
        s["a_log"] = rnd.normal((n, hv), scale=0.5)
        s["dt_bias"] = rnd.normal((n, hv))
    if c["flow"] != "eager":
        p = Batch(c, rng)
        s["prev"] = dict(batch=p, path=_paths(c, p, p.accepted(c, rng), s["width"]))
        s["prev"].update(_rows_of(c, rnd, p.rows_total, dt, c["flow"] == "fused"))
        s["prev"]["x"] = rnd.normal((n, p.rows_total, ch), dt)
    return s


def _attention_inputs(c, seed):
    rng, rnd = np.random.default_rng([int(seed), 1]), Rand(seed)
    b = Batch(c, rng)
    bf = torch.bfloat16
    off = np.concatenate([[0], np.cumsum(_contexts(c))]).astype(np.int32)
    rows, tok = b.rows_total, int(off[-1])
    s = dict(batch=b, off=off)
    s["q"] = rnd.normal((rows, c["h_q"], 128), bf)
    s["kt"], s["vt"] = (rnd.normal((rows, c["h_kv"], 128), bf) for _ in range(2))
    s["kc"], s["vc"] = (rnd.normal((max(tok, 1), c["h_kv"], 128), bf) for _ in range(2))
    return s


def _contexts(c):
    return [max(0, c["ctx"] - r * c["ctx_step"]) for r in range(c["n_req"])]


def prepare(case, seed):
    c = case
    if c["kind"] == "select":
        dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
        i32 = dict(dtype=torch.int32, device=DEV)
        s = dict(c=c, logits=Rand(seed).normal((c["rows"], c["vocab"]), dt, 3.0), spine=torch.zeros(c["rows"], **i32),
                 cand=torch.zeros((c["rows"], c["k"]), **i32))
        s["split"] = L.lumo_draft_select_splits(c["rows"], c["vocab"], L.LUMO_F32 if c["dtype"] == "f32" else L.LUMO_BF16)
        s["ws"] = torch.empty(max(16, L.lumo_draft_select_workspace_bytes(c["rows"], c["k"], s["split"])),
                              dtype=torch.uint8, device=DEV)
        return s
    if c["kind"] == "attention":
        s = _attention_inputs(c, seed)
        s.update(c=c, desc=s["batch"].desc(L.LUMO_POLICY_WY), dims=L.attn_dims(c["n_req"], c["h_q"], c["h_kv"]))
        s["ctx_off"] = torch.from_numpy(s["off"]).to(DEV)
        s["o"] = torch.zeros((s["batch"].rows_total, c["h_q"], 128), dtype=torch.bfloat16, device=DEV)
        s["lse"] = torch.zeros((s["batch"].rows_total, c["h_q"]), device=DEV)
        s["split"] = L.lumo_tree_attention_splits(s["dims"], s["desc"].plan, c["ctx"])
        s["ws"] = torch.empty(L.lumo_tree_attention_workspace_bytes(s["dims"], s["desc"].plan, s["split"]) // 4 + 4,
                              dtype=torch.float32, device=DEV)
        return s
    s = _step_inputs(c, seed)
    R, n, hv, d, b = c["n_req"], c["layers"], c["h_v"], c["d"], s["batch"]
    policy = L.POLICIES[c["policy"]]
    code = L.LUMO_F32 if c["dtype"] == "f32" else L.LUMO_BF16
    s["c"] = c
    s["dims"] = L.dims(R, n, c["h_k"], hv, d, d, code)
    s["desc"] = b.desc(policy)
    s["acc"] = torch.tensor(s["accepted"], dtype=torch.int32, device=DEV)
    s["path"] = torch.full((R, s["width"]), -1, dtype=torch.int32, device=DEV)
    s["plen"] = torch.zeros(R, dtype=torch.int32, device=DEV)
    s["o"] = torch.zeros((n, b.rows_total, hv, d), dtype=s["dt"], device=DEV)
    if c["flow"] != "fused":
        s["y"] = torch.zeros((n, b.rows_total, s["channels"]), dtype=s["dt"], device=DEV)
    s["ws"] = None
    need = L.lumo_tree_gdn_workspace_bytes(s["dims"], s["desc"].plan)
    if need:
        s["ws"] = torch.empty(need // 4, dtype=torch.float32, device=DEV)
    s["prep"] = None
    if c["flow"] == "fused":
        s["prep"] = L.Prep(L.LUMO_PREP_QK_NORM | L.LUMO_PREP_RAW_GATES, 1e-6, s["a_log"], s["dt_bias"])
    if c["flow"] != "eager":
        p = s["prev"]
        p["desc"] = p["batch"].desc(policy)
        p["path"], p["plen"] = (torch.from_numpy(a).to(DEV) for a in p["path"])
    if c["flow"] == "per_layer":
        # every layer its own state bank, history and plan-sharing calls
        s["state"] = [s["state"][:, l:l + 1].contiguous() for l in range(n)]
        s["hist"] = [s["hist"][:, l:l + 1].contiguous() for l in range(n)]
        one = L.dims(R, 1, c["h_k"], hv, d, d, code)
        none = L.TreeDesc.build(np.zeros(R + 1, np.int32), np.zeros(0, np.int32), np.ones(R, np.int32), policy, DEV)
        t, p, s["one"], s["calls"] = s["now"], s["prev"], one, []
        s["xs"] = [s["x"][l] for l in range(n)]
        for l in range(n):
            at = lambda u, names: [u[k][l] for k in names.split()]  # noqa: E731
            pend = (c["accept"], p["path"], p["plen"], *at(p, "k v g beta"))
            verify = L.pending_call(one, s["desc"], *at(t, "q k v g beta"), s["state"][l], s["o"][l],
                                    p["desc"] if l == 0 else none, *pend)
            publish = L.pending_call(one, none, None, None, None, None, None, s["state"][l], None, p["desc"], *pend)
            s["calls"].append((verify, publish))
    return s


# ------------------------------------------------------------------------------ one pass
def run(s):
    c = s["c"]
    if c["kind"] == "select":
        L.lumo_draft_select(s["logits"], c["k"], c["ties"], s["spine"], s["cand"], s["split"], s["ws"])
        return s["spine"], s["cand"]
    if c["kind"] == "attention":
        L.lumo_tree_attention(s["dims"], s["desc"], s["ctx_off"], c["ctx"], 1 / math.sqrt(128), s["q"], s["kc"], s["vc"],
                              s["kt"], s["vt"], s["o"], s["lse"], s["split"], s["ws"])
        return s["o"], s["lse"]
    t, ch, mp, act = s["now"], s["channels"], s["width"], 1
    if c["flow"] == "eager":
        L.lumo_tree_conv_gather(s["dims"], s["desc"], ch, s["x"], s["hist"], s["w"], s["bias"], act, s["y"])
        L.lumo_tree_gdn_verify(s["dims"], s["desc"], t["q"], t["k"], t["v"], t["g"], t["beta"], s["state"], s["o"],
                               workspace=s["ws"])
        L.lumo_gdn_commit(s["dims"], s["desc"], mp, s["acc"], s["path"], s["plen"], t["k"], t["v"], t["g"], t["beta"],
                          s["state"], ch, s["x"], s["hist"])
        return s["y"], s["o"], s["state"], s["hist"], s["path"], s["plen"]
    p = s["prev"]
    if c["flow"] == "fused":
        L.lumo_tree_gdn_verify_conv_pending(s["dims"], s["desc"], ch, s["x"], s["hist"], s["w"], s["bias"], act, t["g"],
                                            t["beta"], s["state"], s["o"], p["desc"], mp, p["path"], p["plen"], p["x"],
                                            p["g"], p["beta"], prep=s["prep"])
        L.lumo_gdn_commit(s["dims"], s["desc"], mp, s["acc"], s["path"], s["plen"], None, None, None, None, None)
        return s["o"], s["state"], s["hist"], s["path"], s["plen"]
    if c["flow"] == "per_layer":
        calls, n = s["calls"], c["layers"]
        for l in range(n):
            L.lumo_tree_conv_gather(s["one"], s["desc"], ch, s["xs"][l], s["hist"][l], s["w"][l],
                                    None if s["bias"] is None else s["bias"][l], act, s["y"][l])
            L.lumo_tree_gdn_verify_pending_pair(calls[l][0], calls[l + 1][1] if l + 1 < n else None)
        L.lumo_gdn_commit_hist_layers(s["dims"], s["desc"], mp, s["acc"], s["path"], s["plen"], ch, s["xs"], s["hist"])
        return s["y"], s["o"], s["state"], s["hist"], s["path"], s["plen"]
    if c["hist"] == "conv":
        L.lumo_tree_conv_gather_pending(s["dims"], s["desc"], ch, s["x"], s["hist"], s["w"], s["bias"], act, s["y"],
                                        p["desc"], mp, p["path"], p["plen"], p["x"])
    else:
        L.lumo_tree_conv_gather(s["dims"], s["desc"], ch, s["x"], s["hist"], s["w"], s["bias"], act, s["y"])
    L.lumo_tree_gdn_verify_pending(s["dims"], s["desc"], t["q"], t["k"], t["v"], t["g"], t["beta"], s["state"], s["o"],
                                   p["desc"], mp, p["path"], p["plen"], p["k"], p["v"], p["g"], p["beta"])
    late = c["hist"] == "commit"
    L.lumo_gdn_commit(s["dims"], s["desc"], mp, s["acc"], s["path"], s["plen"], None, None, None, None, None,
                      ch if late else 0, s["x"] if late else None, s["hist"] if late else None)
    return s["y"], s["o"], s["state"], s["hist"], s["path"], s["plen"]


# ------------------------------------------------------------------------------ work, tolerance
def work(case):
    """Every input read once, every output written once; multiply-adds as two operations."""
    c = case
    if c["kind"] == "select":
        return {"bytes": c["rows"] * (c["vocab"] * (4 if c["dtype"] == "f32" else 2) + 4 * (c["k"] + 1)),
                "flops": c["rows"] * c["vocab"]}
    sizes = _sizes(c)
    if c["kind"] == "attention":
        ctx = _contexts(c)
        kv = 2 * c["h_kv"] * 128 * 2
        by = sum(ctx) * kv + sum(sizes) * (kv + c["h_q"] * (2 * 128 * 2 + 4))
        return {"bytes": by, "flops": 4 * 128 * c["h_q"] * sum(n * (x + min(n, c["depth"])) for n, x in zip(sizes, ctx))}
    n, hk, hv, d, R, N = c["layers"], c["h_k"], c["h_v"], c["d"], c["n_req"], sum(sizes)
    e = 4 if c["dtype"] == "f32" else 2
    ch = 2 * hk * d + hv * d
    lens = sum(_accept_len(c, r, m) for r, m in enumerate(sizes))
    state = R * n * hv * d * d * 4
    node = hv * d * e + 2 * hv * 4  # outputs and gates of a node
    hist = R * n * 3 * ch * e
    by = 2 * state + 2 * hist + n * ch * 16 + n * (N * (node + ch * e) + lens * (2 * hv * 4 + (hk + hv) * d * e))
    by += n * N * ch * e  # fused: the queries, keys and values come from x
    if c["flow"] != "fused":
        by += n * N * ch * e  # y written, and q, k, v read beside x
    return {"bytes": by, "flops": n * hv * d * d * (6 * N + 4 * lens) + 8 * n * ch * N}


def tolerance(case):
    c = case
    if c["kind"] == "select":
        return "exact"
    if c["kind"] == "step" and c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    return {"rel": 5e-3, "max": 4e-2}


# ------------------------------------------------------------------------------ 64-bit results
def _select_exact(s):
    """Whole-number outputs are compared with the start's: nothing to give in 64 bits."""
    return None


def _attention_exact(c, seed):
    s = _attention_inputs(c, seed)
    b, G = s["batch"], c["h_q"] // c["h_kv"]
    o = torch.zeros((b.rows_total, c["h_q"], 128), dtype=torch.float64, device=DEV)
    lse = torch.zeros((b.rows_total, c["h_q"]), dtype=torch.float64, device=DEV)
    for r, n in enumerate(b.sizes):
        lo, row0 = int(b.node_off[r]), int(b.row_off[r])
        see = torch.zeros((n, n), dtype=torch.bool)
        for i in range(n):
            for a in b.path(r, i):
                see[b.row[lo + i] - row0, b.row[a] - row0] = True
        see = see.to(DEV)
        for h in range(c["h_kv"]):
            q = s["q"][row0:row0 + n, h * G:(h + 1) * G].double().reshape(n * G, 128)
            kc, vc = (s[k][int(s["off"][r]):int(s["off"][r + 1]), h].double() for k in ("kc", "vc"))
            kt, vt = (s[k][row0:row0 + n, h].double() for k in ("kt", "vt"))
            sc = torch.cat([q @ kc.T.contiguous(), q @ kt.T.contiguous()], 1) / math.sqrt(128)
            sc[:, kc.shape[0]:].masked_fill_(~see.repeat_interleave(G, 0), -math.inf)
            ls = torch.logsumexp(sc, 1)
            out = torch.exp(sc - ls[:, None]) @ torch.cat([vc, vt], 0)
            o[row0:row0 + n, h * G:(h + 1) * G] = out.reshape(n, G, 128)
            lse[row0:row0 + n, h * G:(h + 1) * G] = ls.reshape(n, G)
    return o, lse


def _history(hist, x, batch, paths, lens):
    """hist [R][n][3][ch] after the accepted paths' x rows."""
    out = hist.clone()
    for r in range(len(lens)):
        rows = [batch.row[int(batch.node_off[r]) + int(i)] for i in paths[r][:int(lens[r])]]
        both = torch.cat([hist[r], x[:, rows]], 1)
        out[r] = both[:, -3:]
    return out


def _conv(hist, x, rows_before, w, bias):
    """Conv outputs [m][ch] of one layer: window rows (m, 4) into cat(x, hist)."""
    src = torch.cat([x, hist.reshape(-1, x.shape[-1])], 0).double()
    y = torch.zeros((rows_before.shape[0], x.shape[-1]), dtype=torch.float64, device=DEV)
    if bias is not None:
        y += bias.double()
    for t in range(4):
        y += w[:, t].double() * src[rows_before[:, t]]
    return y * torch.sigmoid(y)


def _windows(batch, nodes):
    """Per node the four window rows, oldest first: x rows, or rows_total + 3 request + entry."""
    out = []
    for i in nodes:
        r, chain, a = batch.req[i], [], i
        while a >= 0 and len(chain) < 4:
            chain.append(batch.row[a])
            a = batch.flat_parent[a]
        past = [batch.rows_total + 3 * r + 2, batch.rows_total + 3 * r + 1, batch.rows_total + 3 * r]
        out.append((chain + past)[:4][::-1])
    return torch.tensor(out, dtype=torch.int64, device=DEV).reshape(-1, 4)


def _replay(S, paths, lens, batch, k, v, alpha, beta, G):
    """S [R][hv][dk][dv] after every request's path (k, v, alpha, beta by row)."""
    S = S.clone()
    for step in range(int(lens.max()) if len(lens) else 0):
        on = [r for r in range(len(lens)) if step < int(lens[r])]
        rows = [batch.row[int(batch.node_off[r]) + int(paths[r][step])] for r in on]
        S[on] = _update(S[on], k[rows], v[rows], alpha[rows], beta[rows], G)
    return S


def _update(S, k, v, alpha, beta, G):
    k = k.repeat_interleave(G, 1)
    S = S * alpha[..., None, None]
    delta = beta[..., None] * (v - (S * k[..., None]).sum(-2))
    return S + k[..., None] * delta[..., None, :]


def _step_exact(c, seed):
    s = _step_inputs(c, seed)
    b, n, hk, hv, d, G = s["batch"], c["layers"], c["h_k"], c["h_v"], c["d"], c["h_v"] // c["h_k"]
    ch, rows, fused = s["channels"], b.rows_total, c["flow"] == "fused"
    paths, lens = _paths(c, b, s["accepted"], s["width"])
    hist0, prev = s["hist"], s.get("prev")
    hist = hist0
    if prev is not None and (fused or c["flow"] == "deferred" and c["hist"] == "conv"):
        hist = _history(hist0, prev["x"], prev["batch"], *prev["path"])
    f64 = dict(dtype=torch.float64, device=DEV)
    y = None if fused else torch.zeros((n, rows, ch), **f64)
    o, state = torch.zeros((n, rows, hv, d), **f64), torch.zeros(s["state"].shape, **f64)
    nodes = list(range(len(b.row)))
    win, at = _windows(b, nodes), torch.tensor(b.row, device=DEV)
    if fused:
        pw = _windows(prev["batch"], list(range(len(prev["batch"].row))))
        pat = torch.tensor(prev["batch"].row, device=DEV)
    levels = [[i for i in nodes if b.depth[i] == j] for j in range(max(b.depth) + 1)]

    def split(z):  # conv outputs as stored (bf16) to normalised query and key rows, and values
        z = z.to(torch.bfloat16).double()
        q, k, v = z[:, :hk * d], z[:, hk * d:2 * hk * d], z[:, 2 * hk * d:]
        nrm = lambda u: u / torch.sqrt(u.square().sum(-1, keepdim=True) + 1e-6)  # noqa: E731
        return nrm(q.reshape(-1, hk, d)), nrm(k.reshape(-1, hk, d)), v.reshape(-1, hv, d)

    def gates(g, beta, l):
        g, beta = g.double(), beta.double()
        if not fused:
            return torch.exp(g), beta
        return (torch.exp(-torch.exp(s["a_log"][l].double()) * torch.nn.functional.softplus(g + s["dt_bias"][l].double())),
                torch.sigmoid(beta))

    for l in range(n):
        bias = None if s["bias"] is None else s["bias"][l]
        z = _conv(hist[:, l], s["x"][l], win, s["w"][l], bias)
        if fused:
            q, k, v = (torch.zeros((rows,) + u.shape[1:], **f64).index_copy(0, at, u) for u in split(z))
        else:
            y[l, at] = z
            q, k, v = (s["now"][u][l].double() for u in "qkv")
        alpha, beta = gates(s["now"]["g"][l], s["now"]["beta"][l], l)
        S0 = s["state"][:, l].double()
        if prev is not None:
            if fused:
                z = _conv(hist0[:, l], prev["x"][l], pw, s["w"][l], bias)
                _, pk, pv = (torch.zeros((prev["batch"].rows_total,) + u.shape[1:], **f64).index_copy(0, pat, u)
                             for u in split(z))
            else:
                pk, pv = prev["k"][l].double(), prev["v"][l].double()
            S0 = _replay(S0, *prev["path"], prev["batch"], pk, pv, *gates(prev["g"][l], prev["beta"][l], l), G)
        R, where = S0, list(range(c["n_req"]))
        for j, ids in enumerate(levels):
            pos = {i: m for m, i in enumerate(levels[j - 1])} if j else None
            src = [b.req[i] if j == 0 else pos[b.flat_parent[i]] for i in ids]
            rw = [b.row[i] for i in ids]
            R = _update(R[src], k[rw], v[rw], alpha[rw], beta[rw], G)
            o[l, rw] = (R * q[rw].repeat_interleave(G, 1)[..., None]).sum(-2)
        del R, where
        state[:, l] = S0 if prev is not None else _replay(S0, paths, lens, b, k, v, alpha, beta, G)
    if not fused and (c["flow"] in ("eager", "per_layer") or c["hist"] == "commit"):
        hist = _history(hist0, s["x"], b, paths, lens)
    ints = [torch.from_numpy(u).to(DEV) for u in (paths, lens)]
    if c["flow"] == "per_layer":
        state = [state[:, l:l + 1] for l in range(n)]
        hist = [hist[:, l:l + 1] for l in range(n)]
    else:
        hist = hist.double()
    if c["flow"] == "per_layer":
        hist = [h.double() for h in hist]
    out = (o, state, hist, *ints)
    return out if fused else (y,) + out


def exact(case, seed):
    if case["kind"] == "select":
        return _select_exact(case)
    if case["kind"] == "attention":
        return _attention_exact(case, seed)
    return _step_exact(case, seed)
