"""Performance cases of the verification step and of the draft step.

A case is one call (or the two or three calls that a program makes together) of the
package's entry points on one batch, as a decoding loop makes it: the logits, trees,
candidates and uniforms are on the GPU, the workspace was allocated once, and the outputs
come back as device tensors.  Ranges:

  * batches from one position or one tree to a thousand trees (one request being decoded,
    a small server, a large one);
  * vocabularies from 32,000 to 151,936: sizes padded to a multiple of 128, as most
    checkpoints have them, and odd ones, as after a token was added;
  * fp32 and bf16 logits, both residual rules, candidates with and without replacement;
  * the trees of the package's synthetic workloads: chains of a few candidates per level,
    a wide root with chains, random trees, and serving trees.

Inputs are synthetic: target logits follow a Zipf law over random ranks plus Gaussian
noise, draft logits are noisy copies, candidates are drawn from the draft's softmax.
"""
import math

import numpy as np
import torch

from paper_2608_24411_amd import native, synth

# Trees by name: (parent array or a rule for random ones, nodes, depth).
TREES = {
    "chain21": synth.first_child_chain((4, 4, 4, 4, 4)),      # depth 5, 4 candidates a level
    "serving26": synth.first_child_chain((10, 8, 5, 2)),      # widths along the first path
    "wide33": synth.fan_chains(8, 3),                         # 8 children, a chain under each
    "random60": None,                                         # random, breadth first, depth <= 6
}
NODES = {"chain21": 21, "serving26": 26, "wide33": 33, "random60": 60}
DEPTH = {"chain21": 5, "serving26": 4, "wide33": 4, "random60": 6}
# nodes with children per tree (random trees: the mean)
INNER = {"chain21": 5, "serving26": 4, "wide33": 25, "random60": 29}
# rows that a walk reaches, with children and without (means on these inputs)
REACHED = {"chain21": (2.5, 0.3), "serving26": (2.3, 0.4), "wide33": (2.7, 0.1), "random60": (2.9, 0.6)}

CHUNK = 1 << 26      # elements generated or evaluated at once
LARGEST = 2_400_000_000


def _case(name, call, tree, B, V, dtype, mode="resispec", T=1.0, zipf=1.1, sigma=1.25, worep=False, k=0):
    return dict(name=name, call=call, tree=tree, B=B, V=V, dtype=dtype, mode=mode, T=T, zipf=zipf, sigma=sigma,
                worep=worep, k=k)


def listed():
    return [
        # one position of each of 8 requests, no tree: the smallest call
        _case("flat-8x32000-f32", "flat", "", 8, 32000, "f32", sigma=1.5, k=4),
        # positions of a batch without trees, a vocabulary with one token added
        _case("flat-64x128257-bf16", "flat", "", 64, 128257, "bf16", "specinfer", k=6),
        # one request with a serving tree: latency of a single user's step
        _case("one-serving-tree-bf16", "group", "serving26", 1, 151936, "bf16", T=0.8, zipf=1.2, sigma=1.5, worep=True),
        # one request with a small tree over an odd vocabulary
        _case("one-chain-32001-f32", "group", "chain21", 1, 32001, "f32", "specinfer", sigma=1.5),
        # a small server: 8 requests, only the rows that each walk reaches
        _case("path-8-wide-bf16", "path", "wide33", 8, 128256, "bf16", T=0.7, zipf=1.0),
        # a busy server: 128 requests, only the rows that each walk reaches
        _case("path-128-wide-bf16", "path", "wide33", 128, 128256, "bf16", T=0.7, zipf=1.0),
        # every node tested, draws deferred: small rows, where launches and tails count
        _case("deferred-64-chain-f32", "deferred", "chain21", 64, 32000, "f32", sigma=1.5),
        # every node tested, draws deferred: the benchmarked batch
        _case("deferred-128-wide-bf16", "deferred", "wide33", 128, 128256, "bf16", T=0.7, zipf=1.0),
        # the same on a large serving batch: the largest call
        _case("deferred-1024-serving-bf16", "deferred", "serving26", 1024, 151936, "bf16", T=0.8, zipf=1.2, sigma=1.5,
              worep=True),
        # every node's own outcome wanted (statistics, training of drafters): random trees
        _case("nodes-32-random-f32", "nodes", "random60", 32, 128256, "f32", sigma=1.0),
        # the same over an odd vocabulary
        _case("nodes-64-wide-65537-bf16", "nodes", "wide33", 64, 65537, "bf16", T=0.7, zipf=1.0),
        # the draft step of a large serving batch
        _case("draft-256-serving-bf16", "draft", "serving26", 256, 151936, "bf16", T=0.8, zipf=1.2, sigma=1.5,
              worep=True),
    ]


def _between(rng, lo, hi):
    """Whole number from lo to hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    call = rng.choice(("flat", "group", "path", "path", "deferred", "deferred", "nodes", "draft"))
    V = _between(rng, 32000, 151936)
    if rng.random() < 0.5:
        V = (V + 127) // 128 * 128
    most = {"flat": 512, "group": 4, "path": 256, "deferred": 512, "nodes": 256, "draft": 512}[call]
    tree = "" if call == "flat" else rng.choice(("chain21", "serving26", "wide33", "random60"))
    dtype = rng.choice(("f32", "bf16"))
    if tree:      # no more logits than the largest listed case reads
        most = min(most, LARGEST // ((NODES[tree] + INNER[tree]) * V * (4 if dtype == "f32" else 2)))
    case = _case("", call, tree, _between(rng, 1 if call != "deferred" else 8, most), V, dtype,
                 rng.choice(("resispec", "resispec", "specinfer")), round(rng.uniform(0.6, 1.0), 2),
                 round(rng.uniform(1.0, 1.2), 2), round(rng.uniform(1.0, 1.5), 2),
                 worep=call != "flat" and (tree == "serving26" or rng.random() < 0.25),
                 k=rng.randint(1, 8) if call == "flat" else 0)
    del case["name"]
    return case


# --------------------------------------------------------------------- inputs ----

def _parents(case, seed):
    B, tree = case["B"], case["tree"]
    if TREES[tree] is not None:
        return np.broadcast_to(TREES[tree], (B, NODES[tree]))
    # a batch's random trees, drawn from a stock of 32 of this seed
    stock = [synth.random_bfs(np.random.default_rng([seed, b]), NODES[tree], DEPTH[tree],
                              np.array((0.4, 0.3, 0.2, 0.1))) for b in range(min(B, 32))]
    return np.stack([stock[b % 32] for b in range(B)])


def _logits(case, rows, g):
    """Target and draft logits of `rows` rows, in the case's type, and nothing else kept."""
    V = case["V"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    t, d = (torch.empty((rows, V), dtype=dt, device="cuda") for _ in range(2))
    step = max(1, CHUNK // V)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        x = torch.rand((n, V), generator=g, device="cuda").mul_(V).floor_().add_(1.0).log_().mul_(-case["zipf"])
        x += torch.randn((n, V), generator=g, device="cuda")
        t[r:r + n] = x
        x += torch.randn((n, V), generator=g, device="cuda").mul_(case["sigma"])
        d[r:r + n] = x
    return t, d


def _candidates(case, draft, rows, k, g):
    """k candidates of each of the draft rows `rows` (int64 device tensor), from the softmax."""
    out = torch.empty((rows.numel(), k), dtype=torch.int32, device="cuda")
    step = max(1, CHUNK // case["V"])
    for r in range(0, rows.numel(), step):
        p = torch.softmax(draft[rows[r:r + step]].float() / case["T"], dim=1)
        out[r:r + step] = torch.multinomial(p, k, replacement=not case["worep"], generator=g)
    return out


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, V = case["B"], case["V"]
    kw = dict(temperature=case["T"], mode=case["mode"], without_replacement=bool(case["worep"]))
    if case["call"] == "flat":
        t, d = _logits(case, B, g)
        cand = _candidates(case, d, torch.arange(B, device="cuda"), case["k"], g)
        u = torch.rand((B, case["k"] + 1), generator=g, device="cuda")
        kw.pop("without_replacement")
        return dict(case=case, kw=kw, args=(t, d, cand, u[:, :-1].contiguous(), u[:, -1].contiguous()))
    N, depth = NODES[case["tree"]], DEPTH[case["tree"]]
    par = _parents(case, seed)
    t, d = _logits(case, B * N, g)
    t, d = t.view(B, N, V), d.view(B, N, V)
    parent = torch.as_tensor(np.array(par, order="C"), dtype=torch.int32, device="cuda")
    if case["call"] == "draft":
        kw.pop("mode")
        return dict(case=case, kw=dict(kw, seed=seed), args=(d, parent))
    # children of a node in ascending index take its candidates in drawing order
    order = np.zeros((B, N), dtype=np.int64)
    for b in range(B if TREES[case["tree"]] is None else 1):
        seen = {}
        for n in range(1, N):
            order[b, n] = seen.get(int(par[b, n]), 0)
            seen[int(par[b, n])] = order[b, n] + 1
    if TREES[case["tree"]] is not None:
        order[:] = order[:1]
    owner = (np.arange(B)[:, None] * N + par)[:, 1:].reshape(-1)      # the row that each node was drawn from
    inner, where = np.unique(owner, return_inverse=True)
    cand = _candidates(case, d.view(B * N, V), torch.as_tensor(inner, device="cuda"), int(order.max()) + 1, g)
    pick = torch.as_tensor(where * cand.shape[1] + order[:, 1:].reshape(-1), device="cuda")
    token = torch.full((B, N), -1, dtype=torch.int32, device="cuda")
    token[:, 1:] = cand.reshape(-1)[pick].view(B, N - 1)
    u = torch.rand((2, B, N), generator=g, device="cuda")
    need = {"group": lambda: native.resispec_tree_group_workspace_bytes(B, N),
            "path": lambda: native.resispec_path_workspace_bytes(B, V),
            "deferred": lambda: native.resispec_deferred_workspace_bytes(B, N),
            "nodes": lambda: native.resispec_workspace_bytes(B, N)}[case["call"]]()
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = [torch.empty(shape, dtype=torch.int32, device="cuda") for shape in ((B, depth + 1), (B,), (B,))]
    return dict(case=case, kw=dict(kw, workspace=ws), out=out, depth=depth, args=(t, d, token, parent, u[0], u[1]))


def run(state):
    call, args, kw = state["case"]["call"], state["args"], state["kw"]
    if call == "flat":
        return native.resispec_verify(*args, **kw)
    if call == "draft":
        return native.resispec_draft_candidates(*args, **kw)
    if call != "nodes":
        entry = {"group": native.resispec_verify_tree_group, "path": native.resispec_verify_tree_path_group,
                 "deferred": native.resispec_verify_tree_deferred}[call]
        tokens, length, status = state["out"]
        return entry(*args, max_depth=state["depth"], out_tokens=tokens, out_accepted_len=length, out_status=status,
                     **kw)
    native.resispec_verify_nodes(*args, **kw)
    native.resispec_walk(args[2], kw["workspace"], *state["out"], max_depth=state["depth"])
    B, N = args[3].shape
    return state["out"], native.resispec_node_outcomes(kw["workspace"], B, N)


# ------------------------------------------------------------- work, tolerance ----

def work(case):
    """Bytes: the logits rows that the call has to read, each once.  Every node's target
    row and the draft row of every node with children where each node draws or the walk is
    not known; the rows with children alone where draws are deferred; the reached rows on
    the path.  Ids, uniforms and outputs are 28 bytes a node."""
    B, row = case["B"], case["V"] * (2 if case["dtype"] == "bf16" else 4)
    if case["call"] == "flat":
        rows, small = 2 * B, B * (8 * case["k"] + 16)
    else:
        N, inner = NODES[case["tree"]], INNER[case["tree"]]
        reached, ends = REACHED[case["tree"]]
        rows = {"draft": B * inner, "path": B * (2 * reached + ends), "deferred": B * 2 * inner,
                "group": B * (N + inner), "nodes": B * (N + inner)}[case["call"]]
        small = 28 * B * N
    # a scale, an exponential and a sum for each logit
    return {"bytes": int(rows * row + small), "flops": int(3 * rows * case["V"])}


def tolerance(case):
    """Tokens, lengths and node outcomes are whole numbers decided by sums of 32-bit
    elements; a draw or a test within rounding of a boundary can fall either way (against
    sums in 64 bits: up to 0.0016 of the values, over these cases and eight drawn ones)."""
    if case["call"] == "flat" and case["B"] < 100:
        return "exact"
    return {"rel": 0.0, "differ": 0.006}


# ------------------------------------------------------------------ 64 bits ----

def _draw64(R, u):
    """Smallest j whose running sum of R (rows) exceeds u * total; the last j with mass
    where rounding leaves none."""
    c = torch.cumsum(R, dim=1)
    tok = torch.searchsorted(c, (u * c[:, -1]).unsqueeze(1), right=True).squeeze(1)
    last = R.shape[1] - 1 - (R.flip(1) > 0).to(torch.uint8).argmax(dim=1)
    return torch.minimum(tok, last)


def _nodes64(case, p, q, cand, n_cand, u, ur):
    """One node a row: p, q logits [r, V], candidates [r, k] (the first n_cand of each
    row count).  Returns (index of the accepted candidate or -1, token)."""
    T, r = case["T"], p.shape[0]
    R = torch.softmax(p.double() / T, dim=1)
    D = torch.softmax(q.double() / T, dim=1)
    child = torch.full((r,), -1, dtype=torch.int64, device="cuda")
    token = child.clone()
    live = torch.arange(r, device="cuda")          # rows that have accepted nothing yet
    for i in range(cand.shape[1]):
        live = live[(child[live] < 0) & (n_cand[live] > i)]
        if not live.numel():
            break
        x = cand[live, i].long().unsqueeze(1)
        Rx, Dx = R[live].gather(1, x), D[live].gather(1, x)
        ok = u[live, i].double().unsqueeze(1) < Rx / Dx
        hit = live[ok.squeeze(1)]
        child[hit] = i
        token[hit] = cand[hit, i].long()
        no = ~ok.squeeze(1)
        live, x, Rx, Dx = live[no], x[no], Rx[no], Dx[no]
        A, Bd = R[live], D[live]
        if case["mode"] == "specinfer":
            A = (A - Bd).clamp_(min=0.0)
        else:
            A.scatter_(1, x, 0.0)
            Z = Dx - Rx
            m = torch.minimum(Z * Bd, A)
            m.scatter_(1, x, 0.0)
            M, S = m.sum(1, keepdim=True), A.sum(1, keepdim=True)
            a = torch.where(S > M, (Z - M) / (S - M), torch.zeros_like(M))
            A = (1.0 - a) * m + a * A
        R[live] = A / A.sum(1, keepdim=True)
        if case["worep"]:
            Bd = Bd.scatter(1, x, 0.0)
            D[live] = Bd / Bd.sum(1, keepdim=True)
    rest = torch.nonzero(child < 0).squeeze(1)
    if rest.numel():
        token[rest] = _draw64(R[rest], ur[rest].double())
    return child, token


def _tree64(case, s, nodes):
    """Outcomes of the nodes (b, n) in `nodes` ([r, 2], host): (child node or -1, token)."""
    t, d, token, parent, ua, ur = s["args"]
    par = parent.cpu().numpy()
    child = np.full(len(nodes), -1, dtype=np.int64)
    tok = np.full(len(nodes), -1, dtype=np.int64)
    step = max(1, CHUNK // case["V"])
    for r in range(0, len(nodes), step):
        part = nodes[r:r + step]
        kids = [np.flatnonzero(par[b] == n) for b, n in part]
        k = max(1, max(len(x) for x in kids))
        ids = np.zeros((len(part), k), dtype=np.int64)
        for i, x in enumerate(kids):
            ids[i, :len(x)] = x
        bb, nn = (torch.as_tensor(part[:, c], device="cuda") for c in (0, 1))
        idd = torch.as_tensor(ids, device="cuda")
        c, w = _nodes64(case, t[bb, nn], d[bb, nn], token[bb.unsqueeze(1), idd],
                        torch.as_tensor([len(x) for x in kids], device="cuda"), ua[bb.unsqueeze(1), idd], ur[bb, nn])
        c = c.cpu().numpy()
        child[r:r + step] = np.where(c >= 0, ids[np.arange(len(part)), np.maximum(c, 0)], -1)
        tok[r:r + step] = w.cpu().numpy()
    return child, tok


def _philox(n, b, seed):
    """Words 0, 1 and 2 of Philox4x32-10 with counter (n, b, 0, 0) and key `seed` (Salmon,
    Moraes, Dror and Shaw, SC'11), as uniforms with 24 bits."""
    M32 = np.uint64(0xFFFFFFFF)
    c = [x.astype(np.uint64) for x in (n, b, np.zeros_like(n), np.zeros_like(n))]
    k0, k1 = np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32)
    for r in range(10):
        if r:
            k0, k1 = (k0 + np.uint64(0x9E3779B9)) & M32, (k1 + np.uint64(0xBB67AE85)) & M32
        x, y = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(y >> np.uint64(32)) ^ c[1] ^ k0, y & M32, (x >> np.uint64(32)) ^ c[3] ^ k1, x & M32]
    return [(w >> np.uint64(8)).astype(np.float32) * np.float32(2.0 ** -24) for w in c[:3]]


def _draft64(case, s):
    d, parent = s["args"]
    par = parent.cpu().numpy()
    B, N = par.shape
    bb, nn = np.meshgrid(np.arange(B), np.arange(N), indexing="ij")
    ua, ur, uc = _philox(nn, bb, s["kw"]["seed"])
    token = np.full((B, N), -1, dtype=np.int32)
    todo = [(b, n, np.flatnonzero(par[b] == n)) for b in range(B) for n in range(N)]
    todo = [x for x in todo if len(x[2])]
    step = max(1, CHUNK // case["V"])
    for r in range(0, len(todo), step):
        part = todo[r:r + step]
        D = torch.softmax(d[[x[0] for x in part], [x[1] for x in part]].double() / case["T"], dim=1)
        for i in range(max(len(x[2]) for x in part)):
            at = [j for j, x in enumerate(part) if len(x[2]) > i]
            u = torch.as_tensor([float(uc[part[j][0], part[j][2][i]]) for j in at], dtype=torch.float64, device="cuda")
            rows = torch.as_tensor(at, device="cuda")
            x = _draw64(D[rows], u)
            if case["worep"]:
                D[rows, x] = 0.0
            for j, v in zip(at, x.tolist()):
                token[part[j][0], part[j][2][i]] = v
    return token, ua, ur, np.zeros(B, dtype=np.int32)


def exact(case, seed):
    s = prepare(case, seed)
    B = case["B"]
    if case["call"] == "flat":
        t, d, cand, ua, ur = s["args"]
        child, tok = _nodes64(case, t, d, cand, torch.full((B,), case["k"], device="cuda"), ua, ur)
        return tok.int(), (child >= 0).int(), torch.zeros_like(tok).int()
    if case["call"] == "draft":
        return _draft64(case, s)
    token = s["args"][2].cpu().numpy()
    out = np.full((B, s["depth"] + 1), -1, dtype=np.int32)
    length, zero = np.zeros(B, dtype=np.int32), np.zeros(B, dtype=np.int32)
    every = {}
    if case["call"] == "nodes":
        N = NODES[case["tree"]]
        nodes = np.stack(np.meshgrid(np.arange(B), np.arange(N), indexing="ij"), -1).reshape(-1, 2)
        child, tok = _tree64(case, s, nodes)
        every = {(b, n): (c, w) for (b, n), c, w in zip(nodes.tolist(), child, tok)}
    live = [(b, 0) for b in range(B)]
    while live:
        if case["call"] == "nodes":
            got = [every[x] for x in live]
        else:
            got = list(zip(*_tree64(case, s, np.array(live))))
        after = []
        for (b, n), (c, w) in zip(live, got):
            out[b, length[b]] = token[b, c] if c >= 0 else w
            if c >= 0:
                length[b] += 1
                after.append((b, int(c)))
        live = after
    walk = (out, length, zero)
    if case["call"] != "nodes":
        return walk
    shape = (B, NODES[case["tree"]])
    return walk, (child.reshape(shape).astype(np.int32), tok.reshape(shape).astype(np.int32),
                  np.zeros(shape, dtype=np.int32))
