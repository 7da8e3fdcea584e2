"""The work that programs hand to this library, as cases that can be timed and checked.

A speculative decoder calls the library in two phases per cycle.  Drafting grows a candidate pool (one
`draft_expand` per level of the tree, each followed by the depth policy), sizes it (size policy) and cuts
the tree out of it (`select_candidates`).  Verification runs `tree_verify_attn` once per layer of the
target model, then `tree_accept` (greedy) or `tree_accept_sampling` (T > 0) once, then `kv_compact` over
all layers.  The cases are those calls one by one and both phases whole, at batch 1 (a single user, the
latency-bound setting) and in batches, over the head layouts, prefixes and tree sizes of the repository's
workloads: 8B-, 13B-, 14B-, 32B- and 70B-shaped attention, prefixes up to 16384 tokens, trees of 8 to 256
nodes, contiguous and paged caches, bf16 (and fp32, the correctness setting).

All inputs are synthetic and made on the GPU from the seed.
"""
import math
import random

import numpy as np
import torch

import paper_2603_01639_amd as ltd

BEAM = 10  # children per expanded node and leaves kept per round
MAX_NODES = 256
SIZE_DIMS = (2 + 1011, 1024, 256, 12)  # the size policy's layers: state, hidden, hidden, actions
DEPTH_DIMS = (2 + 100, 1024, 2)
PAD = -100.0  # state entries past the pool's end

# (query heads, kv heads, head size) of the attention shapes
H_8B = dict(Hq=32, Hkv=8, d=128)
H_32B = dict(Hq=64, Hkv=8, d=128)  # also 70B-shaped
H_TP8 = dict(Hq=8, Hkv=1, d=128)  # 70B-shaped, one GPU's share under 8-way tensor parallelism
H_14B = dict(Hq=40, Hkv=8, d=128)
H_13B = dict(Hq=40, Hkv=40, d=128)  # no grouped queries
H_D64 = dict(Hq=32, Hkv=8, d=64)
H_TINY = dict(Hq=8, Hkv=8, d=64)


def _attn(name, heads, dtype="bf16", B=1, P=(0, 0), N=(0, 0), block=0):
    """An attention case: prefixes and tree sizes spread over P and N (ends included) across the batch;
    block = rows per block of a paged cache, 0 for a contiguous one."""
    c = dict(kind="attn", dtype=dtype, B=B, P0=P[0], P1=P[1], N0=N[0], N1=N[1], block=block, **heads)
    return dict(name=name, **c) if name else c


def _step(name, heads, layers, B, P, N, voc, block):
    c = _attn(name, heads, "bf16", B, P, N, block)
    c.update(kind="step", layers=layers, voc=voc)
    return c


def listed():
    return [
        # The correctness setting: a tiny fp32 model.  Launch latency is all there is.
        _attn("attn_f32_tiny", H_TINY, "f32", 1, (128, 128), (16, 16)),
        # One user of an 8B-shaped model in a short chat: a 60-node tree over 2048 tokens.
        _attn("attn_8b_p2048_n60", H_8B, "bf16", 1, (2048, 2048), (60, 60)),
        # The same user in long reasoning or with a long document.
        _attn("attn_8b_p16384_n60", H_8B, "bf16", 1, (16384, 16384), (60, 60)),
        # A 32B-shaped model with the smallest and the largest verification sizes.
        _attn("attn_32b_p4096_n8", H_32B, "bf16", 1, (4096, 4096), (8, 8)),
        _attn("attn_32b_p4096_n256", H_32B, "bf16", 1, (4096, 4096), (256, 256)),
        # A serving batch over a paged cache, 70B-shaped, ragged prefixes and trees.
        _attn("attn_70b_b16_paged", H_32B, "bf16", 16, (1024, 8192), (16, 128), 16),
        # The same batch on one GPU of an 8-way tensor-parallel group.
        _attn("attn_70b_b16_paged_tp8", H_TP8, "bf16", 16, (1024, 8192), (16, 128), 16),
        # The whole verification of one user's cycle: 32 layers, greedy acceptance, compaction.
        _step("verify_8b", H_8B, 32, 1, (2048, 2048), (60, 60), 128256, 0),
        # The whole verification of a serving batch on a four-layer pipeline stage with the head.
        _step("verify_70b_b16_paged", H_32B, 4, 16, (1024, 8192), (16, 128), 128256, 16),
        # Acceptance at temperature 1 for one user.
        dict(name="sampling_8b", kind="sampling", B=1, N0=60, N1=60, voc=128256, T=1.0),
        # One user's drafting phase at depth 6: expansion and depth policy per level, size policy,
        # selection.
        dict(name="draft_tree_b1", kind="draft", B=1, levels=6, voc=128256),
        # A serving batch's drafting phase, two levels (the depth policy stops early).
        dict(name="draft_tree_b16", kind="draft", B=16, levels=3, voc=128256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["attn1"] * 5 + ["attnb"] * 3 + ["f32", "step1", "stepb", "sampling", "draft"])
    if kind == "attn1":  # one user: any head layout, contiguous or paged
        P, N = _log_int(rng, 64, 16384), _log_int(rng, 8, 256)
        return _attn("", rng.choice([H_8B, H_32B, H_TP8, H_14B, H_13B, H_D64]), "bf16", 1, (P, P),
                     (N, N), rng.choice([0, 0, 0, 16, 32, 64]))
    if kind == "attnb":
        lo, n0 = _log_int(rng, 64, 2048), _log_int(rng, 8, 32)
        return _attn("", rng.choice([H_8B, H_32B, H_TP8, H_14B, H_D64]), "bf16", rng.randint(2, 16),
                     (lo, min(8192, lo * rng.randint(1, 8))), (n0, n0 * rng.randint(1, 4)),
                     rng.choice([0, 16, 16, 32, 64]))
    if kind == "f32":
        P, N = _log_int(rng, 64, 1024), _log_int(rng, 8, 64)
        heads = rng.choice([H_TINY, dict(Hq=8, Hkv=2, d=128), dict(Hq=16, Hkv=8, d=64)])
        return _attn("", heads, "f32", rng.randint(1, 2), (P, P), (N, N), rng.choice([0, 16]))
    if kind == "step1":
        P, N = _log_int(rng, 256, 8192), _log_int(rng, 8, 128)
        return _step("", rng.choice([H_8B, H_14B, H_TP8]), rng.randint(4, 32), 1, (P, P), (N, N),
                     rng.choice([32000, 128256, 152064]), rng.choice([0, 16]))
    if kind == "stepb":
        lo = _log_int(rng, 256, 2048)
        return _step("", rng.choice([H_8B, H_32B, H_TP8]), rng.randint(1, 4), rng.randint(2, 8),
                     (lo, 4 * lo), (8, rng.randint(16, 96)), rng.choice([32000, 128256, 152064]),
                     rng.choice([16, 32]))
    if kind == "sampling":
        n = _log_int(rng, 8, 128)
        return dict(kind="sampling", B=rng.randint(1, 4), N0=max(1, n // 2), N1=n,
                    voc=rng.choice([32000, 128256, 152064]), T=rng.choice([0.6, 0.8, 1.0]))
    return dict(kind="draft", B=rng.randint(1, 16), levels=rng.randint(2, 6),
                voc=rng.choice([32000, 128256, 152064]))


# ------------------------------------------------------------------ inputs

def _beam_tree(r, n):
    """A draft tree of n nodes: a width-10 beam whose children's probabilities fall off steeply, cut to
    the n most probable candidates and listed level by level.  Returns parents (parents[0] = -1)."""
    par, lvl, score, leaves = [-1], [0], [0.0], [0]
    while len(par) < max(2 * n, 411):
        new = []
        for leaf in leaves:
            p = np.sort(r.dirichlet(np.full(BEAM + 1, 0.5)))[::-1][:BEAM]
            for x in np.log(np.maximum(p, 1e-300)):
                new.append(len(par))
                par.append(leaf)
                lvl.append(lvl[leaf] + 1)
                score.append(score[leaf] + float(x))
        leaves = sorted(new, key=lambda j: -score[j])[:BEAM]
    keep = sorted(sorted(range(len(par)), key=lambda j: (-score[j], j))[:n],
                  key=lambda j: (lvl[j], -score[j]))
    at = {old: k for k, old in enumerate(keep)}
    return [-1] + [at[par[j]] for j in keep[1:]]


def _ragged(r, lo, hi, B):
    """B sizes spread evenly over [lo, hi], odd ones among them (the same ones for every seed, so that
    every pass is the same work), in the seed's order."""
    return [int(lo + (hi - lo) * (i + 0.5) / B) for i in r.permutation(B)]


def _trees(case, seed):
    """Sizes, parents [B][Nmax] and tokens with distinct siblings, on the host."""
    r = np.random.default_rng(seed)
    B, voc, nmax = case["B"], case.get("voc", 128256), case["N1"]
    ns = _ragged(r, case["N0"], case["N1"], B)
    par = np.full((B, nmax), -1, np.int32)
    tok = r.integers(0, voc, (B, nmax)).astype(np.int32)
    for b, n in enumerate(ns):
        par[b, :n] = _beam_tree(r, n)
        for u in range(n):
            kids = np.nonzero(par[b, :n] == u)[0]
            if len(kids):
                tok[b, kids] = r.choice(voc, size=len(kids), replace=False)
    return r, ns, par, tok


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7919 + 17)
    return g


def _randn(g, shape, dtype=torch.float32, std=1.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)


def _i32(a):
    return torch.as_tensor(np.asarray(a, np.int32), device="cuda")


def _cache(case, seed, layers):
    """Prefixes, trees, caches of `layers` layers, queries, outputs and the workspace: what a decoder
    holds for the attention calls of one verification."""
    r, ns, par, tok = _trees(case, seed)
    g = _gen(seed)
    B, Hq, Hkv, d, bs = (case[k] for k in ("B", "Hq", "Hkv", "d", "block"))
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    P = _ragged(r, case["P0"], case["P1"], B)
    rows = [P[b] + ns[b] for b in range(B)]
    s = dict(P=P, ns=ns, par_h=par, prefix=_i32(P), parents=_i32(par), n_nodes=_i32(ns),
             tokens=_i32(tok), tok_h=tok, max_prefix=max(P), layers=layers, table=None, blocks=0)
    if bs:
        per = [-(-x // bs) for x in rows]
        s["blocks"] = sum(-(-x // bs) for x in P) + sum(-(-x // bs) for x in ns)
        perm = r.permutation(s["blocks"]).astype(np.int32)
        table = np.zeros((B, max(per)), np.int32)
        at = 0
        for b, n in enumerate(per):
            table[b, :n] = perm[at:at + n]
            at += n
        s["table_h"], s["table"] = table, _i32(table)
        shape = (layers, s["blocks"], Hkv, bs, d)
    else:
        # capacity for this step and the tokens it may accept, as a decoder allocates it
        shape = (layers, B, Hkv, -(-(max(P) + max(ns)) // 64) * 64, d)
    s["k"] = torch.empty(shape, dtype=dtype, device="cuda")
    s["v"] = torch.empty(shape, dtype=dtype, device="cuda")
    for x in range(layers):
        s["k"][x] = _randn(g, shape[1:], dtype)
        s["v"][x] = _randn(g, shape[1:], dtype)
    nmax = par.shape[1]
    # scaled scores spread over a few units, as attention scores do
    s["q"] = _randn(g, (layers, B, nmax, Hq, d), dtype, 1.5)
    s["out"] = torch.zeros((layers, B, nmax, Hq, d), dtype=dtype, device="cuda")
    code = ltd.DTYPE_BF16 if case["dtype"] == "bf16" else ltd.DTYPE_F32
    s["ws"] = torch.empty(max(1, ltd.attn_workspace_size(B, nmax, Hq, Hkv, d, max(P), code)),
                          dtype=torch.uint8, device="cuda")
    return s, r, g


def _target_logits(s, r, g, voc):
    """Target logits N(0, 1) with each node's prediction raised: with probability 0.7 one of its
    children's tokens (the draft was right), else a token that no child carries."""
    B, nmax = s["par_h"].shape
    lg = _randn(g, (B, nmax, voc))
    pick = r.integers(0, voc, (B, nmax))
    for b, n in enumerate(s["ns"]):
        for u in range(n):
            kids = np.nonzero(s["par_h"][b, :n] == u)[0]
            if len(kids) and r.random() < 0.7:
                pick[b, u] = s["tok_h"][b, r.choice(kids)]
    lg.scatter_(2, torch.as_tensor(pick, device="cuda")[:, :, None], lg.amax(2, keepdim=True) + 1)
    return lg


def _mlp(g, dims):
    out = []
    for i, o in zip(dims[:-1], dims[1:]):
        k = 1.0 / math.sqrt(i)
        out.append(tuple((torch.rand(sh, generator=g, device="cuda") * 2 - 1) * k for sh in ((o, i), (o,))))
    return out


def _zeros(*shape, dtype=torch.int32):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("attn", "step"):
        s, r, g = _cache(case, seed, case.get("layers", 1))
        s["kind"] = kind
        # a decoder holds views of each layer's caches and buffers
        s["per_layer"] = [(s["q"][x], s["k"][x], s["v"][x], s["out"][x]) for x in range(s["layers"])]
        if kind == "step":
            B, nmax = s["par_h"].shape
            s["logits"] = _target_logits(s, r, g, case["voc"])
            s["pred"], s["acc"], s["toks"] = (_zeros(B, nmax) for _ in range(3))
            s["nacc"], s["new_len"] = _zeros(B), _zeros(B)
            s["ws_acc"] = torch.empty(max(1, ltd.accept_workspace_size(B, nmax, case["voc"])),
                                      dtype=torch.uint8, device="cuda")
            s["stride"] = s["k"][0].numel()
        return s
    if kind == "sampling":
        r, ns, par, tok = _trees(case, seed)
        g = _gen(seed)
        B, nmax, voc = case["B"], case["N1"], case["voc"]
        lg = _randn(g, (B, nmax, voc), std=3.0)
        q = torch.zeros((B, nmax, voc), device="cuda")
        # a node's children are drawn without replacement from its draft distribution, which is near
        # the target's; tokens ascend in draw order, as a drafter lists them
        for b, n in enumerate(ns):
            for u in range(n):
                kids = np.nonzero(par[b, :n] == u)[0]
                if len(kids):
                    l = lg[b, u] + _randn(g, (voc,))
                    q[b, u] = torch.softmax(l / case["T"], 0)
                    e = -torch.log(-torch.log(torch.rand(voc, generator=g, device="cuda").clamp(1e-20, 1 - 1e-7)))
                    top = torch.topk(torch.log(q[b, u].clamp_min(1e-38)) + e, len(kids)).indices
                    tok[b, kids] = top.cpu().numpy()
        uni = torch.rand((B, nmax, 2), generator=g, device="cuda")
        ws = torch.empty(max(1, ltd.accept_sampling_workspace_size(B, nmax, voc)), dtype=torch.uint8,
                         device="cuda")
        return dict(kind=kind, logits=lg, q=q, tokens=_i32(tok), parents=_i32(par), n_nodes=_i32(ns),
                    uni=uni, T=case["T"], ws=ws, acc=_zeros(B, nmax), toks=_zeros(B, nmax), nacc=_zeros(B))
    g = _gen(seed)
    B, voc, pool = case["B"], case["voc"], 1024
    s = dict(kind=kind, B=B)
    # draft logits: a broad body and, at each node, thirty likely continuations
    s["logits"] = []
    for x in range(case["levels"] - 1):
        lg = _randn(g, (B, BEAM if x else 1, voc), std=2.0)
        at = torch.randint(0, voc, (B, lg.shape[1], 1), generator=g, device="cuda")
        at = (at + 1021 * torch.arange(30, device="cuda")) % voc  # distinct
        up = 12.0 - 1.5 * torch.log(torch.arange(1, 31, device="cuda", dtype=torch.float32))
        lg.scatter_add_(2, at, up.expand_as(at) * 0.7)
        s["logits"].append(lg)
    s["scores"] = _zeros(B, pool, dtype=torch.float32)
    s["pp"], s["pt"] = _zeros(B, pool), _zeros(B, pool)
    s["pp"][:, 0] = -1
    s["size"], s["root"] = _zeros(B), _zeros(B, 1)
    s["fronts"] = [_zeros(B, BEAM) for _ in s["logits"]]
    s["ctx"] = torch.randint(128, 16385, (B,), generator=g, device="cuda", dtype=torch.int32)
    s["depths"] = [torch.full((B,), x + 2, dtype=torch.int32, device="cuda") for x in range(case["levels"] - 1)]
    s["dnet"], s["snet"] = _mlp(g, DEPTH_DIMS), _mlp(g, SIZE_DIMS)
    s["dlog"] = [_zeros(B, 2, dtype=torch.float32) for _ in s["logits"]]
    s["dact"] = [_zeros(B) for _ in s["logits"]]
    s["slog"], s["V"] = _zeros(B, 12, dtype=torch.float32), _zeros(B)
    s["parents"], s["tokens"], s["sel"] = (_zeros(B, MAX_NODES) for _ in range(3))
    s["n"] = _zeros(B)
    size = max(ltd.draft_expand_workspace_size(B, BEAM, voc, BEAM), ltd.policy_workspace_size(B, 1024, 256))
    s["ws"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    return s


# ---------------------------------------------------------------- the calls

def run(s):
    kind = s["kind"]
    if kind in ("attn", "step"):
        for q, k, v, out in s["per_layer"]:
            ltd.tree_verify_attn(q, k, v, s["prefix"], s["parents"], s["n_nodes"], out,
                                 max_prefix=s["max_prefix"], block_table=s["table"],
                                 num_blocks=s["blocks"], workspace=s["ws"])
        if kind == "attn":
            return s["out"]
        ltd.tree_accept(s["logits"], s["tokens"], s["parents"], s["n_nodes"], s["pred"], s["acc"],
                        s["toks"], s["nacc"], workspace=s["ws_acc"])
        ltd.kv_compact(s["k"], s["v"], s["prefix"], s["new_len"], s["acc"], s["nacc"],
                       block_table=s["table"], num_blocks=s["blocks"], num_layers=s["layers"],
                       layer_stride_elems=s["stride"])
        return {k: s[k] for k in ("out", "pred", "acc", "toks", "nacc", "new_len", "k", "v")}
    if kind == "sampling":
        ltd.tree_accept_sampling(s["logits"], s["q"], s["tokens"], s["parents"], s["n_nodes"], s["uni"],
                                 s["acc"], s["toks"], s["nacc"], temperature=s["T"], workspace=s["ws"])
        return {k: s[k] for k in ("acc", "toks", "nacc")}
    s["size"].fill_(1)  # a new cycle starts from the root alone
    front = s["root"]
    for x, lg in enumerate(s["logits"]):
        ltd.draft_expand(lg, front, s["scores"], s["pp"], s["pt"], s["size"], s["fronts"][x], W=BEAM,
                         workspace=s["ws"])
        front = s["fronts"][x]
        ltd.policy_forward(ltd.POLICY_DEPTH, s["scores"], s["size"], s["depths"][x], s["ctx"], s["dnet"],
                           s["dlog"][x], s["dact"][x], pad=PAD, workspace=s["ws"])
    ltd.policy_forward(ltd.POLICY_SIZE, s["scores"], s["size"], s["depths"][-1], s["ctx"], s["snet"],
                       s["slog"], s["V"], pad=PAD, action_offset=20, action_scale=20, workspace=s["ws"])
    ltd.select_candidates(s["scores"], s["pp"], s["pt"], s["size"], s["V"], s["parents"], s["tokens"],
                          s["n"], selected=s["sel"])
    return {k: s[k] for k in ("scores", "pp", "pt", "size", "fronts", "dlog", "dact", "slog", "V",
                              "parents", "tokens", "sel", "n")}


# ------------------------------------------------------ what a pass cannot do without

def _sizes(case):
    """Mean prefix and tree size of a batch."""
    return 0.5 * (case["P0"] + case["P1"]), 0.5 * (case["N0"] + case["N1"])


def work(case):
    kind = case["kind"]
    if kind in ("attn", "step"):
        P, N = _sizes(case)
        B, Hq, Hkv, d = (case[k] for k in ("B", "Hq", "Hkv", "d"))
        e, L = (2 if case["dtype"] == "bf16" else 4), case.get("layers", 1)
        nbytes = L * B * ((P + N) * Hkv * d * 2 * e + 2 * N * Hq * d * e)
        flops = L * B * 4 * Hq * N * (P + 0.5 * N) * d
        if kind == "step":
            nbytes += B * N * case["voc"] * 4
            flops += B * N * case["voc"]
        return {"bytes": nbytes, "flops": flops}
    if kind == "sampling":
        # the logits of every node, the draft rows of those with children (about a third)
        N = 0.5 * (case["N0"] + case["N1"])
        n = case["B"] * N * case["voc"]
        return {"bytes": n * 4 * 4 / 3, "flops": 4 * n}
    B, voc, x = case["B"], case["voc"], case["levels"] - 1
    rows = 1 + BEAM * (x - 1)
    net = lambda dims: sum(i * o for i, o in zip(dims[:-1], dims[1:]))  # noqa: E731
    return {"bytes": B * rows * voc * 4 + 4 * (net(SIZE_DIMS) + net(DEPTH_DIMS)),
            "flops": 2 * B * (rows * voc + net(SIZE_DIMS) + x * net(DEPTH_DIMS))}


def tolerance(case):
    kind = case["kind"]
    if kind == "sampling":
        return "exact"  # whole numbers; a decision moves only where a uniform meets its threshold
    if kind == "draft":
        return {"rel": 1e-6, "max": 4e-6, "differ": 0.0}
    return {"rel": 1.2e-2, "max": 6e-2, "differ": 0.0} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}


# ------------------------------------------------------------ 64-bit results

def _rows64(case, s, x, cache, b):
    """Rows [0, P + N) of layer x's cache for sequence b, as [Hkv][rows][d] in 64 bits."""
    n = s["P"][b] + s["ns"][b]
    if s["table"] is None:
        return cache[x, b, :, :n].double()
    ids = torch.as_tensor(s["table_h"][b, :-(-n // case["block"])].astype(np.int64), device="cuda")
    return cache[x, ids].double().permute(1, 0, 2, 3).reshape(case["Hkv"], -1, case["d"])[:, :n].contiguous()


def _attn64(case, s):
    out = torch.zeros(s["out"].shape, dtype=torch.float64, device="cuda")
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    G = Hq // Hkv
    for b, (P, n) in enumerate(zip(s["P"], s["ns"])):
        seen = np.zeros((n, n), bool)
        for i in range(n):
            if i:
                seen[i] = seen[s["par_h"][b, i]]
            seen[i, i] = True
        hide = ~torch.as_tensor(seen, device="cuda").repeat_interleave(G, 0)
        for x in range(s["layers"]):
            k, v = _rows64(case, s, x, s["k"], b), _rows64(case, s, x, s["v"], b)
            for h in range(Hkv):
                q = s["q"][x, b, :n, h * G:(h + 1) * G].double().reshape(n * G, d)
                w = (q @ k[h].t().contiguous()) * d ** -0.5
                w[:, P:].masked_fill_(hide, float("-inf"))
                out[x, b, :n, h * G:(h + 1) * G] = (torch.softmax(w, 1) @ v[h]).reshape(n, G, d)
    return out


def _accept(s, lg):
    """Predictions and the longest accepted root path of each tree, on the host."""
    pred = lg.argmax(2).cpu().numpy()
    got = {k: np.zeros(s["par_h"].shape, np.int64) for k in ("pred", "acc", "toks")}
    nacc = []
    for b, n in enumerate(s["ns"]):
        depth, best = [0] * n, 0
        for c in range(1, n):
            u = s["par_h"][b, c]
            fits = depth[u] >= 0 and s["tok_h"][b, c] == pred[b, u]
            depth[c] = depth[u] + 1 if fits else -1
            best = c if depth[c] > depth[best] else best
        path = [best]
        while path[0]:
            path.insert(0, int(s["par_h"][b, path[0]]))
        got["pred"][b, :n] = pred[b, :n]
        got["acc"][b, :len(path)] = path
        got["toks"][b, :len(path)] = [s["tok_h"][b, c] for c in path[1:]] + [pred[b, best]]
        nacc.append(len(path))
    return got, nacc


def exact(case, seed):
    kind = case["kind"]
    if kind == "sampling":
        return None  # whole numbers alone
    s = prepare(case, seed)
    if kind == "draft":
        return _draft64(case, s)
    out = _attn64(case, s)
    if kind == "attn":
        return out
    got, nacc = _accept(s, s["logits"])
    k, v = s["k"], s["v"]
    for b, n in enumerate(nacc):
        path = got["acc"][b, :n]
        P = s["P"][b]
        for c in (k, v):
            if s["table"] is None:
                c[:, b, :, P:P + n] = c[:, b][:, :, torch.as_tensor(P + path, device="cuda")].clone()
            else:
                bs = case["block"]
                at = lambda rows: (torch.as_tensor(s["table_h"][b, rows // bs].astype(np.int64), device="cuda"),  # noqa: E731
                                   torch.as_tensor(rows % bs, device="cuda"))
                i, o = at(P + path)
                moved = c[:, i, :, o].clone()
                i, o = at(P + np.arange(n))
                c[:, i, :, o] = moved
    return {"out": out, **got, "nacc": np.array(nacc), "new_len": np.array(s["P"]) + nacc, "k": k.float(),
            "v": v.float()}


def _policy64(net, state):
    x = state
    for i, (w, b) in enumerate(net):
        x = x @ w.double().t().contiguous() + b.double()
        x = x.clamp_min(0) if i + 1 < len(net) else x
    return x


def _draft64(case, s):
    B = s["B"]
    scores = torch.zeros((B, s["scores"].shape[1]), dtype=torch.float64, device="cuda")
    rows = torch.arange(B, device="cuda")
    front, size, dlog = torch.zeros((B, 1), dtype=torch.int64, device="cuda"), 1, []
    for x, lg in enumerate(s["logits"]):
        F = lg.shape[1]
        top = torch.sort(lg, dim=2, descending=True, stable=True).values[:, :, :BEAM].double()
        kids = scores[rows[:, None], front][:, :, None] + top - torch.logsumexp(lg.double(), 2, keepdim=True)
        kids = kids.reshape(B, F * BEAM)
        scores[:, size:size + F * BEAM] = kids
        front = size + torch.sort(kids.float(), dim=1, descending=True, stable=True).indices[:, :BEAM]
        size += F * BEAM
        w = DEPTH_DIMS[0] - 2
        state = torch.full((B, w + 2), PAD, dtype=torch.float64, device="cuda")
        m = min(w, size)
        state[:, w - m:w] = scores[:, size - m:size].float().double()
        state[:, w], state[:, w + 1] = s["depths"][x].double(), s["ctx"].double()
        dlog.append(_policy64(s["dnet"], state))
    state = torch.full((B, SIZE_DIMS[0]), PAD, dtype=torch.float64, device="cuda")
    state[:, 0], state[:, 1] = s["depths"][-1].double(), s["ctx"].double()
    state[:, 2:2 + size] = scores[:, :size].float().double()
    return {"scores": scores, "dlog": dlog, "slog": _policy64(s["snet"], state), "pp": None, "pt": None,
            "size": None, "fronts": None, "dact": None, "V": None, "parents": None, "tokens": None,
            "sel": None, "n": None}


if __name__ == "__main__":  # each case once
    for c in listed() + [draw(random.Random(k)) for k in range(4)]:
        st = prepare(c, 1)
        run(st)
        torch.cuda.synchronize()
        print(c.get("name", c), work(c), flush=True)
