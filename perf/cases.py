"""The verification path's work at the sizes a serving engine gives it.

One decoding step of an engine drafts a tree per request, then runs the gate
(which draft nodes to verify), flatten & pack (their slots and masks), the
attention of every layer, and the acceptance; a paged engine also commits the
accepted rows to its cache.  The cases are that step in one call at five model
and batch shapes, one layer's attention in the forms an engine calls it in
(paged, decode only), the other gate policies, and the end of the step from the
model's logits.  Sizes are those of the workload presets; what ``draw`` gives
lies in the ranges that they span, odd and ragged sizes among them.
"""
import functools
import math

import numpy as np
import torch

import paper_2604_09603_amd as echo

D = echo.HEAD_DIM
MAX_DEPTH = echo.MAX_DEPTH
DEV = "cuda:0"

# What a drawn case may cost at most: the listed cases' largest cache, products,
# candidate pool and logits.
MAX_KV_BYTES = 1.25e9
MAX_FLOPS = 1.6e11
MAX_POOL = 90880
MAX_LOGITS = 384 * 151936


def _case(kind, name=None, **kw):
    c = dict(kind=kind, R=32, depth=6, branch=8, ragged=False, sigma=3.0, vocab=128256, budget=128,
             hq=32, hkv=8, p_lo=512, p_hi=2048, q_scale=1.0, page=64, seed_salt=0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a few interactive users of a small model: five launches' latency
        _case("step", "step_tiny", R=4, depth=4, branch=4, sigma=2.0, vocab=32, budget=16, hq=8,
              hkv=8, p_lo=256, p_hi=256),
        # an 8B-class model (32 query / 8 KV heads), a batch of 32 chats
        _case("step", "step_8b"),
        # a 70B-class model (64 / 8 heads), a batch of 64
        _case("step", "step_70b", R=64, depth=8, budget=256, hq=64, p_lo=1024, p_hi=4096),
        # a 235B-class mixture of experts (64 / 4 heads), high concurrency: the benchmark's default
        _case("step", "step_235b", R=128, depth=8, branch=10, vocab=151936, budget=256, hq=64,
              hkv=4, p_lo=1024, p_hi=8192),
        # the same model on long documents: few requests, many verified nodes each
        _case("step", "step_long", R=16, depth=10, branch=6, sigma=4.0, vocab=151936, budget=192,
              hq=64, hkv=4, p_lo=16384, p_hi=32768),
        # one GPU's share of the 235B layer under 4-way tensor parallelism: one KV head
        _case("step", "step_235b_tp4", R=128, depth=8, branch=10, vocab=151936, budget=256, hq=16,
              hkv=1, p_lo=1024, p_hi=8192),
        # one layer's attention over a paged cache: what an engine calls once per layer;
        # sharper queries, trees cut at different depths, an odd batch
        _case("attn_paged", "attn_paged_70b", R=61, depth=8, ragged=True, budget=251, hq=64,
              p_lo=1000, p_hi=4096, q_scale=2.0),
        # one layer's attention in plain decoding (no drafts), one query head per KV head
        _case("attn", "attn_decode_g1", R=64, depth=4, branch=4, sigma=2.0, vocab=32000, budget=0,
              hq=8, hkv=8, p_lo=1024, p_hi=8192),
        # Alg. 1's elastic scheduler and flatten & pack on the largest pool
        _case("front_elastic", "front_elastic_235b", R=128, depth=8, branch=10, vocab=151936,
              budget=256, p_lo=1024, p_hi=8192),
        # checkpoint gating and flatten & pack on a 70B batch's pool
        _case("front_sparse", "front_sparse_70b", R=64, depth=8, ragged=True, budget=256,
              p_lo=1024, p_hi=4096),
        # the end of a serving step: argmax of the logits, acceptance, commit to the pages
        _case("accept_commit", "accept_commit_235b", R=128, depth=8, branch=10, vocab=151936,
              budget=256, hq=64, hkv=4, p_lo=64, p_hi=512),
        # a whole serving step of the 8B-class model over a paged cache
        _case("serve", "serve_8b", ragged=True),
    ]


HEADS = [(8, 8), (16, 8), (32, 8), (64, 8), (64, 4), (32, 4), (16, 2), (16, 1), (8, 1)]
KINDS = ["step"] * 5 + ["attn_paged", "attn_paged", "attn", "attn", "front_elastic", "front_sparse",
                        "accept_commit", "serve"]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(KINDS)
    R = log_int(3, 128)
    depth, branch = rng.randint(3, 10), rng.randint(3, 10)
    while R * (branch + (depth - 1) * branch * branch) > MAX_POOL:
        branch -= 1
    budget = 0 if kind == "attn" and rng.random() < 0.3 else log_int(8, 256)
    budget = min(budget, 384 - R)
    hq, hkv = rng.choice(HEADS)
    p_hi = log_int(48, 32768)
    p_hi = int(min(p_hi, MAX_KV_BYTES / (R * hkv * 512), MAX_FLOPS / (512.0 * hq * (R + budget))))
    p_hi = max(p_hi, 33)
    p_lo = rng.randint(max(1, p_hi // 8), p_hi)
    vocab = min(log_int(1000, 151936), MAX_LOGITS // (R + budget))
    if kind in ("accept_commit",):
        p_hi = min(p_hi, 1024)
        p_lo = min(p_lo, p_hi)
    return _case(kind, R=R, depth=depth, branch=branch, ragged=rng.random() < 0.5,
                 sigma=rng.choice([2.0, 3.0, 4.0]), vocab=vocab, budget=budget, hq=hq, hkv=hkv,
                 p_lo=p_lo, p_hi=p_hi, q_scale=rng.choice([1.0, 1.0, 2.0]),
                 page=rng.choice([32, 64, 128, 256]), seed_salt=rng.randrange(1 << 20))


# ---- inputs ---------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _template(depth, branch):
    """Parents, depths and expanded nodes of one request's full drafted tree: the root's
    `branch` children, then per depth the children of the `branch` nodes that come first
    in the order (frontier rank of the parent + sibling rank, sibling rank, parent rank)."""
    k = branch
    parent, dep, expanded = [-1] * k, [1] * k, [-1]
    level = [(i, 0, i) for i in range(k)]
    for d in range(2, depth + 1):
        level.sort(key=lambda t: (t[1] + t[2], t[2], t[1]))
        nxt = []
        for rank, (f, _, _) in enumerate(level[:k]):
            expanded.append(f)
            for c in range(k):
                nxt.append((len(parent), rank, c))
                parent.append(f)
                dep.append(d)
        level = nxt
    return np.array(parent, np.int32), np.array(dep, np.int32), np.array(expanded, np.int32)


def _top_logq(rng, n, k, vocab, sigma):
    """log-softmax of the k largest of `vocab` logits N(0, 1) * sigma, n times: the order
    statistics through their joint law (ratios of uniforms), the rest of the sum by its
    mean below the k-th."""
    k = min(k, vocab)
    u = rng.random((n, k)) ** (1.0 / (vocab - np.arange(k)))
    u = np.minimum(np.cumprod(u, axis=1), 1.0 - 1e-12)
    z = torch.special.ndtri(torch.from_numpy(u)).numpy()
    below = torch.special.ndtr(torch.from_numpy(z[:, -1] - sigma)).numpy()
    rest = (vocab - k) * math.exp(0.5 * sigma * sigma) * below
    lse = np.log(np.exp(sigma * z).sum(axis=1) + rest)
    return (sigma * z - lse[:, None]).astype(np.float32)


def _pool(case, rng):
    """The drafted candidate pool (request-major) and the target token after every node."""
    R, k, V = case["R"], case["branch"], case["vocab"]
    par, dep, expanded = _template(case["depth"], k)
    offs, cols = np.zeros(R + 1, np.int32), {x: [] for x in ("parent", "token", "logq", "target", "depth")}
    root_token = rng.integers(0, V, R).astype(np.int32)
    root_target = np.empty(R, np.int32)
    # how deep each request's draft went: the case's own, so that its sizes are too
    depths = np.full(R, case["depth"])
    if case["ragged"]:
        depths = np.random.default_rng([case["seed_salt"], 5]).integers(
            max(1, case["depth"] // 2), case["depth"] + 1, R)
    for r in range(R):
        d = int(depths[r])
        ne = 1 + (d - 1) * k
        n = ne * k
        logq = np.full((ne, k), -np.inf, np.float32)
        top = _top_logq(rng, ne, k, V, case["sigma"])
        logq[:, :top.shape[1]] = top
        token = (rng.integers(0, V, (ne, 1)) + np.arange(k) * 7).astype(np.int64) % V
        p_accept = rng.beta(6.0, 3.0)
        target = rng.integers(0, V, n + 1)
        hit = rng.random(n + 1) < p_accept
        ex = expanded[:ne] + 1  # 0: the root
        target[ex] = np.where(hit[ex], token[:, 0], target[ex])
        root_target[r] = target[0]
        offs[r + 1] = offs[r] + n
        for x, v in (("parent", par[:n]), ("token", token.ravel()), ("logq", logq.ravel()),
                     ("target", target[1:]), ("depth", dep[:n])):
            cols[x].append(v)
    out = {x: np.concatenate(v).astype(np.float32 if x == "logq" else np.int32) for x, v in cols.items()}
    return dict(out, cand_offsets=offs, root_token=root_token, root_target=root_target)


def _checkpoints(case):
    """(depth, ln tau) of the checkpoints: about half of the requests stop at each."""
    return [(d, -3.0 - 2.6 * (d - 1)) for d in (1, 3, 5) if d <= case["depth"]]


def _scores(pool):
    """Path scores, one binary32 add per level, and the same in float64."""
    par = pool["parent"].astype(np.int64)
    sizes = np.diff(pool["cand_offsets"])
    start = np.repeat(pool["cand_offsets"][:-1].astype(np.int64), sizes)
    s32, s64 = pool["logq"].copy(), pool["logq"].astype(np.float64)
    for d in range(2, int(pool["depth"].max(initial=1)) + 1):
        i = np.nonzero(pool["depth"] == d)[0]
        g = start[i] + par[i]
        s32[i] = s32[g] + pool["logq"][i]
        s64[i] = s64[g] + pool["logq"][i].astype(np.float64)
    return s32, s64


def _slots(case, pool, prefix_len):
    """The top-B selection of the pool, flattened: offsets, slots and masks."""
    R, B = case["R"], case["budget"]
    s32, s64 = _scores(pool)
    finite = np.nonzero(np.isfinite(s32))[0]
    order = finite[np.lexsort((finite, -s32[finite].astype(np.float64)))][:B]
    sel = np.sort(order)
    cap, W = R + B, (B + 1 + 31) // 32
    offs = pool["cand_offsets"]
    m = {x: np.zeros(cap, np.int32) for x in ("slot_cand", "slot_parent", "slot_token", "position_ids",
                                              "target")}
    q_offsets = np.zeros(R + 1, np.int32)
    mask = np.zeros((cap, W), np.uint32)
    s = 0
    for r in range(R):
        mine = sel[np.searchsorted(sel, offs[r]):np.searchsorted(sel, offs[r + 1])]
        local = {int(g) - int(offs[r]): j + 1 for j, g in enumerate(mine)}
        for j in range(len(mine) + 1):
            g = -1 if j == 0 else int(mine[j - 1])
            p = -1 if j == 0 else local.get(int(pool["parent"][g]), 0)
            m["slot_cand"][s], m["slot_parent"][s] = g, p
            m["slot_token"][s] = pool["root_token"][r] if j == 0 else pool["token"][g]
            m["target"][s] = pool["root_target"][r] if j == 0 else pool["target"][g]
            m["position_ids"][s] = prefix_len[r] + (0 if j == 0 else pool["depth"][g])
            if j > 0:
                mask[s] = mask[s - j + p]
            mask[s, j >> 5] |= np.uint32(1 << (j & 31))
            s += 1
        q_offsets[r + 1] = s
    return dict(m, q_offsets=q_offsets, tree_mask=mask.view(np.int32), s64=s64, nq=s)


HAS_ATTENTION = ("step", "attn", "attn_paged", "serve")
HAS_PAGES = ("attn_paged", "accept_commit", "serve")


def _inputs(case, seed):
    """Everything drawn for a case, from the seed alone: the pool and lengths on the host, the
    attention's tensors and the logits on the GPU."""
    rng = np.random.default_rng([seed, case["seed_salt"], 11])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(rng.integers(1 << 62)))
    R, cap = case["R"], case["R"] + case["budget"]
    pool = _pool(case, rng)
    P = rng.integers(case["p_lo"], case["p_hi"] + 1, R).astype(np.int32)
    x = dict(pool=pool, P=P, slots=_slots(case, pool, P))
    kv_offsets = np.zeros(R + 1, np.int64)
    kv_offsets[1:] = np.cumsum(P.astype(np.int64))
    x["kv_offsets"] = kv_offsets

    def normal(*shape, scale=1.0):
        t = torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, 1.0, generator=gen)
        return t if scale == 1.0 else t.mul_(scale)

    if case["kind"] in HAS_ATTENTION:
        x["q"] = normal(cap, case["hq"], D, scale=case["q_scale"])
    if case["kind"] in HAS_ATTENTION or case["kind"] in HAS_PAGES:
        T = int(kv_offsets[-1])
        for n in ("k", "v"):
            x[n + "_new"] = normal(cap, case["hkv"], D)
            x[n + "_cache"] = normal(T, case["hkv"], D)
    if case["kind"] in HAS_PAGES:
        # the prefixes over shuffled pages of a pool for R requests of the longest
        # prefix, with room for one step's commits
        S = case["page"]
        npg = (P.astype(np.int64) + MAX_DEPTH + S) // S
        most = (case["p_hi"] + MAX_DEPTH + S) // S
        total = R * most
        perm = rng.permutation(total)
        bt = np.full((R, most), -1, np.int32)
        dest = np.empty(int(kv_offsets[-1]), np.int64)
        at = 0
        for r in range(R):
            ids = perm[at:at + npg[r]]
            at += int(npg[r])
            bt[r, :npg[r]] = ids
            pos = np.arange(P[r])
            dest[kv_offsets[r]:kv_offsets[r + 1]] = ids[pos // S] * S + pos % S
        x["block_table"] = bt
        dest = torch.from_numpy(dest).to(DEV)
        for n in ("k", "v"):
            pages = torch.zeros((total * S, case["hkv"], D), dtype=torch.bfloat16, device=DEV)
            pages[dest] = x[n + "_cache"]
            x[n + "_pages"] = pages.view(total, S, case["hkv"], D)
    if case["kind"] in ("accept_commit", "serve"):
        logits = normal(cap, case["vocab"])
        top = torch.from_numpy(x["slots"]["target"].astype(np.int64)).to(DEV)
        logits.scatter_(1, top[:, None], 9.0)
        x["logits"] = logits
    return x


# ---- the calls ------------------------------------------------------------

def _workspace(nbytes):
    raw = torch.empty(max(int(nbytes), 1) + 256, dtype=torch.uint8, device=DEV)
    off = (-raw.data_ptr()) % 256
    return raw[off:off + max(int(nbytes), 1)]


def prepare(case, seed):
    x = _inputs(case, seed)
    kind, R, B, hq, hkv = case["kind"], case["R"], case["budget"], case["hq"], case["hkv"]
    pool, slots = x["pool"], x["slots"]
    cap, W, N = R + B, (B + 1 + 31) // 32, len(pool["logq"])
    s = dict(kind=kind, R=R, B=B, N=N, cap=cap, W=W, hq=hq, hkv=hkv, page=case["page"],
             kv_rows=int(x["kv_offsets"][-1]), sm_scale=1.0 / math.sqrt(D),
             w_max=case["branch"], depths=[d for d, _ in _checkpoints(case)],
             taus=[t for _, t in _checkpoints(case)])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    i32 = lambda *shape: torch.zeros(shape, dtype=torch.int32, device=DEV)  # noqa: E731
    for n in ("cand_offsets", "parent", "token", "logq", "root_token"):
        s[n] = dev(pool[n])
    s["prefix_len"], s["kv_offsets"] = dev(x["P"]), dev(x["kv_offsets"])
    for n in ("q", "k_new", "v_new", "k_cache", "v_cache", "k_pages", "v_pages"):
        if n in x and not (n.endswith("_cache") and kind in HAS_PAGES):
            s[n] = x[n].view(torch.int16)
    s["status"] = i32(1)
    s["target"] = dev(slots["target"])
    if kind in HAS_PAGES:
        s["block_table"], s["cached_len"] = dev(x["block_table"]), dev(x["P"])
    if "logits" in x:
        s["logits"] = x["logits"].view(torch.int16)
    # outputs and workspaces, kept from step to step
    fronts = ("step", "serve", "front_sparse", "front_elastic")
    s["path_score"] = torch.zeros(N, dtype=torch.float32, device=DEV)
    s["selected"] = torch.zeros(N, dtype=torch.uint8, device=DEV)
    s["num_selected"], s["trunc_depth"] = i32(1), i32(R)
    for n in ("slot_cand", "slot_parent", "slot_token", "position_ids"):
        s[n] = i32(cap) if kind in fronts else dev(slots[n])
    s["q_offsets"] = i32(R + 1) if kind in fronts else dev(slots["q_offsets"])
    s["tree_mask"] = i32(cap, W) if kind in fronts else dev(slots["tree_mask"])
    s["accept_len"], s["accept_slots"], s["bonus"] = i32(R), i32(R, MAX_DEPTH), i32(R)
    s["target_out"] = i32(cap)
    if kind in fronts:
        size = echo.gate_elastic_workspace_size if kind == "front_elastic" else echo.gate_workspace_size
        s["gate_ws"] = _workspace(size(R, N, B))
    if kind in HAS_ATTENTION:
        s["out"] = torch.zeros((cap, hq, D), dtype=torch.float32, device=DEV)
        s["lse"] = torch.zeros((cap, hq), dtype=torch.float32, device=DEV)
        s["attn_ws"] = _workspace(echo.tree_verify_attn_workspace_size(R, cap, hq, hkv))
    return s


FRONT = ("path_score", "selected", "num_selected")
SLOTS = ("q_offsets", "slot_cand", "slot_parent", "slot_token", "position_ids", "tree_mask")
ACCEPT = ("accept_len", "accept_slots", "bonus")
PAGES = ("target_out", "cached_len", "k_pages", "v_pages")
OUTPUTS = {
    "step": FRONT + SLOTS + ("out", "lse") + ACCEPT + ("status",),
    "attn": ("out", "lse", "status"),
    "attn_paged": ("out", "lse", "status"),
    "front_elastic": FRONT + ("trunc_depth",) + SLOTS + ("status",),
    "front_sparse": FRONT + ("trunc_depth",) + SLOTS + ("status",),
    "accept_commit": ACCEPT + PAGES + ("status",),
    "serve": FRONT + SLOTS + ("out", "lse") + ACCEPT + PAGES + ("status",),
}


def _mask(s):
    echo.echo_build_tree_mask(
        s["cand_offsets"], s["parent"], s["token"], s["selected"], s["root_token"], s["prefix_len"],
        s["R"], s["N"], s["B"], s["q_offsets"], s["slot_cand"], s["slot_parent"], s["slot_token"],
        s["position_ids"], s["tree_mask"], s["W"], status=s["status"])


def _attn_paged(s):
    echo.echo_tree_verify_attn_paged(
        s["q"], s["k_new"], s["v_new"], s["k_pages"], s["v_pages"], s["page"], s["block_table"],
        s["cached_len"], s["q_offsets"], s["tree_mask"], s["W"], s["R"], s["cap"], s["hq"], s["hkv"],
        D, s["sm_scale"], s["out"], s["lse"], s["attn_ws"], status=s["status"])


def _accept_commit(s):
    echo.echo_accept_logits(
        s["q_offsets"], s["slot_parent"], s["slot_token"], s["logits"], s["R"], s["cap"], MAX_DEPTH,
        s["target_out"], s["accept_len"], s["accept_slots"], s["bonus"], status=s["status"])
    echo.echo_commit_kv(
        s["q_offsets"], s["accept_len"], s["accept_slots"], MAX_DEPTH, s["k_new"], s["v_new"], s["R"],
        s["cap"], s["hkv"], s["k_pages"], s["v_pages"], s["page"], s["block_table"], s["cached_len"],
        status=s["status"])


def run(s):
    kind = s["kind"]
    if kind == "step":
        echo.echo_verify_step(
            s["cand_offsets"], s["parent"], s["logq"], s["token"], s["R"], s["N"], s["B"],
            s["path_score"], s["selected"], s["num_selected"], s["gate_ws"], s["root_token"],
            s["prefix_len"], s["q_offsets"], s["slot_cand"], s["slot_parent"], s["slot_token"],
            s["position_ids"], s["tree_mask"], s["W"], s["q"], s["k_new"], s["v_new"], s["k_cache"],
            s["v_cache"], s["kv_offsets"], s["kv_rows"], s["cap"], s["hq"], s["hkv"], D,
            s["sm_scale"], s["out"], s["lse"], s["attn_ws"], s["target"], MAX_DEPTH,
            s["accept_len"], s["accept_slots"], s["bonus"], status=s["status"])
    elif kind == "attn":
        echo.echo_tree_verify_attn(
            s["q"], s["k_new"], s["v_new"], s["k_cache"], s["v_cache"], s["kv_offsets"],
            s["kv_rows"], s["q_offsets"], s["tree_mask"], s["W"], s["R"], s["cap"], s["hq"],
            s["hkv"], D, s["sm_scale"], s["out"], s["lse"], s["attn_ws"], status=s["status"])
    elif kind == "attn_paged":
        _attn_paged(s)
    elif kind == "front_elastic":
        echo.echo_gate_elastic(
            s["cand_offsets"], s["parent"], s["logq"], s["R"], s["N"], s["B"], s["depths"],
            s["taus"], 2, s["w_max"], s["path_score"], s["selected"], s["num_selected"],
            s["gate_ws"], trunc_depth=s["trunc_depth"], status=s["status"])
        _mask(s)
    elif kind == "front_sparse":
        echo.echo_gate_sparse(
            s["cand_offsets"], s["parent"], s["logq"], s["R"], s["N"], s["B"], s["depths"],
            s["taus"], s["path_score"], s["selected"], s["num_selected"], s["gate_ws"],
            trunc_depth=s["trunc_depth"], status=s["status"])
        _mask(s)
    elif kind == "accept_commit":
        s["cached_len"].copy_(s["prefix_len"])  # this pass commits the same step again
        _accept_commit(s)
    elif kind == "serve":
        s["cached_len"].copy_(s["prefix_len"])
        echo.echo_gate(s["cand_offsets"], s["parent"], s["logq"], s["R"], s["N"], s["B"],
                       s["path_score"], s["selected"], s["num_selected"], s["gate_ws"],
                       status=s["status"])
        _mask(s)
        _attn_paged(s)
        _accept_commit(s)
    else:
        raise ValueError(kind)
    return {n: s[n] for n in OUTPUTS[kind]}


# ---- what a pass cannot do without, and how far two correct ones may differ ----

def work(case):
    kind, R, B, hq, hkv = case["kind"], case["R"], case["budget"], case["hq"], case["hkv"]
    rows = R + B
    k, d = case["branch"], case["depth"]
    if case["ragged"]:
        d = 0.5 * (max(1, d // 2) + d)
    N = R * (k + (d - 1) * k * k)
    P = 0.5 * (case["p_lo"] + case["p_hi"])
    nbytes = flops = 0.0
    if kind in ("step", "serve", "front_elastic", "front_sparse"):
        # parents, log q and scores; flags; tokens and slots of the selected
        nbytes += N * (4 + 4 + 4 + 1) + rows * (8 + 16 + 4 * ((B + 32) // 32)) + 16 * R
        flops += N
    if kind in HAS_ATTENTION:
        nbytes += R * P * hkv * D * 4 + rows * (hq * (2 * D + 4 * D + 4) + hkv * D * 4)
        flops += 4.0 * D * hq * rows * P
    if kind in ("accept_commit", "serve"):
        nbytes += rows * case["vocab"] * 2 + 3 * R * hkv * D * 8  # about three rows a request
        flops += rows * case["vocab"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Attention's probabilities enter the second product in bf16 (2^-9 each), so the
    # outputs of two correct orders differ by about 1.5e-3 in norm; the rest is whole
    # numbers, copied bits and binary32 sums in a fixed order.
    if case["kind"] in HAS_ATTENTION:
        return {"rel": 6e-3, "max": 5e-2}
    return "exact"


def exact(case, seed):
    if case["kind"] == "accept_commit":
        return None  # whole numbers and copied bits only
    x = _inputs(case, seed)
    got = {n: None for n in OUTPUTS[case["kind"]]}
    sl = x["slots"]
    if "path_score" in got:
        got["path_score"] = sl["s64"]
    if case["kind"] in HAS_ATTENTION:
        hq, hkv, cap = case["hq"], case["hkv"], case["R"] + case["budget"]
        G = hq // hkv
        out = torch.zeros((cap, hq, D), dtype=torch.float64, device=DEV)
        lse = torch.zeros((cap, hq), dtype=torch.float64, device=DEV)
        scale = float(np.float32(1.0 / math.sqrt(D)))
        for r in range(case["R"]):
            a, b = int(sl["q_offsets"][r]), int(sl["q_offsets"][r + 1])
            k0, k1 = int(x["kv_offsets"][r]), int(x["kv_offsets"][r + 1])
            n, P = b - a, k1 - k0
            bits = torch.from_numpy(sl["tree_mask"][a:b].view(np.uint32).astype(np.int64)).to(DEV)
            j = torch.arange(n, device=DEV)
            see = ((bits[:, j >> 5] >> (j & 31)) & 1).bool()           # [n, n]
            see = torch.cat([torch.ones((n, P), dtype=torch.bool, device=DEV), see], 1)
            see = see[:, None, :].expand(n, G, P + n).reshape(n * G, P + n)
            for h in range(hkv):
                K = torch.cat([x["k_cache"][k0:k1, h], x["k_new"][a:b, h]]).double()
                V = torch.cat([x["v_cache"][k0:k1, h], x["v_new"][a:b, h]]).double()
                Q = x["q"][a:b, h * G:(h + 1) * G].double().reshape(n * G, D)
                z = (Q @ K.T.contiguous()) * scale
                z = z.masked_fill(~see, -math.inf)
                lse[a:b, h * G:(h + 1) * G] = torch.logsumexp(z, 1).view(n, G)
                out[a:b, h * G:(h + 1) * G] = (torch.softmax(z, 1) @ V).view(n, G, D)
        got["out"], got["lse"] = out, lse
    return got
