"""What a user of this library has it do, as cases that can be timed: decoding steps, drafting passes, vocabulary
reductions and output projections, through the public calls of paper_2602_00523_amd.sage.

Four kinds of case, each over a range of sizes:
  step     one decoding step: planning of the next tree, tree attention of every layer, the target's greedy tokens,
           acceptance, and (with `commit`) the closing of the step on the device;
  draft    one drafting pass: the draft model's attention, called once per tree level for the new level's rows;
  topk     entropy, top-k and confidence of stored logits (draft rows), or greedy tokens (target rows);
  project  the same straight from an output projection, without stored logits.
`launch` says how the program issues its calls: "direct" (the plain calls, marshalled each time), "prepared"
(sage.prepare, for hot loops) or "graph" (prepared calls captured once as a HIP graph and replayed).

The steps carry their state on the device like a decoding loop does: two tree buffers change roles at every step, the
accepted path joins the cache and the depth limit follows the acceptance history.  The cache has room for a few more
positions than its initial length; once it is full the length stays, so that repeated passes do the same work.
"""
import math
import random

import numpy as np
import torch

from paper_2602_00523_amd import sage, workloads

NODES = sage.MAX_NODES
ROOM = 16                        # cache positions past the initial length
# tree parameters: the paper's, the configurations' narrower and wider ones, and a set that always fills the 64 nodes
# (with the planted candidate distribution of `_draft_rows`)
TREES = {
    "toy": dict(workloads.CONFIGS["toy"]["tree"]),
    "paper": dict(workloads.CONFIGS["c2"]["tree"]),
    "video": dict(workloads.CONFIGS["c3"]["tree"]),
    "full": dict(d_min=31, d_max=31, w_min=16, w_max=16, k=64, n_max=64),
}
MEAN_NODES = {"toy": 8, "paper": 12, "video": 15, "full": 64}       # typical tree sizes under these parameters
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _step(name, *, dtype="bf16", B=1, Hq=64, Hkv=8, d=128, kv_lo, kv_hi, vocab=152064, layers=1, tree="paper", entropy=2.0,
          commit=True, launch="prepared"):
    return dict(name=name, kind="step", dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, d=d, kv_lo=kv_lo, kv_hi=kv_hi, vocab=vocab,
                layers=layers, tree=tree, entropy=entropy, commit=commit, launch=launch)


def _draft(name, *, Hq=28, Hkv=4, kv, nodes, spread=6, launch="graph"):
    return dict(name=name, kind="draft", dtype="bf16", Hq=Hq, Hkv=Hkv, d=128, kv=kv, nodes=nodes, spread=spread, launch=launch)


def _topk(name, *, dtype="bf16", rows, live, vocab=152064, k, launch="prepared"):
    return dict(name=name, kind="topk", dtype=dtype, rows=rows, live=live, vocab=vocab, k=k, launch=launch)


def _project(name, *, rows, live, dim, vocab=152064, k, launch="prepared"):
    return dict(name=name, kind="project", dtype="bf16", rows=rows, live=live, dim=dim, vocab=vocab, k=k, launch=launch)


def listed():
    return [
        # full-precision checks of a small model: every call a few microseconds, the separate calls one after the other
        _step("step_f32_small", dtype="f32", Hq=4, Hkv=1, d=64, kv_lo=256, kv_hi=256, vocab=1024, tree="toy", launch="direct"),
        # one layer of a 72B-shape target over an image-sized context, the closed loop of the fused calls
        _step("step_4k", kv_lo=4096, kv_hi=4096),
        # a video-length context with the wide parameter set, the step replayed as a HIP graph
        _step("step_16k_graph", kv_lo=16384, kv_hi=16384, tree="video", entropy=3.0, launch="graph"),
        # a batch of eight conversations of very different lengths in one packed launch
        _step("step_batch8_ragged", B=8, kv_lo=2048, kv_hi=12288),
        # three short chats over a few layers at odd lengths, called directly: launches and host work count
        _step("step_batch3_short", B=3, kv_lo=301, kv_hi=1999, layers=4, launch="direct"),
        # the whole 80-layer attention stack of a verify pass over a long video, 64 nodes in the tree: the largest
        _step("stack_32k_64nodes", kv_lo=32768, kv_hi=32768, layers=80, tree="full", commit=False),
        # the draft model (7B shape: 28/4 heads) growing a tree level by level over a pruned cache
        _draft("draft_levels", kv=2560, nodes=25),
        # the target's greedy tokens of a batch of eight trees, stored logits, every node live
        _topk("greedy_512_rows", rows=512, live=512, k=1),
        # confidence of a few draft rows whose logits were left in fp32
        _topk("draft_rows_f32", dtype="f32", rows=8, live=8, k=10, launch="direct"),
        # greedy tokens of one tree straight from the 72B output projection: the weight matrix is the work
        _project("project_64", rows=64, live=64, dim=8192, k=1),
        # the same for a batch of eight trees with every node live: the contraction is the work
        _project("project_512", rows=512, live=512, dim=8192, k=1),
        # the draft model's projection (hidden 3584) of a tree level, ten candidates per row
        _project("project_draft", rows=16, live=16, dim=3584, k=10),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    launch = rng.choice(["direct", "prepared", "graph"])
    kind = rng.choice(["step", "step", "step", "draft", "topk", "project", "project"])
    vocab = rng.choice([152064, _log_int(rng, 32000, 152064)])
    if kind == "step" and rng.random() < 0.2:
        return _strip(_step("", dtype="f32", B=rng.randint(1, 2), Hq=4, Hkv=rng.choice([1, 2]), d=64, kv_lo=rng.randint(64, 128),
                            kv_hi=rng.randint(128, 512), vocab=rng.randint(700, 4100), tree="toy", launch=launch))
    if kind == "step":
        B = rng.choice([1, 1, 2, rng.randint(3, 12)])
        hi = _log_int(rng, 256, 32768)
        lo = hi if B == 1 else _log_int(rng, max(64, hi // 8), hi)
        room = 80 * 32768 // (B * hi)            # layers that cost no more than the largest listed case
        return _strip(_step("", B=B, kv_lo=lo, kv_hi=hi, vocab=vocab, layers=_log_int(rng, 1, min(32, max(1, room))),
                            tree=rng.choice(["paper", "paper", "video", "full"]), entropy=round(rng.uniform(0.05, 5.0), 2),
                            commit=rng.random() < 0.5, launch=launch))
    if kind == "draft":
        return _strip(_draft("", kv=_log_int(rng, 300, 8192), nodes=rng.randint(4, 40), spread=rng.randint(2, 8), launch=launch))
    if kind == "topk":
        if rng.random() < 0.5:
            rows = 64 * rng.randint(1, 8)
            return _strip(_topk("", rows=rows, live=rng.randint(rows // 4, rows), vocab=vocab, k=1, launch=launch))
        rows = rng.randint(1, 12)
        return _strip(_topk("", dtype=rng.choice(["bf16", "f32"]), rows=rows, live=rows, vocab=vocab, k=rng.randint(2, 40), launch=launch))
    if rng.random() < 0.4:
        rows = rng.randint(1, 48)
        return _strip(_project("", rows=rows, live=rows, dim=128 * rng.randint(8, 32), vocab=vocab, k=rng.randint(2, 16), launch=launch))
    rows = 64 * rng.choice([1, 1, 2, 4, 8])
    return _strip(_project("", rows=rows, live=rng.randint(rows // 4, rows), dim=128 * rng.randint(16, 64), vocab=vocab, k=1,
                           launch=launch))


def _strip(case):
    return {key: value for key, value in case.items() if key != "name"}


# ---- inputs ------------------------------------------------------------------------------------------------------

def _kv_lens(case):
    if case["B"] == 1:
        return [case["kv_hi"]]
    r = random.Random(case["B"] * 1000003 + case["kv_lo"] * 131 + case["kv_hi"])
    return [r.randint(case["kv_lo"], case["kv_hi"]) for _ in range(case["B"])]


def _group_live(case):
    """Live rows of each group of 64 target rows (the node counts of a batch of trees)."""
    groups = -(-case["rows"] // NODES)
    base, extra = divmod(case["live"], groups)
    return [base + (1 if g < extra else 0) for g in range(groups)]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _padded(rows, vocab, dtype):
    """Logit rows with a row pitch of whole 16-byte pieces, as an allocator for odd vocabularies lays them out."""
    pitch = -(-vocab // 8) * 8
    return torch.zeros(rows, pitch, device="cuda", dtype=dtype)[:, :vocab]


def _draft_rows(case, gen):
    """[B, vocab] fp32 draft logits of the wanted entropy, and the scale of their noise."""
    B, vocab = case["B"], case["vocab"]
    z = torch.randn(B, vocab, generator=gen, device="cuda")
    if case["tree"] == "full":                  # a geometric top 64: the rule then fills all 64 nodes
        z = z * 0.05 - 60.0
        for b in range(B):
            at = torch.randperm(vocab, generator=gen, device="cuda")[:64]
            z[b, at] = -math.log(2.0) * torch.arange(64, device="cuda", dtype=torch.float32)
        return z, 1.0
    beta = 1.5 if case["tree"] == "toy" else workloads.scale_for_entropy(case["entropy"])
    return z * beta, beta


def _tree_buffers(B):
    i32 = dict(device="cuda", dtype=torch.int32)
    return dict(n_nodes=torch.ones(B, **i32), parent=torch.full((B, NODES), -1, **i32), depth=torch.zeros(B, NODES, **i32),
                rank=torch.full((B, NODES), -1, **i32), anc_mask=torch.ones(B, NODES, device="cuda", dtype=torch.int64),
                node_token=torch.full((B, NODES), -1, **i32))


def _row_outputs(rows, k):
    f = lambda *shape: torch.zeros(*shape, device="cuda")  # noqa: E731
    return dict(entropy=f(rows), topk_idx=torch.zeros(rows, k, device="cuda", dtype=torch.int32), topk_prob=f(rows, k),
                topk_renorm=f(rows, k), topk_entropy=f(rows), alpha=f(rows))


def _bytes(n):
    return torch.empty(n, device="cuda", dtype=torch.uint8)


def prepare(case, seed):
    return {"step": _prepare_step, "draft": _prepare_draft, "topk": _prepare_topk, "project": _prepare_project}[case["kind"]](case, seed)


def _program(case, calls_of_pass, outputs):
    """The passes a program alternates between, in the way it launches them.  `calls_of_pass` is a list (one per parity
    of the pass) of lists of (call name, positional arguments, keyword arguments)."""
    state = dict(outputs=outputs, at=0)
    if case["launch"] == "direct":
        state["passes"] = [[(getattr(sage, name), a, kw) for name, a, kw in calls] for calls in calls_of_pass]
        state["how"] = "direct"
    elif case["launch"] == "prepared":
        state["passes"] = [[sage.prepare(name, *a, **kw) for name, a, kw in calls] for calls in calls_of_pass]
        state["how"] = "prepared"
    else:
        side = torch.cuda.Stream()
        state["passes"] = []
        for calls in calls_of_pass:
            prepared = [sage.prepare(name, *a, stream=side, **kw) for name, a, kw in calls]
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                for call in prepared:
                    call()
            state["passes"].append(graph)
        state["how"] = "graph"
        state["keep"] = calls_of_pass
    return state


def _prepare_step(case, seed):
    gen = _generator(seed)
    dtype = DTYPES[case["dtype"]]
    B, Hq, Hkv, d, V, layers = case["B"], case["Hq"], case["Hkv"], case["d"], case["vocab"], case["layers"]
    prm = TREES[case["tree"]]
    k, cap = prm["k"], case["kv_hi"] + ROOM
    params = sage.tree_params(**prm)
    code = sage.F32 if dtype == torch.float32 else sage.BF16

    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda", dtype=dtype)  # noqa: E731
    lens = _kv_lens(case)
    kv_start = torch.arange(B, device="cuda", dtype=torch.int64) * cap
    kv_len = torch.tensor(lens, device="cuda", dtype=torch.int32)
    Kc, Vc = randn(layers, B * cap, Hkv, d), randn(layers, B * cap, Hkv, d)
    Q, O = randn(layers, B, NODES, Hq, d), torch.zeros(layers, B, NODES, Hq, d, device="cuda", dtype=dtype)
    Kt, Vt = randn(layers, B, NODES, Hkv, d), randn(layers, B, NODES, Hkv, d)

    # the tree being verified was planned from this draft row, and the target mostly agrees with it
    row, beta = _draft_rows(case, gen)
    draft, target = _padded(B, V, dtype), _padded(B * NODES, V, dtype)
    draft.copy_(row)
    for b in range(B):
        target[b * NODES:(b + 1) * NODES] = row[b] + 0.5 * beta * torch.randn(NODES, V, generator=gen, device="cuda")
    del row

    tree = [_tree_buffers(B), _tree_buffers(B)]
    plan, tgt = _row_outputs(B, k), _row_outputs(B * NODES, 1)
    ws_draft = _bytes(sage.sage_entropy_topk_workspace_bytes(B, V, k))
    ws_target = _bytes(sage.sage_entropy_topk_workspace_bytes(B * NODES, V, 1))
    ws_att = _bytes(sage.sage_tree_attention_workspace_bytes(code, B, Hq, Hkv, d, cap))
    i32 = dict(device="cuda", dtype=torch.int32)
    path_cap = prm["d_max"] + 1
    acc = dict(accept_len=torch.zeros(B, **i32), best_node=torch.zeros(B, **i32), path_nodes=torch.zeros(B, path_cap, **i32),
               out_tokens=torch.zeros(B, path_cap, **i32))
    hist, count = torch.zeros(B, 10, **i32), torch.zeros(B, **i32)
    d_max = [torch.full((B,), prm["d_max"], **i32) for _ in range(2)]
    scale, strides = 1.0 / math.sqrt(d), (Hkv * d, d)

    row_out = [plan[n] for n in ("entropy", "topk_idx", "topk_prob", "topk_renorm", "topk_entropy", "alpha")]
    tgt_idx = tgt["topk_idx"].view(B, NODES)
    close_limits = (2.0, 3.0, prm["d_min"], prm["d_max"])

    # the first tree and the draft row's slices, as the step before leaves them
    sage.sage_entropy_topk(draft, k, *row_out, ws_draft)
    t = tree[0]
    sage.sage_build_tree(plan["topk_renorm"], plan["alpha"], params, t["n_nodes"], t["parent"], t["depth"], t["rank"], t["anc_mask"],
                         None, plan["topk_idx"], t["node_token"])
    sage.sage_entropy_topk_slices(draft, k, ws_draft)

    def attention(layer, now):
        return (Q[layer], Kc[layer], Vc[layer], Kt[layer], Vt[layer], O[layer], kv_start, kv_len, cap, *strides, now["anc_mask"],
                now["n_nodes"], scale, ws_att)

    def calls_of(cur):
        now, nxt = tree[cur], tree[cur ^ 1]
        planned = [nxt[n] for n in ("n_nodes", "parent", "depth", "rank", "anc_mask")]
        accepted = [acc[n] for n in ("accept_len", "best_node", "path_nodes", "out_tokens")]
        close = (kv_start, kv_len, cap, *strides)
        calls = []
        if case["dtype"] == "f32":              # the separate calls
            calls.append(("sage_entropy_topk", (draft, k, *row_out, ws_draft), {}))
            calls.append(("sage_build_tree", (plan["topk_renorm"], plan["alpha"], params, *planned, None, plan["topk_idx"],
                                              nxt["node_token"]), dict(d_max_seq=d_max[cur])))
            calls += [("sage_tree_attention", attention(layer, now), {}) for layer in range(layers)]
            calls.append(("sage_entropy_topk", (target, 1, *[tgt[n] for n in ("entropy", "topk_idx", "topk_prob", "topk_renorm",
                                                                              "topk_entropy", "alpha")], ws_target, now["n_nodes"], NODES), {}))
            calls.append(("sage_verify_accept", (now["node_token"], tgt_idx, now["parent"], now["depth"], now["anc_mask"],
                                                 now["n_nodes"], path_cap, *accepted), {}))
        else:                                   # planning rides in the first layer's attention, slice passes share a launch
            calls.append(("sage_tree_attention_with_plan", (*attention(0, now), ws_draft, V, params, *row_out, *planned, None,
                                                            nxt["node_token"]), dict(d_max_seq=d_max[cur])))
            calls += [("sage_tree_attention", attention(layer, now), {}) for layer in range(1, layers)]
            calls.append(("sage_entropy_topk_slices_pair", (target, now["n_nodes"], NODES, ws_target, draft, k, ws_draft), {}))
            verify = (ws_target, V, now["node_token"], now["parent"], now["depth"], now["anc_mask"], now["n_nodes"], path_cap,
                      tgt["entropy"], tgt_idx, *accepted)
            if case["commit"] and layers == 1:
                calls.append(("sage_verify_accept_close_from_slices", (*verify, Kt[0], Vt[0], Kc[0], Vc[0], *close, hist, count,
                                                                       d_max[cur], d_max[cur ^ 1], *close_limits), {}))
                return calls
            calls.append(("sage_verify_accept_from_slices", verify, {}))
        if case["commit"]:
            calls += [("sage_commit_path", (Kt[i], Vt[i], Kc[i], Vc[i], *close, acc["path_nodes"], acc["accept_len"]), {})
                      for i in range(layers - 1)]
            last = layers - 1
            calls.append(("sage_close_step", (Kt[last], Vt[last], Kc[last], Vc[last], *close, acc["path_nodes"], acc["accept_len"],
                                              hist, count, d_max[cur], d_max[cur ^ 1], *close_limits), {}))
        return calls

    outputs = dict(O=O, plan=plan, target=dict(entropy=tgt["entropy"], topk_idx=tgt["topk_idx"]), accepted=acc, trees=tree)
    if case["commit"]:
        outputs.update(kv_len=kv_len, hist=hist, count=count, d_max=d_max, Kc=Kc, Vc=Vc)
    return _program(case, [calls_of(0), calls_of(1)], outputs)


def _prepare_draft(case, seed):
    gen = _generator(seed)
    Hq, Hkv, d, L, n = case["Hq"], case["Hkv"], case["d"], case["kv"], case["nodes"]
    r = random.Random(n * 1009 + case["spread"])         # the tree's shape belongs to the case, the values to the seed
    parent = [-1] + [r.randint(max(0, v - case["spread"]), v - 1) for v in range(1, n)]
    depth = [0] * n
    for v in range(1, n):
        depth[v] = depth[parent[v]] + 1
    order = sorted(range(n), key=lambda v: (depth[v], v))        # level order
    place = {old: new for new, old in enumerate(order)}
    mask = np.zeros((1, NODES), np.uint64)
    for new, old in enumerate(order):
        mask[0, new] = np.uint64(1 << new) | (mask[0, place[parent[old]]] if old else np.uint64(0))
    upto = [sum(1 for x in depth if x <= level) for level in range(max(depth) + 1)]

    randn = lambda *shape: torch.randn(*shape, generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    Kc, Vc = randn(L, Hkv, d), randn(L, Hkv, d)
    Q, Kt, Vt = randn(1, NODES, Hq, d), randn(1, NODES, Hkv, d), randn(1, NODES, Hkv, d)
    O = torch.zeros_like(Q)
    anc = torch.from_numpy(mask.view(np.int64)).cuda()
    i32 = dict(device="cuda", dtype=torch.int32)
    kv_start, kv_len = torch.zeros(1, device="cuda", dtype=torch.int64), torch.full((1,), L, **i32)
    ws = _bytes(sage.sage_tree_attention_workspace_bytes(sage.BF16, 1, Hq, Hkv, d, L))
    calls = []
    for first, count in zip([0] + upto[:-1], upto):
        calls.append(("sage_tree_attention", (Q, Kc, Vc, Kt, Vt, O, kv_start, kv_len, L, Hkv * d, d, anc,
                                              torch.full((1,), count, **i32), 1.0 / math.sqrt(d), ws),
                      dict(first_node=torch.full((1,), first, **i32))))
    return _program(case, [calls], O)


def _rows_case(case, name, source, workspace):
    """The call of a topk or project case: `source` = its leading tensors."""
    k = case["k"]
    out = _row_outputs(case["rows"], k)
    if k == 1:                                   # greedy tokens of grouped rows
        live = torch.tensor(_group_live(case), device="cuda", dtype=torch.int32)
        kept = [out["entropy"], out["topk_idx"], None, None, None, None]
        calls = [(name, (*source, k, *kept, workspace, live, NODES), {})]
        out = dict(entropy=out["entropy"], topk_idx=out["topk_idx"])
    else:
        calls = [(name, (*source, k, *[out[n] for n in ("entropy", "topk_idx", "topk_prob", "topk_renorm", "topk_entropy", "alpha")],
                         workspace), {})]
    return _program(case, [calls], out)


def _prepare_topk(case, seed):
    gen = _generator(seed)
    rows, V = case["rows"], case["vocab"]
    logits = _padded(rows, V, DTYPES[case["dtype"]])
    for r in range(0, rows, NODES):
        part = logits[r:r + NODES]
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda") * 4.0)
    ws = _bytes(sage.sage_entropy_topk_workspace_bytes(rows, V, case["k"]))
    return _rows_case(case, "sage_entropy_topk", (logits,), ws)


def _prepare_project(case, seed):
    gen = _generator(seed)
    rows, dim, V = case["rows"], case["dim"], case["vocab"]
    hidden = torch.randn(rows, dim, generator=gen, device="cuda", dtype=torch.bfloat16)
    weight = torch.randn(V, dim, generator=gen, device="cuda", dtype=torch.bfloat16) * (3.0 / math.sqrt(dim))
    ws = _bytes(sage.sage_lm_head_topk_workspace_bytes(rows, V, case["k"]))
    return _rows_case(case, "sage_lm_head_topk", (hidden, weight), ws)


# ---- one pass ----------------------------------------------------------------------------------------------------

def run(state):
    todo = state["passes"][state["at"]]
    state["at"] = (state["at"] + 1) % len(state["passes"])
    if state["how"] == "direct":
        for call, a, kw in todo:
            call(*a, **kw)
    elif state["how"] == "prepared":
        for call in todo:
            call()
    else:
        todo.replay()
    return state["outputs"]


def work(case):
    esz = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "step":
        n, B, V = MEAN_NODES[case["tree"]], case["B"], case["vocab"]
        positions = sum(_kv_lens(case))
        kv_row, q_row = 2 * case["Hkv"] * case["d"] * esz, 2 * case["Hq"] * case["d"] * esz
        attention = positions * kv_row + B * n * (kv_row + q_row)
        flops = 4.0 * n * case["Hq"] * case["d"] * (positions + B * n)
        return {"bytes": case["layers"] * attention + B * (n + 1) * V * esz, "flops": case["layers"] * flops}
    if case["kind"] == "draft":                  # every level's call reads the cache; each node's row is computed once
        r = _levels(case)
        kv_row, q_row = 2 * case["Hkv"] * case["d"] * esz, 2 * case["Hq"] * case["d"] * esz
        return {"bytes": r * case["kv"] * kv_row + case["nodes"] * (kv_row + q_row),
                "flops": 4.0 * case["nodes"] * case["Hq"] * case["d"] * (case["kv"] + case["nodes"])}
    live, V = case["live"], case["vocab"]
    if case["kind"] == "topk":
        return {"bytes": live * V * esz, "flops": 0}
    return {"bytes": (V + live) * case["dim"] * esz, "flops": 2.0 * live * V * case["dim"]}


def _levels(case):
    r = random.Random(case["nodes"] * 1009 + case["spread"])
    depth = [0]
    for v in range(1, case["nodes"]):
        depth.append(depth[r.randint(max(0, v - case["spread"]), v - 1)] + 1)
    return max(depth) + 1


def tolerance(case):
    """Indices, trees, tokens, committed bytes and state are whole numbers and stay the same, except where a projection's
    sums decide between two logits that fp32 accumulation cannot tell apart."""
    if case["kind"] == "project":
        return {"rel": 1e-4, "max": 1e-3, "differ": 0.01}
    if case["kind"] == "topk" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}
