"""GPU parity: every call of the C-ABI HIP library against the CPU oracle on the same seeded inputs.

Integer outputs (top-k indices, trees, masks, acceptance) are bit-exact; entropies/probabilities agree to 1e-5
(the kernels compute them in fp32 whatever the logits' storage type); attention outputs agree per (node, head)
row to 1e-5 (fp32) / 2e-2 (bf16) in relative L2 norm and in max error relative to the row's largest magnitude.
"""
import numpy as np
import pytest

import oracle
from helpers import MAX_NODES, chain_parents, pad_tree, random_parents, star_parents
from paper_2602_00523_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def gu():
    import gpu_utils
    from paper_2602_00523_amd import sage
    print("\n[lib]", sage.sage_build_info(), flush=True)
    return gpu_utils


def close(gpu, ref, tol=1e-5):
    return np.abs(gpu.astype(np.float64) - ref) <= tol * np.maximum(np.abs(ref), 1.0)


def check_entropy(gu, logits, k, n_valid=None, rpg=1, tol=1e-5):
    o = oracle.entropy_topk(logits, k, n_valid, rpg)
    g = gu.gpu_entropy_topk(logits, k, n_valid, rpg)
    rows = logits.shape[0]
    valid = np.ones(rows, bool) if n_valid is None else np.array([(r % rpg) < n_valid[r // rpg] for r in range(rows)])
    np.testing.assert_array_equal(g["topk_idx"][valid], o["topk_idx"][valid])
    for key in ("entropy", "topk_entropy", "alpha"):
        assert close(g[key][valid], o[key][valid], tol).all(), key
    for key in ("topk_prob", "topk_renorm"):
        assert close(g[key][valid], o[key][valid], tol).all(), key
        rel = np.abs(g[key][valid] - o[key][valid]) <= 1e-4 * o[key][valid] + 1e-30
        assert rel.all(), key + " (relative)"
    # skipped rows are untouched
    assert (g["topk_idx"][~valid] == -1).all() and np.isnan(g["entropy"][~valid]).all()
    return o, g


# ------------------------------------------------------------------ a1 / a1'

def test_entropy_topk_toy_rows(gu):
    temps = wl.toy_temperatures(32)
    z = wl.gaussian(wl.seed_for("toy", 0, 1), (32, 1024), "f32")
    logits = (z / temps[:, None].astype(np.float32)).astype(np.float32)
    o, _ = check_entropy(gu, logits, 8)
    assert o["entropy"].min() < 4.0 and o["entropy"].max() > 6.5        # spans peaked to near-uniform rows


@pytest.mark.parametrize("vocab,k,dtype", [(152064, 10, "bf16"), (152064, 16, "bf16"), (152064, 1, "bf16"),
                                           (4099, 5, "f32"), (1000, 64, "f32"), (70001, 3, "bf16"),
                                           (300000, 32, "bf16"),      # candidate lists too long for the second pass's LDS
                                           (1048576, 64, "f32"),      # the largest vocabulary and k the call takes
                                           (1048576, 1, "bf16")])
def test_entropy_topk_shapes(gu, vocab, k, dtype):
    rows = 6
    stride = (vocab + 15) // 16 * 16
    scales = np.array([0.3, 1.0, 3.5, 5.0, 9.0, 40.0], np.float32)
    z = wl.rng(vocab + k).standard_normal((rows, stride), dtype=np.float32) * scales[:, None]
    buf = wl.to_storage(z, dtype)
    check_entropy(gu, buf[:, :vocab], k)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab,k", [(64, 64), (700, 8), (1024, 1), (1024, 17), (1025, 1), (2048, 5), (2049, 5), (2050, 64), (4096, 1), (4097, 1)])
def test_entropy_topk_few_slices(gu, vocab, k, dtype):
    """Vocabularies up to and just past what one launch takes, with groups of which only some rows count."""
    rows, rpg, n_valid = 11, 4, np.array([3, 0, 4], np.int32)
    z = wl.rng(vocab + k).standard_normal((rows, (vocab + 15) // 16 * 16), dtype=np.float32) * 4.0
    buf = wl.to_storage(z, dtype)[:, :vocab]
    check_entropy(gu, buf, k)
    check_entropy(gu, buf, k, n_valid, rpg)


def test_entropy_topk_closed_forms_and_ties(gu):
    V = 152064
    x = np.zeros((4, V), np.float32)
    x[1] = -np.inf
    x[1, 777] = 2.0
    x[2] = -np.inf
    x[2, 5] = x[2, 150000] = 1.0
    x[3, :] = 7.25                                   # uniform with a tie everywhere: top-k = lowest indices
    o, g = check_entropy(gu, wl.to_storage(x, "bf16"), 10)
    assert abs(g["entropy"][0] - np.log(V)) < 1e-4 and abs(g["alpha"][0]) < 1e-6
    assert g["entropy"][1] == 0.0 and g["alpha"][1] == 1.0 and g["topk_idx"][1, 0] == 777
    assert abs(g["entropy"][2] - np.log(2)) < 1e-6 and list(g["topk_idx"][2, :2]) == [5, 150000]
    assert list(g["topk_idx"][3]) == list(range(10))


def test_entropy_topk_row_groups_k1(gu):
    V, rpg = 152064, 64
    n_valid = np.array([9, 0, 64], np.int32)
    z = wl.gaussian(77, (3 * rpg, V), "bf16", 4.0)
    o, g = check_entropy(gu, z, 1, n_valid, rpg)
    assert (g["alpha"][:9] == 1.0).all()


def selection_rows(kind, vocab, dtype):
    """Rows whose winners sit where a selection can go wrong."""
    g = wl.rng(4200 + vocab)
    x = g.standard_normal((2, vocab)).astype(np.float32)
    if kind == "equal":                                  # every logit the same: the lowest indices win
        x[:] = 1.5
    elif kind == "levels":                               # a handful of values: long runs of ties at the threshold
        x[:] = g.integers(0, 3, size=x.shape)
    elif kind == "one slice":                            # all winners in one stretch of 1024 logits, and in its last ones
        x[0, 1024:2048] += 50.0
        x[1, vocab - 70:] += 50.0
    elif kind == "planted":                              # 64 (row 1: 20) distinct large logits over a level floor of equal ones
        x[:] = -60.0
        for r, many in enumerate((64, 20)):
            x[r, g.permutation(vocab)[:many]] = -0.5 * np.arange(many)
    elif kind == "few finite":                           # fewer finite logits than k
        x[:] = -np.inf
        x[0, [5, vocab // 2, vocab - 1]] = [1.0, 2.0, 2.0]
        x[1, vocab - 1] = 0.25
    buf = wl.to_storage(np.pad(x, ((0, 0), (0, -vocab % 16))), dtype)      # (rows are 16-byte aligned)
    return buf[:, :vocab]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,vocab,k", [
    ("equal", 3000, 64), ("equal", 300000, 16), ("levels", 40000, 64), ("levels", 152064, 10), ("one slice", 5000, 64),
    ("one slice", 152064, 16), ("gaussian", 40000, 64), ("gaussian", 70001, 40), ("gaussian", 1025, 17), ("gaussian", 2049, 2),
    ("planted", 152064, 64), ("planted", 152064, 16), ("planted", 5000, 33), ("planted", 3000, 21),
    ("few finite", 3000, 10), ("few finite", 9000, 40)])
def test_topk_selection_edges(gu, dtype, kind, vocab, k):
    """Ties at the threshold, concentrated winners, a last slice of one logit, fewer candidates than k: indices exact."""
    x = selection_rows(kind, vocab, dtype)
    g1, o1 = gu.gpu_entropy_topk(x, k), oracle.entropy_topk(x, k)
    assert (g1["topk_idx"] == o1["topk_idx"]).all()
    np.testing.assert_allclose(g1["topk_prob"], o1["topk_prob"], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 6, 17])
def test_topk_short_last_slice(gu, dtype, k):
    """A last slice of 1024 with fewer logits than k, about k, and the winners of a row among them; in one call, and through
    the pair of slice passes and the planning call."""
    import torch
    from paper_2602_00523_amd import sage
    prm = dict(d_min=1, d_max=4, w_min=1, w_max=k, k=k, n_max=16)
    for vocab in [1024 * m + r for m in (1, 3) for r in sorted({1, k - 1, k, k + 1})]:
        tail = vocab % 1024
        x = wl.rng(vocab * 64 + k).standard_normal((3, vocab)).astype(np.float32)
        x[0, -tail:] += 20.0                             # row 0: all of the last slice wins; row 1: none of it
        x[1, -tail:] -= 20.0
        x[2, 7] = x[2, -1] = 30.0                        # row 2: an equal pair, the second in the last slice
        x = wl.to_storage(np.pad(x, ((0, 0), (0, -vocab % 16))), dtype)[:, :vocab]
        want = oracle.entropy_topk(x, k)["topk_idx"]
        np.testing.assert_array_equal(gu.gpu_entropy_topk(x, k)["topk_idx"], want, err_msg=f"vocab {vocab}")
        dev = gu.to_dev(x.base)[:, :vocab]
        ws_a, ws_b = (gu.workspace(sage.sage_entropy_topk_workspace_bytes(3, vocab, n)) for n in (1, k))
        sage.sage_entropy_topk_slices_pair(dev, torch.tensor([3], device=dev.device, dtype=torch.int32), 3, ws_a, dev, k, ws_b)
        f = lambda *s: torch.zeros(*s, device=dev.device)  # noqa: E731
        i32 = lambda *s: torch.zeros(*s, device=dev.device, dtype=torch.int32)  # noqa: E731
        idx, alpha = i32(3, k), f(3)
        sage.sage_build_tree_from_slices(ws_b, vocab, sage.tree_params(**prm), None, idx, None, f(3, k), None, alpha, i32(3),
                                         i32(3, MAX_NODES), i32(3, MAX_NODES), i32(3, MAX_NODES),
                                         torch.zeros(3, MAX_NODES, device=dev.device, dtype=torch.int64))
        np.testing.assert_array_equal(idx.cpu().numpy(), want, err_msg=f"vocab {vocab}, pair")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k", [2, 10, 33, 48])
@pytest.mark.parametrize("vocab", [700, 1024 + 63, 2048 + 64, 1024 + 65, 3072 + 127, 1024 + 130, 4000])
def test_topk_by_waves(gu, vocab, k, dtype):
    """Lists of up to 48 candidates, which a wave finds in a slice: winners that share lanes (rising and falling rows, runs of eight and sixteen
    at the top, one lane's sixteen logits alone above the rest), more equal values at the threshold than the list has room for, few logits above
    -inf, the last slice about the size of the list, and all of it below zero."""
    rng = wl.rng(vocab * 31 + k)
    x = rng.standard_normal((12, vocab)).astype(np.float32)
    x[0] = np.sort(x[0])
    x[1] = np.sort(x[1])[::-1]
    x[2] = np.linspace(-3.0, 3.0, vocab)
    x[3, 40:40 + 16] += 9.0
    lane = 5 * (8 if dtype == "bf16" else 4)             # one lane's logits of a slice, in its loads of 64 lanes each
    per_load = 512 if dtype == "bf16" else 256
    for first in range(0, min(vocab, 1024), per_load):
        x[4, first + lane:first + lane + per_load // 64] += 9.0
    x[5] = np.round(x[5] * 2.0)                          # few levels
    x[6] = np.where(rng.random(vocab) < 0.2, 1.5, -2.0)  # two
    x[7] = -np.inf
    x[7, rng.permutation(vocab)[:6]] = rng.standard_normal(6)
    x[8] -= 100.0
    x[9, -70:] += 5.0
    x[10] = 0.0
    x[11, ::3] = -np.inf
    x = wl.to_storage(np.pad(x, ((0, 0), (0, -vocab % 16))), dtype)[:, :vocab]
    g1, o1 = gu.gpu_entropy_topk(x, k), oracle.entropy_topk(x, k)
    np.testing.assert_array_equal(g1["topk_idx"], o1["topk_idx"])
    np.testing.assert_allclose(g1["topk_prob"], o1["topk_prob"], rtol=1e-5, atol=1e-7)
    np.testing.assert_allclose(g1["entropy"], o1["entropy"], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("rows,vocab,dtype", [(448, 152061, "bf16"), (224, 152061, "f32"), (900, 80000, "bf16")])
@pytest.mark.parametrize("grouped", [False, True])
def test_greedy_rows_of_many_logits(gu, rows, vocab, dtype, grouped):
    """More than 128 MB of logits are read with other loads: every row has the bits that it has in a call over half of the rows, which the
    other tests hold to the oracle."""
    import torch
    from paper_2602_00523_amd import sage
    half, esz, rpg = rows // 2, 4 if dtype == "f32" else 2, 56 if rows < 900 else 50
    assert half * vocab * esz <= 128 << 20 < rows * vocab * esz
    g = torch.Generator(device="cuda:0")
    g.manual_seed(vocab + rows)
    x = (torch.randn(rows, -(-vocab // 8) * 8, generator=g, device="cuda:0") * 3.0).to(torch.float32 if dtype == "f32" else torch.bfloat16)[:, :vocab]
    live = torch.tensor([1 + 11 * i % rpg for i in range(rows // rpg)], device="cuda:0", dtype=torch.int32) if grouped else None
    ws = torch.empty(sage.sage_entropy_topk_workspace_bytes(rows, vocab, 1), device="cuda:0", dtype=torch.uint8)

    def run(n):
        ent = torch.full((n,), -1.0, device="cuda:0")
        idx = torch.full((n, 1), -1, device="cuda:0", dtype=torch.int32)
        sage.sage_entropy_topk(x[:n], 1, ent, idx, None, None, None, None, ws, live, rpg if grouped else 1)
        torch.cuda.synchronize()
        return ent, idx

    (e, i), (eh, ih) = run(rows), run(half)
    assert torch.equal(e[:half], eh) and torch.equal(i[:half], ih) and (ih >= 0).any()
    counted = torch.ones(rows, dtype=torch.bool, device="cuda:0") if live is None else torch.arange(rows, device="cuda:0") % rpg < live.repeat_interleave(rpg)
    assert (i[~counted] == -1).all() and (i[counted, 0].long() == x[counted].max(-1).values[:, None].eq(x[counted]).int().argmax(-1)).all()


@pytest.mark.parametrize("rows,rpg,n_valid,vocab,dtype", [
    (150, 64, [64, 33, 22], 5000, "f32"),            # a short last group (22 rows): every one of its rows counts
    (150, 64, [17, 0, 99], 70008, "bf16"),           # n_valid beyond the group's rows is clamped
    (40, 5, [5, 0, 1, 3, 5, 2, 4, 0], 2048, "bf16"), # groups smaller than the row phases of a launch
    (7, 1, [1, 0, 1, 1, 0, 0, 1], 3000, "f32"),
])
def test_entropy_topk_row_groups_k1_shapes(gu, rows, rpg, n_valid, vocab, dtype):
    z = wl.rng(rows * 7 + vocab).standard_normal((rows, vocab), dtype=np.float32) * 3.0
    check_entropy(gu, wl.to_storage(z, dtype), 1, np.array(n_valid, np.int32), rpg)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab", [1024, 1025, 2048, 3001, 9000])
def test_greedy_token_among_equal_maxima(gu, vocab, dtype):
    """k = 1: the first of equal largest logits, wherever in a slice they are (loads, lanes, elements of a lane, slices), zeros of
    both signs, slices of -inf only, a row whose only number is its last logit; the two-group and three-group phases of rows."""
    rng = wl.rng(vocab)
    rows, pairs = 192, [0, 1, 7, 8, 63, 64, 255, 256, 511, 512, 1023, vocab - 2, vocab - 1]
    x = rng.standard_normal((rows, vocab)).astype(np.float32)
    for r in range(rows):
        if r % 4 == 0:                                    # a pair at places of note
            x[r, [pairs[r // 4 % 13], pairs[(r // 4 * 5 + 3) % 13]]] = 9.0
        elif r % 4 == 1:                                  # several anywhere
            x[r, rng.integers(0, vocab, 5)] = 9.0
        elif r % 4 == 2:                                  # zeros of either sign are the largest, and equal
            x[r] = -np.abs(x[r]) - 0.5
            x[r, rng.integers(0, vocab, 4)] = np.array([0.0, -0.0, 0.0, -0.0], np.float32)
        else:
            x[r] = -np.inf
            x[r, vocab - 1 if r & 4 else rng.integers(0, vocab)] = -3.0
    x = wl.to_storage(np.pad(x, ((0, 0), (0, -vocab % 16))), dtype)[:, :vocab]
    for groups in (1, 2, 3):
        rpg = 64 * 3 // groups
        check_entropy(gu, x, 1, np.full(groups, rpg, np.int32), rpg)


@pytest.mark.parametrize("dtype,bits", [("bf16", 0x7F81), ("bf16", 0xFFA0), ("bf16", 0x7FC0), ("f32", 0x7F800001), ("f32", 0xFFA00000), ("f32", 0x7FC00000)])
@pytest.mark.parametrize("vocab", [1024, 3001])
def test_greedy_token_among_nans(gu, vocab, dtype, bits):
    """k = 1: logits that are no numbers, signalling or quiet, take no number's place, wherever they stand beside the largest one."""
    rng = wl.rng(vocab + bits)
    rows = 192
    x = rng.standard_normal((rows, vocab)).astype(np.float32)
    best = rng.integers(0, vocab, rows)
    nan = rng.random((rows, vocab)) < 0.05
    for r in range(rows):                                 # the largest among its lane's sixteen, one to all of the others NaNs
        x[r, best[r]] = 9.0
        lane = best[r] // 8 * 8 + np.arange(8) if dtype == "bf16" else best[r] // 4 * 4 + np.arange(4)
        lane = np.concatenate([lane, lane ^ (512 if dtype == "bf16" else 256)])
        nan[r, rng.permutation(lane)[:1 + r % len(lane)].clip(0, vocab - 1)] = True
        nan[r, best[r]] = False
    x = wl.to_storage(np.pad(x, ((0, 0), (0, -vocab % 16))), dtype)
    x.view(np.uint16 if dtype == "bf16" else np.uint32)[:, :vocab][nan] = bits
    for groups in (0, 1, 2, 3):                           # (0: every row valid, not in groups)
        rpg = rows // max(groups, 1)
        got = gu.gpu_entropy_topk(x[:, :vocab], 1, np.full(groups, rpg, np.int32) if groups else None, rpg if groups else 1)["topk_idx"]
        np.testing.assert_array_equal(got[:, 0], best)


@pytest.mark.parametrize("k", [4, 8, 9, 40])
@pytest.mark.parametrize("bits", [0x7FFFFFFF, 0xFFFFFFFF])
def test_topk_of_extreme_nans(gu, bits, k):
    """Rows of the NaNs whose codes are the largest and the smallest word: k tokens of the row (equal values: the first k)."""
    vocab = 5000
    x = np.full((2, vocab), bits, np.uint32).view(np.float32)
    x[1, 1030:1060] = 1.0                            # fewer numbers in a slice than k = 40, more than the others
    g = gu.gpu_entropy_topk(x, k)
    np.testing.assert_array_equal(g["topk_idx"][0], np.arange(k))
    idx = g["topk_idx"][1]
    assert ((0 <= idx) & (idx < vocab)).all() and len(set(idx.tolist())) == k


# ------------------------------------------------------------------ a2

def test_build_tree_bit_exact(gu):
    g = wl.rng(2024)
    cases = [("paper", wl.CONFIGS["c2"]["tree"]), ("c3", wl.CONFIGS["c3"]["tree"]), ("toy", wl.CONFIGS["toy"]["tree"]),
             ("cap", dict(d_min=8, d_max=20, w_min=6, w_max=12, k=12, n_max=20)),
             ("one", dict(d_min=1, d_max=1, w_min=1, w_max=1, k=1, n_max=1))]
    for name, prm in cases:
        B, k = 512, prm["k"]
        pt = np.sort(g.random((B, k)) ** g.integers(1, 7, size=(B, 1)), axis=1)[:, ::-1]
        pt = (pt / pt.sum(1, keepdims=True)).astype(np.float32)
        alpha = g.random(B).astype(np.float32)
        alpha[:4] = [0.0, 1.0, 0.5, 0.1]
        pt[4] = 0
        pt[4, 0] = 1                                 # one-hot
        pt[5] = 1.0 / k                              # flat
        ids = g.integers(0, 152064, size=(B, k)).astype(np.int32)
        o = oracle.build_tree(pt, alpha, prm, ids)
        t = gu.gpu_build_tree(pt, alpha, prm, ids)
        np.testing.assert_array_equal(t["n_nodes"], o["n_nodes"], err_msg=name)
        for key in ("parent", "depth", "rank", "anc_mask", "cum_prob", "node_token"):
            for b in range(B):
                n = int(o["n_nodes"][b])
                np.testing.assert_array_equal(t[key][b, :n], o[key][b, :n], err_msg=f"{name} {key} seq {b}")
            if key != "cum_prob":
                assert (t[key][:, :][np.arange(MAX_NODES)[None, :] >= o["n_nodes"][:, None]] == (0 if key == "anc_mask" else -2)).all()
        assert o["n_nodes"].max() == prm["n_max"] or name in ("paper", "toy", "c3")


# ------------------------------------------------------------------ a4

def test_verify_accept_bit_exact(gu):
    g = wl.rng(99)
    B = 600
    parent = np.full((B, MAX_NODES), -7, np.int32)
    depth = np.full((B, MAX_NODES), -7, np.int32)
    mask = np.zeros((B, MAX_NODES), np.uint64)
    nn = np.zeros(B, np.int32)
    tok = g.integers(0, 3, (B, MAX_NODES)).astype(np.int32)
    tgt = g.integers(0, 3, (B, MAX_NODES)).astype(np.int32)
    for b in range(B):
        n = int(g.integers(1, 65)) if b > 3 else (1, 64, 2, 33)[b]
        par = random_parents(g, n, chain_bias=float(g.random()))
        p, d, m, _ = pad_tree(par)
        parent[b], depth[b], mask[b], nn[b] = p[0], d[0], m[0], n
        if b % 5 == 0:                               # force long accepted paths
            tok[b, 1:n] = tgt[b, par[1:]]
            if n > 3 and b % 10 == 0:
                tok[b, n // 2] = 9
    cap = 65
    o = oracle.verify_accept(tok, tgt, parent, depth, nn, cap)
    r = gu.gpu_verify_accept(tok, tgt, parent, depth, mask, nn, cap)
    for key in ("accept_len", "best_node", "path_nodes", "out_tokens"):
        np.testing.assert_array_equal(r[key], o[key], err_msg=key)
    assert o["accept_len"].max() >= 10 and o["accept_len"].min() == 0


# ------------------------------------------------------------------ a3

def tree_batch(g, B, sizes=None, kind="random"):
    mask = np.zeros((B, MAX_NODES), np.uint64)
    nn = np.zeros(B, np.int32)
    for b in range(B):
        n = int(sizes[b]) if sizes is not None else int(g.integers(1, 65))
        par = {"random": lambda: random_parents(g, n, chain_bias=0.5), "chain": lambda: chain_parents(n),
               "star": lambda: star_parents(n)}[kind]()
        _, _, m, _ = pad_tree(par)
        mask[b], nn[b] = m[0], n
    return mask, nn


def run_attention_case(gu, seed, dtype, B, Hq, Hkv, d, lens, sizes=None, kind="random", pad=3):
    g = wl.rng(seed)
    inp = wl.attention_inputs(seed, B, Hq, Hkv, d, lens, dtype, pad_tokens=pad)
    mask, nn = tree_batch(g, B, sizes, kind)
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, Hq, Hkv, d)
    got, raw = gu.gpu_tree_attention(inp, mask, nn, Hq, Hkv, d, fill=12345.0)
    worst = gu.assert_attention_close(got, ref, nn, TOL[dtype])
    for b in range(B):                               # rows at or beyond n_nodes are not written
        assert (got[b, int(nn[b]):] == 12345.0).all() or dtype == "bf16" and np.allclose(got[b, int(nn[b]):], 12352.0)
    return worst


def test_attention_toy_f32(gu):
    w = run_attention_case(gu, wl.seed_for("toy"), "f32", 1, 4, 1, 64, [256], sizes=[16])
    print(f" worst rel err {w:.2e}", flush=True)


@pytest.mark.parametrize("B,Hq,Hkv,d,lens", [(2, 4, 2, 64, [300, 0]), (1, 6, 3, 32, [1]), (3, 8, 1, 128, [511, 257, 64]),
                                             (1, 2, 2, 256, [1000]), (2, 2, 1, 4, [5, 288]), (3, 2, 1, 60, [223, 224, 289]),
                                             (2, 4, 2, 68, [63, 130]), (1, 2, 1, 132, [66]), (2, 1, 1, 192, [3, 0])])
def test_attention_f32_shapes(gu, B, Hq, Hkv, d, lens):
    run_attention_case(gu, 5 + B + d, "f32", B, Hq, Hkv, d, lens)


@pytest.mark.parametrize("d,L,at", [(64, 9, 8), (64, 9, 0), (128, 300, 299), (256, 30, 17), (32, 1, 0), (64, 12, "tree"), (128, 28, "tree")])
def test_attention_f32_nan_key(gu, d, L, at):
    """A NaN key makes the rows that admit it NaN, also where a wave of the kernel has no other key; other rows do not see it."""
    inp = wl.attention_inputs(700 + d + L, 1, 2, 2, d, [L], "f32", pad_tokens=1)
    mask, nn = tree_batch(wl.rng(L), 1, [7], kind="star")
    if at == "tree":
        inp["Kt"][0, 6, 0, d // 2] = np.nan                  # a leaf's key: a row of its own admits it
    else:
        inp["Kc"][at, 0, d // 2] = np.nan
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, 2, 2, d)[0, :7]
    got = gu.gpu_tree_attention(inp, mask, nn, 2, 2, d)[0][0, :7]
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    assert np.isnan(ref).any() and not np.isnan(ref).all()
    fine = ~np.isnan(ref)
    assert np.abs(got[fine] - ref[fine]).max() <= TOL["f32"] * np.abs(ref[fine]).max()


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("d,L,low", [(64, 9, {8: -200}), (128, 40, {39: -150, 0: -300}), (256, 700, {3: -150, 699: -200}), (60, 0, {"tree": -200}),
                                     (64, 12, {4: -60, 5: -60, 6: -60, 7: -125})])
def test_attention_f32_value_without_weight(gu, d, L, low, value):
    """An infinite or NaN value does not count where its key's weight in the row is zero in fp32 (exp(-105) is), also where that
    key has the largest score of its wave, or of the wave's weight only a part."""
    inp = wl.attention_inputs(900 + d + L, 1, 2, 1, d, [L], "f32", pad_tokens=1)
    mask, nn = tree_batch(wl.rng(L), 1, [7], kind="star")
    inp["Q"][..., 0] = 1.0
    for at, score in low.items():
        k, v = (inp["Kt"][0, 6, 0], inp["Vt"][0, 6, 0]) if at == "tree" else (inp["Kc"][at, 0], inp["Vc"][at, 0])
        k[:] = 0.0
        k[0] = score * np.sqrt(d)
        v[:] = 0.0                                           # what the oracle sees
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, 2, 1, d)[0, :7]
    at = list(low)[-1]
    v = inp["Vt"][0, 6, 0] if at == "tree" else inp["Vc"][at, 0]
    v[1::3] = value
    got = gu.gpu_tree_attention(inp, mask, nn, 2, 1, d)[0][0, :7]
    assert np.abs(got - ref).max() <= TOL["f32"] * np.abs(ref).max()


@pytest.mark.parametrize("d,L", [(64, 300), (4, 5), (132, 66), (256, 70)])
def test_attention_f32_alignment(gu, d, L):
    """fp32 rows need be aligned like their elements only: the same bits from buffers that begin 4, 8 and 12 bytes past 16."""
    B, Hq, Hkv = 1, 4, 2
    inp = wl.attention_inputs(800 + d, B, Hq, Hkv, d, [L], "f32")
    mask, nn = tree_batch(wl.rng(d), B, [13])
    want = gu.gpu_tree_attention(inp, mask, nn, Hq, Hkv, d)[0]
    m, n = gu.to_dev(mask), gu.to_dev(nn)
    start, length = gu.to_dev(np.asarray(inp["kv_start"], np.int64)), gu.to_dev(np.asarray(inp["kv_len"], np.int32))
    ws = gu.workspace(gu.sage.sage_tree_attention_workspace_bytes(gu.sage.F32, B, Hq, Hkv, d, L))
    for off in (1, 2, 3):
        def moved(a):
            x = gu.torch.zeros(a.size + 4, device=gu.DEV, dtype=gu.torch.float32)
            x[off:off + a.size] = gu.to_dev(a.reshape(-1))
            return x[off:off + a.size].view(a.shape)
        Q, Kc, Vc, Kt, Vt = (moved(inp[k]) for k in ("Q", "Kc", "Vc", "Kt", "Vt"))
        O = moved(np.zeros_like(inp["Q"]))
        gu.sage.sage_tree_attention(Q, Kc, Vc, Kt, Vt, O, start, length, L, inp["kv_token_stride"], inp["kv_head_stride"], m, n,
                                    1.0 / float(np.sqrt(d)), ws)
        np.testing.assert_array_equal(gu.to_host(O)[0, :13], want[0, :13])


@pytest.mark.parametrize("kind,sizes,lens", [
    ("random", [64], [1000]),           # several tiles and a ragged tail, full tree
    ("random", [1], [64]),              # single node, exactly one tile
    ("chain", [9], [777]),              # deep-narrow tree of the confident regime
    ("star", [17], [130]),              # shallow-wide tree
    ("random", [33], [0]),              # empty cache: tree keys only
    ("random", [5], [63]),
    ("random", [20], [4096]),
])
def test_attention_bf16_72b_heads_single(gu, kind, sizes, lens):
    w = run_attention_case(gu, 40 + sizes[0] + lens[0], "bf16", 1, 64, 8, 128, lens, sizes, kind)
    print(f" worst rel err {w:.2e}", flush=True)


def test_attention_bf16_ragged_batch(gu):
    g = wl.rng(8)
    B = 5
    lens = g.integers(0, 700, size=B)
    sizes = [8, 64, 1, 30, 47]
    run_attention_case(gu, 81, "bf16", B, 64, 8, 128, lens, sizes)


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (16, 4), (32, 2), (28, 4), (12, 4), (10, 2), (13, 1)])
def test_attention_bf16_other_group_sizes(gu, Hq, Hkv):
    run_attention_case(gu, 90 + Hq, "bf16", 2, Hq, Hkv, 128, [333, 70], sizes=[64, 11])


@pytest.mark.parametrize("layout", ["head_major", "padded", "shifted", "reversed"])
@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 64, 8, 128), ("bf16", 28, 4, 128), ("f32", 4, 2, 64)])
def test_attention_cache_layouts(gu, layout, dtype, Hq, Hkv, d):
    """The cache stored head-major, with padded rows, shifted, or with the sequences in another order: the kernels get
    the re-laid-out buffers and strides, the reference is the oracle on the packed layout."""
    from helpers import relayout_cache
    B, lens, sizes = 3, [300, 0, 1000], [20, 5, 64]
    g = wl.rng(500 + Hq)
    inp = wl.attention_inputs(600 + Hq, B, Hq, Hkv, d, lens, dtype)
    mask, nn = tree_batch(g, B, sizes)
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, Hq, Hkv, d)
    got, _ = gu.gpu_tree_attention(relayout_cache(inp, layout), mask, nn, Hq, Hkv, d)
    gu.assert_attention_close(got, ref, nn, TOL[dtype])


@pytest.mark.parametrize("Hq,Hkv,L,n,rows_only", [(28, 4, 1638, 25, False), (64, 8, 300, 64, False),
                                                   (28, 4, 1638, 25, True), (64, 8, 300, 64, True), (32, 2, 700, 64, True)])
def test_attention_level_by_level_growth(gu, Hq, Hkv, L, n, rows_only):
    """A tree drafted one level per forward pass (the draft side of Alg. 1 Phase 1): call l sees the nodes of levels
    0..l, a prefix of the level-ordered tree, and the rows of level l must come out as in the oracle's single pass over
    the whole tree, because a node attends only to the cache and its ancestors.  With rows_only the call is also told
    where level l starts (first_node) and must leave the rows of the levels before it alone."""
    from helpers import depth_by_walk, level_order
    g = wl.rng(7000 + n)
    par = level_order(random_parents(g, n, chain_bias=0.3))
    dep = depth_by_walk(par)
    assert (np.diff(dep) >= 0).all() and dep.max() >= 3
    _, _, mask, nn = pad_tree(par)
    inp = wl.attention_inputs(7100 + n, 1, Hq, Hkv, 128, [L], "bf16")
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, Hq, Hkv, 128)
    for level in range(int(dep.max()) + 1):
        upto = np.array([int((dep <= level).sum())], np.int32)
        first = np.array([int((dep < level).sum())], np.int32)
        got, _ = gu.gpu_tree_attention(inp, mask, upto, Hq, Hkv, 128, fill=7.0, first_node_np=first if rows_only else None)
        rows = np.nonzero(dep == level)[0]
        g_l, r_l = got[0, rows], ref[0, rows]
        err = np.abs(g_l - r_l).max(-1) / np.maximum(np.abs(r_l).max(-1), 1e-300)
        assert err.max() <= TOL["bf16"], (level, float(err.max()))
        assert (got[0, int(upto[0]):] == 7.0).all()             # nodes of deeper levels are not there yet
        if rows_only:
            assert (got[0, :int(first[0])] == 7.0).all()        # and the levels before are not computed again


@pytest.mark.parametrize("dtype,B,Hq,Hkv,d", [("bf16", 3, 32, 4, 128), ("bf16", 1, 64, 4, 128), ("f32", 2, 4, 2, 64)])
def test_attention_first_node_batches_and_clamping(gu, dtype, B, Hq, Hkv, d):
    """first_node per sequence: rows [first, n) equal the call without it bit for bit (the same keys, the same split
    boundaries only if the row count leaves the decomposition alone, so compare to the oracle as well), rows outside
    stay untouched; values outside [0, n) are clamped into it."""
    g = wl.rng(7300 + B)
    lens = [int(x) for x in g.integers(100, 1500, size=B)]
    sizes = [64, 9, 33][:B]
    masks = np.zeros((B, 64), np.uint64)
    for b in range(B):
        masks[b] = pad_tree(random_parents(g, sizes[b], 0.4))[2][0]
    nn = np.array(sizes, np.int32)
    inp = wl.attention_inputs(7400 + B, B, Hq, Hkv, d, lens, dtype)
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], masks, nn, Hq, Hkv, d)
    for first in ([10, 8, 32][:B], [63, 0, 1][:B], [-5, 100, 33][:B]):
        got, _ = gu.gpu_tree_attention(inp, masks, nn, Hq, Hkv, d, fill=7.0, first_node_np=np.array(first, np.int32))
        for b in range(B):
            f = min(max(first[b], 0), sizes[b] - 1)
            assert (got[b, :f] == 7.0).all() and (got[b, sizes[b]:] == 7.0).all()
            g_l, r_l = got[b, f:sizes[b]], ref[b, f:sizes[b]]
            err = np.abs(g_l - r_l).max(-1) / np.maximum(np.abs(r_l).max(-1), 1e-300)
            assert err.max() <= TOL[dtype], (first, b, float(err.max()))


@pytest.mark.parametrize("seed", range(24))
def test_attention_bf16_random_configurations(gu, seed):
    """Random head counts (any group size up to 16), batch sizes, ragged lengths around tile and split boundaries,
    tree sizes and shapes."""
    g = wl.rng(1000 + seed)
    Hkv = int(g.choice([1, 2, 4, 8]))
    G = int(g.integers(1, 17))
    B = int(g.integers(1, 5))
    edges = np.array([0, 1, 63, 64, 65, 127, 128, 129, 191, 192, 255, 256, 257, 2047, 2048, 2049])
    lens = [int(g.choice(edges)) if g.random() < 0.6 else int(g.integers(0, 3000)) for _ in range(B)]
    sizes = [int(g.choice([1, 2, 4, 16, 17, 32, 33, 64])) if g.random() < 0.5 else int(g.integers(1, 65)) for _ in range(B)]
    kind = str(g.choice(["random", "chain", "star"]))
    if kind == "chain":
        sizes = [min(n, 32) for n in sizes]
    run_attention_case(gu, 2000 + seed, "bf16", B, Hkv * G, Hkv, 128, lens, sizes, kind, pad=int(g.integers(0, 5)))


@pytest.mark.parametrize("B,Hq,Hkv,max_len,seed", [
    (64, 16, 2, 300, 1),       # every workgroup's range spans several short sequences (some of them empty)
    (33, 64, 8, 900, 2),       # 72B heads: ranges cut sequences and column groups at arbitrary tiles
    (8, 64, 8, 3000, 3),
    (2, 8, 1, 5000, 4),        # one KV head: 256 ranges over two sequences
    (70, 8, 2, 200, 5),        # more sequences than the batched decomposition takes: per-sequence splits
])
def test_attention_bf16_many_sequences(gu, B, Hq, Hkv, max_len, seed):
    g = wl.rng(300 + seed)
    lens = g.integers(0, max_len + 1, size=B)
    lens[g.integers(0, B)] = 0
    lens[g.integers(0, B)] = max_len
    sizes = [int(g.choice([1, 3, 16, 17, 40, 64])) for _ in range(B)]
    run_attention_case(gu, 3000 + seed, "bf16", B, Hq, Hkv, 128, lens, sizes)


@pytest.mark.parametrize("lens,nodes", [([301, 1999, 1200], 12), ([212, 613], 12), ([4096, 3500], 15), ([301, 1999, 1200], 64), ([90, 0], 3)])
def test_attention_bf16_cut_of_batches(gu, monkeypatch, lens, nodes):
    """Where a batch is cut, as the partials that are written say it: the result's bits depend on it.  Every (sequence, group of 256
    rows) takes 6 positions of a line and one per 32 keys, and the line goes to up to 256 / Hkv workgroups (as many as the workspace
    has slots for beyond one per segment of 64 nodes), at least 6 positions each."""
    Hq, Hkv, slot_bytes = 64, 8, 256 * 272
    kept, workspace = [], gu.workspace
    monkeypatch.setattr(gu, "workspace", lambda n: kept.append(workspace(n)) or kept[-1])
    run_attention_case(gu, 3500, "bf16", len(lens), Hq, Hkv, 128, lens, [nodes] * len(lens))
    slots = kept[-1].numel() // (Hkv * slot_bytes)
    rows = kept[-1][:Hkv * slots * slot_bytes].view(Hkv, slots, slot_bytes)[:, :, 256:264]     # maximum and sum of a slot's first row
    groups = -(-nodes * (Hq // Hkv) // 256)
    segments = [6 + -(-n // 32) + -(-nodes // 32) for n in lens for _ in range(groups)]
    length = max(6, -(-sum(segments) // (slots - 2 * len(lens))))
    want, at = set(), 0
    for i, segment in enumerate(segments):
        want |= {p // length + i for p in range(at + 6, at + segment)}    # a slot per range and segment, in the order of both
        at += segment
    written = (rows != 0xFF).any(-1).cpu().numpy()
    for head in written:
        assert set(np.flatnonzero(head)) == want


@pytest.mark.parametrize("lens,nodes", [([301, 1900, 1200], [16, 17, 12]), ([6000, 2500], [32, 4]), ([900, 2100, 0, 5000], [33, 64, 1, 48]),
                                        ([4000, 2000, 3000], [49, 20, 64]), ([90, 10], [3, 40])])
def test_attention_bf16_cut_of_mixed_batches(gu, monkeypatch, lens, nodes):
    """The same for batches in which some groups have more than 128 rows and others do not: a block takes 4 positions there and 3 here,
    belongs to the range that its first one lies in, and the line is cut as if it were 24 positions longer."""
    Hq, Hkv, slot_bytes = 64, 8, 256 * 272
    kept, workspace = [], gu.workspace
    monkeypatch.setattr(gu, "workspace", lambda n: kept.append(workspace(n)) or kept[-1])
    run_attention_case(gu, 3600, "bf16", len(lens), Hq, Hkv, 128, lens, nodes)
    slots = kept[-1].numel() // (Hkv * slot_bytes)
    rows = kept[-1][:Hkv * slots * slot_bytes].view(Hkv, slots, slot_bytes)[:, :, 256:264]
    groups = [(min(256, n * (Hq // Hkv) - first), 6 + -(-L // 32) + -(-n // 32)) for L, n in zip(lens, nodes) for first in range(0, n * (Hq // Hkv), 256)]
    costs = [4 if rows_of > 128 else 3 for rows_of, _ in groups]
    mixed = len(set(costs)) == 2
    assert mixed == (lens != [4000, 2000, 3000])
    costs = costs if mixed else [1] * len(groups)
    total = sum(c * segment for c, (_, segment) in zip(costs, groups))
    length = max(18 if mixed else 6, -(-(total + (24 if mixed else 0)) // (slots - 2 * len(lens))))
    want, at = set(), 0
    for i, (c, (_, segment)) in enumerate(zip(costs, groups)):
        want |= {(at + c * block) // length + i for block in range(6, segment)}
        at += c * segment
    written = (rows != 0xFF).any(-1).cpu().numpy()
    for head in written:
        assert set(np.flatnonzero(head)) == want


@pytest.mark.parametrize("tiles", [32, 33, 48, 49, 64, 65, 128, 129])
def test_attention_bf16_split_counts(gu, tiles):
    """One sequence and two KV heads: a split per 64-token tile up to 128, so the merge takes every one of its widths at its
    last count, the next one's first, and several passes of the widest."""
    run_attention_case(gu, 4000 + tiles, "bf16", 1, 4, 2, 128, [64 * (tiles - 1) - 3], sizes=[3])


@pytest.mark.parametrize("B", [1, 2])
@pytest.mark.parametrize("splits", [7, 8, 9, 16, 17, 24, 25, 32])
def test_attention_bf16_merge_widths(gu, splits, B):
    """Splits of a row about the steps of 8 in which the merge asks for them: two blocks of 32 keys a split with one sequence, six beside
    an empty sequence."""
    lens = [64 * splits - 32] if B == 1 else [192 * splits - 40, 0]
    run_attention_case(gu, 4200 + splits, "bf16", B, 8, 8, 128, lens, sizes=[5, 3][:B])


@pytest.mark.parametrize("lens,sizes", [([24576], [9]), ([24577], [9]), ([24700], [33]), ([8193, 8192, 8300], [9, 20, 40])])
def test_attention_bf16_of_long_caches(gu, lens, sizes):
    """Sequences at and past the length from which the cache is read with other loads (24576 positions of 8 KV heads, by the number of
    sequences), of one and of two row groups, alone and beside shorter ones; the launch that carries planning along gives the same bits."""
    B, Hq, Hkv, d = len(lens), 64, 8, 128
    run_attention_case(gu, 4400 + lens[0], "bf16", B, Hq, Hkv, d, lens, sizes=sizes)
    inp = wl.attention_inputs(4400 + lens[0], B, Hq, Hkv, d, lens, "bf16", pad_tokens=3)
    mask, nn = tree_batch(wl.rng(4400 + lens[0]), B, sizes)
    _, raw = gu.gpu_tree_attention(inp, mask, nn, Hq, Hkv, d)
    x = wl.gaussian(4400, (B, 5000), "bf16", 3.0)
    O, _, _ = gu.gpu_attention_with_plan(inp, mask, nn, Hq, Hkv, d, x, 8, wl.CONFIGS["toy"]["tree"])
    assert (gu.to_host(raw) == O).all()


@pytest.mark.parametrize("nodes", [4, 16, 17, 32, 33])
@pytest.mark.parametrize("blocks,tail", [(1, 0), (1, 31), (2, 1), (3, 16), (4, 0), (5, 31), (7, 1)])
def test_attention_bf16_pass_lengths(gu, nodes, blocks, tail):
    """One sequence, many KV heads and so few splits: passes of `blocks` 32-token blocks, of which the cache's last holds
    32 - tail tokens, at the row counts on either side of 128 (the reference in one step or in two) and of one and two groups.  Half of the
    lengths with scores that grow along the cache, so that the reference maximum has to move in every block."""
    Hq, Hkv = 512, 64                                     # four splits of a KV head (two where there are two groups)
    splits, tree = (2 if nodes > 32 else 4), (2 if nodes > 32 else 1)
    L = max(32 * (splits * blocks - tree) - tail, 0)
    inp = wl.attention_inputs(5000 + nodes + blocks, 1, Hq, Hkv, 128, [L], "bf16", pad_tokens=2)
    if blocks & 1 and L:
        ramp = np.linspace(0.5, 24.0, L, dtype=np.float32)[:, None, None]
        inp["Kc"][:L] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(inp["Kc"][:L]) * ramp)
    mask, nn = tree_batch(wl.rng(blocks), 1, [nodes])
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, Hq, Hkv, 128)
    got, _ = gu.gpu_tree_attention(inp, mask, nn, Hq, Hkv, 128, fill=12345.0)
    gu.assert_attention_close(got, ref, nn, TOL["bf16"])


@pytest.mark.parametrize("nodes", [4, 17, 33])
@pytest.mark.parametrize("blocks,tail", [(8, 0), (9, 1), (10, 31), (11, 0), (12, 16), (13, 1), (14, 0), (15, 31), (19, 1)])
def test_attention_bf16_long_passes(gu, nodes, blocks, tail):
    """Passes of `blocks` blocks about the lengths at which the loop takes none, one, two or three rounds of four blocks, full and
    with a cut last cache block; scores that grow in every other, so that the reference moves inside the rounds."""
    Hq, Hkv = 512, 64
    splits, tree = (2 if nodes > 32 else 4), (2 if nodes > 32 else 1)
    L = 32 * (splits * blocks - tree) - tail
    inp = wl.attention_inputs(5500 + nodes + blocks, 1, Hq, Hkv, 128, [L], "bf16", pad_tokens=2)
    if blocks & 1:
        ramp = np.linspace(0.5, 24.0, L, dtype=np.float32)[:, None, None]
        inp["Kc"][:L] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(inp["Kc"][:L]) * ramp)
    mask, nn = tree_batch(wl.rng(blocks), 1, [nodes])
    ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                inp["kv_token_stride"], inp["kv_head_stride"], mask, nn, Hq, Hkv, 128)
    got, _ = gu.gpu_tree_attention(inp, mask, nn, Hq, Hkv, 128, fill=12345.0)
    gu.assert_attention_close(got, ref, nn, TOL["bf16"])


def test_attention_is_deterministic(gu):
    inp = wl.attention_inputs(3, 1, 64, 8, 128, [2000], "bf16")
    mask, nn = tree_batch(wl.rng(3), 1, [40])
    a, _ = gu.gpu_tree_attention(inp, mask, nn, 64, 8, 128)
    b, _ = gu.gpu_tree_attention(inp, mask, nn, 64, 8, 128)
    np.testing.assert_array_equal(a, b)


# ------------------------------------------------------------------ whole step, Toy configuration

def test_toy_pipeline_32_steps(gu):
    cfg = wl.CONFIGS["toy"]
    prm, k, V = cfg["tree"], cfg["tree"]["k"], cfg["vocab"]
    temps = wl.toy_temperatures(cfg["steps"])
    taus = []
    for step in range(cfg["steps"]):
        seed = wl.seed_for("toy", step)
        z = wl.gaussian(seed, (1, V), "f32")
        draft = (z / np.float32(temps[step])).astype(np.float32)
        # a1: confidence from the draft distribution
        o1 = oracle.entropy_topk(draft, k)
        g1 = gu.gpu_entropy_topk(draft, k)
        np.testing.assert_array_equal(g1["topk_idx"], o1["topk_idx"])
        assert close(g1["alpha"], o1["alpha"]).all() and close(g1["topk_renorm"], o1["topk_renorm"]).all()
        # a2: the oracle consumes the GPU's fp32 bits so a 1-ulp difference upstream cannot pose as a tree mismatch
        o2 = oracle.build_tree(g1["topk_renorm"], g1["alpha"], prm, g1["topk_idx"])
        g2 = gu.gpu_build_tree(g1["topk_renorm"], g1["alpha"], prm, g1["topk_idx"])
        n = int(o2["n_nodes"][0])
        assert g2["n_nodes"][0] == n
        for key in ("parent", "depth", "rank", "anc_mask", "node_token"):
            np.testing.assert_array_equal(g2[key][0, :n], o2[key][0, :n])
        # a3
        inp = wl.attention_inputs(seed + 50000, 1, cfg["Hq"], cfg["Hkv"], cfg["d"], [cfg["kv_len"]], "f32")
        ref = oracle.tree_attention(inp["Q"], inp["Kc"], inp["Vc"], inp["Kt"], inp["Vt"], inp["kv_start"], inp["kv_len"],
                                    inp["kv_token_stride"], inp["kv_head_stride"], o2["anc_mask"], o2["n_nodes"],
                                    cfg["Hq"], cfg["Hkv"], cfg["d"])
        got, _ = gu.gpu_tree_attention(inp, g2["anc_mask"], g2["n_nodes"], cfg["Hq"], cfg["Hkv"], cfg["d"])
        gu.assert_attention_close(got, ref, o2["n_nodes"], 1e-5)
        # a1': the target's greedy token per node; node tokens are the draft's top-k candidates by rank
        tgt_logits = np.zeros((MAX_NODES, V), np.float32)
        tgt_logits[:n] = wl.target_logits_from_draft(seed + 60000, draft[0], n, "f32", 0.35 / temps[step])
        o1t = oracle.entropy_topk(tgt_logits, 1, o2["n_nodes"], MAX_NODES)
        g1t = gu.gpu_entropy_topk(tgt_logits, 1, g2["n_nodes"], MAX_NODES)
        np.testing.assert_array_equal(g1t["topk_idx"][:n], o1t["topk_idx"][:n])
        token = g2["node_token"]
        assert (token[0, 1:n] == g1["topk_idx"][0, g2["rank"][0, 1:n]]).all() and token[0, 0] == -1
        tgt = g1t["topk_idx"][:, 0].reshape(1, MAX_NODES)
        # a4
        o4 = oracle.verify_accept(token, tgt, o2["parent"], o2["depth"], o2["n_nodes"], prm["d_max"] + 1)
        g4 = gu.gpu_verify_accept(token, tgt, g2["parent"], g2["depth"], g2["anc_mask"], g2["n_nodes"], prm["d_max"] + 1)
        for key in ("accept_len", "best_node", "path_nodes", "out_tokens"):
            np.testing.assert_array_equal(g4[key], o4[key], err_msg=f"step {step} {key}")
        taus.append(int(o4["accept_len"][0]))
    print(f" accepted lengths over 32 steps: mean {np.mean(taus):.2f}, max {max(taus)}", flush=True)
    assert max(taus) >= 2
