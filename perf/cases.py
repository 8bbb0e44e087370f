"""The workloads this framework's speed is judged by: what they are, how their inputs are made, what one pass runs.

A user of the library drafts a token tree with a small model (sx_draft_tree: batches of at most 128 nodes through a
7B-shaped decoder, then the expansion step), verifies it with a large one (sx_verify_tree: hundreds to thousands of
nodes through 70B-shaped layers), walks it and commits the accepted K/V.  The listed cases are these calls and their
blocks at the sizes of the repository's own configurations (7B: d 4096, 32 heads, FFN 11008; 70B: d 8192, 64/8 heads,
FFN 28672; vocabularies 1024, 32000 and 128256), with ragged row counts among them; draw() spreads the same kinds over
their ranges.  Whole models have one or two layers: a layer repeats, and one pass of all 80 would time the same kernels.
"""
import heapq
import math

import numpy as np
import torch

import paper_2406_02532_amd as sx

SHAPES = {  # d_model, query heads, KV heads, head_dim, d_ffn
    "tiny": (256, 4, 4, 64, 688),
    "7b": (4096, 32, 32, 128, 11008),
    "70b": (8192, 64, 8, 128, 28672),
}
GROUP = 128  # group size of the 4-bit weights


def listed():
    return [
        # Smallest calls: a whole draft tree and a whole verification round of the tiny fp32 configuration, a few
        # dozen launches of microseconds each -- latency and launch count.
        dict(name="draft_tree_tiny_f32", kind="draft", P=128, V=1024, K=64, D=6, B=16, k=4),
        dict(name="round_tiny_f32", kind="round", P=128, V=1024, T=64),
        # One iteration of the draft loop: a full batch of 128 new nodes through the 7B-shaped draft model, attending
        # to 2048 cached tokens and to the 640 nodes drafted before it; the same with the decoder in 4 bits and a
        # batch, a prefix and a tree that fill no tile.
        dict(name="draft_forward_7b", kind="forward", shape="7b", layers=2, w4=False, P=2048, first=640, n=128, V=32000),
        dict(name="draft_forward_7b_w4", kind="forward", shape="7b", layers=2, w4=True, P=1501, first=300, n=100, V=32000),
        # The verification forward of the 70B-shaped target over a full tree: the headline step, two of its layers.
        dict(name="verify_70b_2048", kind="forward", shape="70b", layers=2, w4=False, P=2048, first=0, n=2048, V=32000),
        # One attention block of the target (QKV + rotary, tree attention, O) for a tree of odd size; the paper's
        # trees have 128 to 2048 nodes.
        dict(name="attn_block_70b_1000", kind="attn", shape="70b", P=1111, T=1000),
        # MLP blocks: a batch of the draft model, and a small verification tree through the target.
        dict(name="mlp_7b_100", kind="mlp", shape="7b", M=100),
        dict(name="mlp_70b_300", kind="mlp", shape="70b", M=300),
        # Head and expansion step of a draft model with a 128k vocabulary.
        dict(name="head_expand_128k", kind="head", d=4096, V=128256, M=100, k=32, B=2048),
        # Acceptance walk over the logits of a 2048-node tree (t = 0.6, top-p 0.9) as peaked as a trained model's, and
        # the walk that accepts with P_target / P_draft on a 128k vocabulary.
        dict(name="walk_32k", kind="walk", T=2048, V=32000, ratio=False, temperature=0.6, top_p=0.9),
        dict(name="walk_ratio_128k", kind="walk", T=384, V=128256, ratio=True, temperature=0.6, top_p=0.9),
        # The paper-sized expansion step alone.
        dict(name="expand_32k", kind="expand", N=2048, V=32000, k=32, B=2048),
    ]


def _log(rng, lo, hi):
    """An integer between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["draft", "round", "forward", "forward", "verify", "attn", "mlp", "mlp", "head", "walk", "expand"])
    if kind == "draft":
        B = rng.randint(4, 32)
        D = rng.randint(3, 8)
        return dict(kind=kind, P=_log(rng, 1, 512), V=rng.randint(500, 4000), K=rng.randint(B, B * D), D=D, B=B, k=rng.randint(2, 8))
    if kind == "round":
        return dict(kind=kind, P=_log(rng, 1, 512), V=rng.randint(500, 4000), T=_log(rng, 1, 256))
    if kind == "forward":
        return dict(kind=kind, shape="7b", layers=rng.randint(1, 2), w4=rng.random() < 0.5, P=_log(rng, 16, 4096),
                    first=rng.randint(0, 2000), n=_log(rng, 1, 128), V=rng.choice([32000, rng.randint(20000, 50000)]))
    if kind == "verify":
        return dict(kind="forward", shape=rng.choice(["7b", "70b"]), layers=1, w4=rng.random() < 0.25, P=_log(rng, 16, 3000),
                    first=0, n=_log(rng, 129, 2048), V=32000)
    if kind == "attn":
        return dict(kind=kind, shape=rng.choice(["7b", "70b"]), P=_log(rng, 1, 4096), T=_log(rng, 129, 2048))
    if kind == "mlp":
        return dict(kind=kind, shape=rng.choice(["7b", "70b"]), M=_log(rng, 1, 2048))
    if kind == "head":
        return dict(kind=kind, d=rng.choice([2048, 4096]), V=rng.choice([32000, 128256, rng.randint(30000, 131072)]),
                    M=_log(rng, 1, 128), k=_log(rng, 4, 200), B=_log(rng, 64, 4096))
    if kind == "walk":
        return dict(kind=kind, T=_log(rng, 16, 2048), V=rng.choice([1024, 32000, rng.randint(1000, 50000)]), ratio=rng.random() < 0.3,
                    temperature=rng.choice([0.0, 0.6, 1.0]), top_p=rng.choice([0.8, 0.9, 1.0]))
    return dict(kind=kind, N=_log(rng, 16, 2048), V=rng.choice([32000, rng.randint(1000, 60000)]), k=_log(rng, 4, 128),
                B=_log(rng, 64, 8192))


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------

class Cfg:
    """Decoder shape, as paper_2406_02532_amd.ModelWeights reads it."""

    def __init__(self, shape, layers, vocab, dtype):
        self.d_model, self.n_q_heads, self.n_kv_heads, self.head_dim, self.d_ffn = SHAPES[shape]
        self.n_layers, self.vocab, self.dtype = layers, vocab, dtype
        self.rope_base, self.rms_eps = 10000.0, 1e-5
        self.torch_dtype = torch.bfloat16 if dtype == "bf16" else torch.float32


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, std, dtype, mean=0.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(dtype)


def _matrix(g, n, k, dtype, std=0.02):
    out = torch.empty((n, k), dtype=dtype, device="cuda")
    step = max(1, (1 << 26) // k)  # bounded fp32 scratch for the large matrices
    for i in range(0, n, step):
        out[i:i + step] = _normal(g, (min(step, n - i), k), std, dtype)
    return out


def _w4(g, n, k):
    """Codes, scales and zero points of a 4-bit [n][k] matrix: values of the size of the 16-bit one's."""
    q = torch.randint(-2 ** 31, 2 ** 31 - 1, (n, k // 8), dtype=torch.int32, device="cuda", generator=g)
    s = (torch.rand((n, k // GROUP), device="cuda", generator=g) * 0.0054 + 0.0006).to(torch.bfloat16)
    z = torch.randint(0, 16, (n, k // GROUP), dtype=torch.uint8, device="cuda", generator=g)
    return q, s, z


def _model(cfg, g, w4=False, head_std=0.02):
    d, F, dt = cfg.d_model, cfg.d_ffn, cfg.torch_dtype
    nq, nkv = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim
    mats = dict(wq=(nq, d), wk=(nkv, d), wv=(nkv, d), wo=(d, nq), w_gate=(F, d), w_up=(F, d), w_down=(d, F))
    w = dict(layers=[], embed=_matrix(g, cfg.vocab, d, dt), final_norm=_normal(g, (d,), 0.1, dt, 1.0),
             lm_head=_matrix(g, cfg.vocab, d, dt, head_std))
    if w4:
        w.update(layers_w4=[], w4_group=GROUP)
    for _ in range(cfg.n_layers):
        layer = {n: _normal(g, (d,), 0.1, dt, 1.0) for n in ("attn_norm", "ffn_norm")}
        if w4:
            w["layers_w4"].append({n: _w4(g, *s) for n, s in mats.items()})
        else:
            layer.update({n: _matrix(g, *s, dt) for n, s in mats.items()})
        w["layers"].append(layer)
    return w


def _tree(T, V, seed, width=8, max_depth=32):
    """A best-first draft tree: peaked next-token distributions (the likeliest child holds 30 to 95 % of the mass), nodes
    in the order in which a search by cumulative probability takes them.  Parents come first, siblings differ."""
    r = np.random.default_rng(seed)
    tok, par = np.zeros(T, np.int32), np.full(T, -1, np.int32)
    heap, serial, n = [(0.0, 0, -1, int(r.integers(V)), 0)], 1, 0
    while n < T:
        nll, _, p, t, depth = heapq.heappop(heap)
        tok[n], par[n] = t, p
        if depth < max_depth:
            q = r.uniform(0.3, 0.95)
            rest = r.exponential(1.0, 2 * width)
            probs = np.sort(np.concatenate([[q], (1 - q) * rest / rest.sum()]))[::-1][:width]
            start = int(r.integers(V))
            for c, pr in enumerate(probs):
                heapq.heappush(heap, (nll - math.log(pr), serial, n, (start + 37 * c) % V, depth + 1))
                serial += 1
        n += 1
    return tok, par


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    s = dict(case=case)
    if kind in ("draft", "round"):
        cfg = Cfg("tiny", 2, case["V"], "fp32")
        P, rows = case["P"], case["P"] + case.get("T", 0)
        s.update(cfg=cfg, w=_model(cfg, g, head_std=0.16))  # next-token distributions sharper than a flat start's
        s["mw"] = sx.ModelWeights(cfg, s["w"])
        kv = (cfg.n_layers, rows, cfg.n_kv_heads, cfg.head_dim)
        s["k"], s["v"] = _normal(g, kv, 1.0, torch.float32), _normal(g, kv, 1.0, torch.float32)
        if kind == "draft":
            s["root"] = torch.randint(0, case["V"], (1,), dtype=torch.int32, device="cuda", generator=g)
            i32 = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")  # noqa: E731
            s["out"] = (i32(case["K"]), i32(case["K"]), torch.zeros(case["K"], device="cuda"), i32(1))
            # the first call makes the workspace, which a decoding loop keeps
            s["ws"] = sx.draft_tree(s["mw"], s["k"], s["v"], P, s["root"], case["K"], case["D"], case["B"], case["k"])[4]
        else:
            s["k"][:, P:] = 0
            s["v"][:, P:] = 0
            tok, par = _tree(case["T"], case["V"], seed)
            s.update(tok=_dev(tok), par=_dev(par), buf=sx.RoundBuffers(s["mw"], rows, case["T"]), seed=seed)
            s["buf"].path.zero_()
            s["buf"].tokens.zero_()
    elif kind == "forward":
        cfg = Cfg(case["shape"], case["layers"], case["V"], "bf16")
        P, first, T = case["P"], case["first"], case["first"] + case["n"]
        s.update(cfg=cfg, w=_model(cfg, g, case["w4"]))
        s["mw"] = sx.ModelWeights(cfg, s["w"])
        pre, tree = (cfg.n_layers, P, cfg.n_kv_heads, 128), (cfg.n_layers, T, cfg.n_kv_heads, 128)
        s["pk"], s["pv"] = _normal(g, pre, 1.0, torch.bfloat16), _normal(g, pre, 1.0, torch.bfloat16)
        s["tk"], s["tv"] = _normal(g, tree, 1.0, torch.bfloat16), _normal(g, tree, 1.0, torch.bfloat16)
        tok, par = _tree(T, case["V"], seed)
        s.update(tok=_dev(tok), par=_dev(par), ws=_workspace(s["mw"].workspace_bytes(P, T)),
                 logits=torch.empty((case["n"], case["V"]), device="cuda"))
    elif kind == "attn":
        d, hq, hkv, _, _ = SHAPES[case["shape"]]
        T, P, bf = case["T"], case["P"], torch.bfloat16
        tok, par = _tree(T, 32000, seed)
        depth = np.zeros(T, np.int32)
        for i in range(1, T):
            depth[i] = depth[par[i]] + 1
        s.update(x=_normal(g, (T, d), 1.0, bf), wq=_matrix(g, hq * 128, d, bf), wk=_matrix(g, hkv * 128, d, bf),
                 wv=_matrix(g, hkv * 128, d, bf), wo=_matrix(g, d, hq * 128, bf), par=_dev(par), pos=_dev(depth + P),
                 pk=_normal(g, (P, hkv, 128), 1.0, bf), pv=_normal(g, (P, hkv, 128), 1.0, bf),
                 y=torch.empty((T, d), device="cuda"), ws=_workspace(sx.lib.sx_tree_attention_workspace(T, hq, hkv)))
        s["gemm_ws"] = torch.zeros(sx.lib.sx_gemm_bf16_workspace(), dtype=torch.uint8, device="cuda")
    elif kind == "mlp":
        d, F, M, bf = SHAPES[case["shape"]][0], SHAPES[case["shape"]][4], case["M"], torch.bfloat16
        s.update(x=_normal(g, (M, d), 1.0, bf), wg=_matrix(g, F, d, bf), wu=_matrix(g, F, d, bf), wd=_matrix(g, d, F, bf),
                 act=torch.empty((M, F), dtype=bf, device="cuda"), y=torch.empty((M, d), device="cuda"))
        s["gemm_ws"] = torch.zeros(sx.lib.sx_gemm_bf16_workspace(), dtype=torch.uint8, device="cuda")
    elif kind in ("head", "expand"):
        N, V = case.get("M") or case["N"], case["V"]
        if kind == "head":
            s.update(x=_normal(g, (N, case["d"]), 1.0, torch.bfloat16),
                     w=_matrix(g, V, case["d"], torch.bfloat16, 3.0 / math.sqrt(case["d"])),  # logits of deviation 3
                     logits=torch.empty((N, V), device="cuda"))
            s["gemm_ws"] = torch.zeros(sx.lib.sx_gemm_bf16_workspace(), dtype=torch.uint8, device="cuda")
        else:
            s["logits"] = _normal(g, (N, V), 3.0, torch.float32)
        s["cum"] = -torch.empty(N, device="cuda").exponential_(1.0, generator=g) * torch.randint(1, 33, (N,), device="cuda", generator=g)
        i32 = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")  # noqa: E731
        s.update(row=i32(case["B"]), token=i32(case["B"]), score=torch.zeros(case["B"], device="cuda"), n=i32(1),
                 ws=_workspace(sx.lib.sx_expand_topk_workspace(N, V, case["k"], case["B"])))
    elif kind == "walk":
        T, V = case["T"], case["V"]
        tok, par = _tree(T, V, seed)
        r = np.random.default_rng(seed + 1)
        logits = _normal(g, (T, V), 1.0, torch.float32, -12.0)
        # a handful of likely tokens per row, well apart, and one of the node's children ahead of them: mostly the one
        # that the draft model put first, so that a walk goes some ten levels down as in the paper's measurements
        alt = torch.randint(0, V, (T, 4), device="cuda", generator=g)
        logits.scatter_(1, alt, torch.rand((T, 4), device="cuda", generator=g) * 7.0)
        kids = [[] for _ in range(T)]
        for i in range(1, T):
            kids[par[i]].append(i)
        inner = [i for i in range(T) if kids[i]]
        if inner:
            chosen = [tok[kids[i][0 if r.random() < 0.95 else int(r.integers(len(kids[i])))]] for i in inner]
            logits[_dev(np.array(inner, np.int64)), _dev(np.array(chosen, np.int64))] = 8.0
        draft = None
        if case["ratio"]:  # the draft's view of the same rows, half a unit off
            draft = torch.softmax(logits + _normal(g, (T, V), 0.5, torch.float32), dim=1)
        i32 = lambda n: torch.zeros(n, dtype=torch.int32, device="cuda")  # noqa: E731
        s.update(logits=logits, draft=draft, tok=_dev(tok), par=_dev(par), seed=seed, path=i32(T), tokens=i32(T), n=i32(1),
                 ws=_workspace(sx.lib.sx_accept_walk_workspace(T, V)))
    return s


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "draft":
        t, p, cum, n, _ = sx.draft_tree(s["mw"], s["k"], s["v"], c["P"], s["root"], c["K"], c["D"], c["B"], c["k"],
                                        workspace=s["ws"], out=s["out"])
        return dict(tokens=t, parent=p, cum_logp=cum, n=n)
    if kind == "round":
        b = sx.specexec_round(s["mw"], s["k"], s["v"], c["P"], s["tok"], s["par"], 0.6, 0.9, s["seed"], s["buf"])
        return dict(logits=b.logits, tree_k=b.tree_k, tree_v=b.tree_v, path=b.path, tokens=b.tokens, n=b.n, cache_k=s["k"],
                    cache_v=s["v"])
    if kind == "forward":
        if c["first"] == 0:
            sx.verify_tree(s["mw"], s["pk"], s["pv"], s["tok"], s["par"], logits_out=s["logits"], tree_k_out=s["tk"],
                           tree_v_out=s["tv"], workspace=s["ws"])
        else:
            sx.verify_tree_range(s["mw"], s["pk"], s["pv"], c["P"], s["tok"], s["par"], c["first"], s["tk"], s["tv"],
                                 logits_out=s["logits"], workspace=s["ws"])
        return dict(logits=s["logits"], tree_k=s["tk"], tree_v=s["tv"])
    if kind == "attn":
        q, k, v = sx.qkv_rope_bf16(s["x"], s["wq"], s["wk"], s["wv"], s["pos"], 10000.0)
        o, _ = sx.tree_attention_bf16(q, k, v, s["pk"], s["pv"], s["par"], workspace=s["ws"])
        sx.gemm_bf16(o.view(c["T"], -1), s["wo"], s["y"], workspace=s["gemm_ws"])
        return dict(q=q, k=k, v=v, o=o, y=s["y"])
    if kind == "mlp":
        sx.gemm_bf16(s["x"], s["wg"], s["act"], mode=2, W2=s["wu"], workspace=s["gemm_ws"])
        sx.gemm_bf16(s["act"], s["wd"], s["y"], workspace=s["gemm_ws"])
        return dict(act=s["act"], y=s["y"])
    if kind in ("head", "expand"):
        out = {}
        if kind == "head":
            out["logits"] = sx.gemm_bf16(s["x"], s["w"], s["logits"], workspace=s["gemm_ws"])
        sx.expand_topk(s["logits"], s["cum"], c["k"], c["B"], out_row=s["row"], out_token=s["token"], out_cum_logp=s["score"],
                       n_out=s["n"], workspace=s["ws"])
        return dict(out, row=s["row"], token=s["token"], cum_logp=s["score"], n=s["n"])
    sx.accept_walk(s["logits"], s["tok"], s["par"], c["temperature"], c["top_p"], s["seed"], 2048, path_out=s["path"],
                   tokens_out=s["tokens"], n_out=s["n"], workspace=s["ws"], draft_probs=s["draft"])
    return dict(path=s["path"], tokens=s["tokens"], n=s["n"])


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------

def _forward_work(shape, layers, P, first, n, V, es, w4):
    d, hq, hkv, dh, F = SHAPES[shape]
    per_layer = d * (2 * hq + 2 * hkv) * dh + 3 * d * F
    weight_bytes = per_layer * ((0.5 + 3.0 / GROUP) if w4 else es) * layers + V * d * es + n * d * es
    kv = 2 * (P + first + n) * hkv * dh * es * layers
    flops = 2.0 * n * (per_layer * layers + d * V) + 4.0 * n * (P + 8) * hq * dh * layers
    return dict(bytes=weight_bytes + kv + 4.0 * n * V, flops=flops)


def work(case):
    kind = case["kind"]
    if kind == "draft":
        one = [_forward_work("tiny", 2, case["P"], i * case["B"], case["B"], case["V"], 4, False) for i in range(case["D"])]
        return {k: sum(o[k] for o in one) for k in ("bytes", "flops")}
    if kind == "round":
        return _forward_work("tiny", 2, case["P"], 0, case["T"], case["V"], 4, False)
    if kind == "forward":
        return _forward_work(case["shape"], case["layers"], case["P"], case["first"], case["n"], case["V"], 2, case["w4"])
    if kind == "attn":
        d, hq, hkv, dh, _ = SHAPES[case["shape"]]
        T, P, cols = case["T"], case["P"], (hq + 2 * hkv) * dh
        return dict(bytes=2.0 * d * (cols + hq * dh) + 2.0 * T * d + 4.0 * P * hkv * dh + 2.0 * T * (cols + hq * dh) + 4.0 * T * d,
                    flops=2.0 * T * d * (cols + hq * dh) + 4.0 * T * (P + 8) * hq * dh)
    if kind == "mlp":
        d, F, M = SHAPES[case["shape"]][0], SHAPES[case["shape"]][4], case["M"]
        return dict(bytes=6.0 * d * F + 2.0 * M * (d + F) + 4.0 * M * d, flops=6.0 * M * d * F)
    if kind == "head":
        return dict(bytes=2.0 * case["V"] * case["d"] + 2.0 * case["M"] * case["d"] + 4.0 * case["M"] * case["V"],
                    flops=2.0 * case["M"] * case["d"] * case["V"])
    if kind == "expand":
        return dict(bytes=4.0 * case["N"] * case["V"], flops=0)
    steps = min(case["T"], 12)  # rows visited: one per level that the walk goes down
    return dict(bytes=4.0 * steps * case["V"] * (2 if case["ratio"] else 1), flops=0)


def tolerance(case):
    kind = case["kind"]
    if kind == "walk":
        return "exact"  # decisions far from a tie; whole numbers
    if kind in ("draft", "round"):  # fp32 throughout: 9e-7 from the 64-bit result
        return dict(rel=5e-6, max=1e-3)
    if kind in ("head", "expand"):  # fp32 sums: 4e-7; neighbours whose scores agree to 32 bits may change places
        return dict(rel=2e-6, max=1e-3, differ=0.01)
    # bf16 tensors between the products: what was measured against 64 bits without any rounding is 1.7e-3 for an MLP (one
    # rounding), 4.4e-3 for an attention block, 7e-3 to 1.2e-2 for the logits of one or two layers
    if kind == "mlp":
        return dict(rel=5e-3, max=0.05)
    return dict(rel=1.5e-2, max=0.2) if kind == "attn" else dict(rel=2.5e-2, max=0.3)


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------------

def _w64(w, name, layer):
    """The matrix `name` of a layer in 64 bits; a 4-bit one as its format says: bf16(scale * (code - zero))."""
    if "layers_w4" not in w:
        return w["layers"][layer][name].double()
    q, s, z = w["layers_w4"][layer][name]
    codes = torch.stack([(q >> (4 * j)) & 15 for j in range(8)], dim=2).reshape(q.shape[0], -1)
    s, z = s.float().repeat_interleave(GROUP, 1), z.float().repeat_interleave(GROUP, 1)
    return (s * (codes.float() - z)).to(torch.bfloat16).double()


def _rope64(x, pos):
    half = x.shape[-1] // 2
    inv = 10000.0 ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    a = (pos.double()[:, None] * inv)[:, None, :]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * a.cos() - hi * a.sin(), lo * a.sin() + hi * a.cos()], dim=-1)


def _norm64(h, gain):
    return h / torch.sqrt((h * h).mean(1, keepdim=True) + 1e-5) * gain.double()


def _depth_mask(par):
    """(depth of every node, [T][T] matrix: node i attends to node j)."""
    T = len(par)
    seen, depth = np.zeros((T, T), bool), np.zeros(T, np.int64)
    for i in range(T):
        if par[i] >= 0:
            seen[i] = seen[par[i]]
            depth[i] = depth[par[i]] + 1
        seen[i, i] = True
    return depth, seen


def _attend64(q, k, v, pk, pv, mask):
    """q [n][Hq][Dh] over the prefix rows and the tree rows that `mask` [n][T] names, one KV head at a time."""
    n, hq, dh = q.shape
    hkv = k.shape[1]
    G, P = hq // hkv, pk.shape[0]
    out = torch.empty_like(q)
    for h in range(hkv):
        keys, vals = torch.cat([pk[:, h].double(), k[:, h]]), torch.cat([pv[:, h].double(), v[:, h]])
        for e in range(h * G, h * G + G):
            sc = q[:, e] @ keys.T / math.sqrt(dh)
            sc[:, P:].masked_fill_(~mask, -math.inf)
            out[:, e] = torch.softmax(sc, dim=1) @ vals
    return out


def _forward64(cfg, w, pk, pv, P, tok, par, first, tk=None, tv=None):
    """(logits, tree K, tree V) of nodes first .. T-1; the earlier nodes' rows of tree K/V come from tk, tv."""
    T, dev = len(par), pk.device
    depth, seen = _depth_mask(par)
    mask, pos = _dev(seen[first:]), _dev(depth[first:] + P)
    h = w["embed"][torch.as_tensor(tok[first:], dtype=torch.long, device=dev)].double()
    hq, hkv, dh = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    out_k, out_v = [], []
    for l in range(cfg.n_layers):
        x = _norm64(h, w["layers"][l]["attn_norm"])
        q = _rope64((x @ _w64(w, "wq", l).T).view(-1, hq, dh), pos)
        k = _rope64((x @ _w64(w, "wk", l).T).view(-1, hkv, dh), pos)
        v = (x @ _w64(w, "wv", l).T).view(-1, hkv, dh)
        if first:
            k, v = torch.cat([tk[l, :first].double(), k]), torch.cat([tv[l, :first].double(), v])
        out_k.append(k)
        out_v.append(v)
        h = h + _attend64(q, k, v, pk[l, :P], pv[l, :P], mask).reshape(T - first, -1) @ _w64(w, "wo", l).T
        x = _norm64(h, w["layers"][l]["ffn_norm"])
        gate = x @ _w64(w, "w_gate", l).T
        h = h + (gate * torch.sigmoid(gate) * (x @ _w64(w, "w_up", l).T)) @ _w64(w, "w_down", l).T
    return _norm64(h, w["final_norm"]) @ w["lm_head"].double().T, torch.stack(out_k), torch.stack(out_v)


def _draft64(s):
    """Cumulative log-probabilities of the tree that Alg. 2 builds, in the order of insertion."""
    c = s["case"]
    K, k = c["K"], c["k"]
    tok, par, cum = [], [], []
    queue, serial, thr = [(0.0, 0, int(s["root"][0]), -1)], 1, -math.inf
    for _ in range(c["D"]):
        queue = sorted(queue)[:K]
        popped, queue = queue[:c["B"]], queue[c["B"]:]
        batch = [q for q in popped if -q[0] > thr]
        if not batch:
            break
        base = len(tok)
        for nll, _, t, p in batch:
            tok.append(t)
            par.append(p)
            cum.append(-nll)
        if len(cum) >= K:
            thr = sorted(cum, reverse=True)[K - 1]
        lg, _, _ = _forward64(s["cfg"], s["w"], s["k"], s["v"], c["P"], np.array(tok), np.array(par), 0)
        top = torch.log_softmax(lg[base:], dim=1).topk(k, dim=1)
        val, idx = top.values.cpu().numpy(), top.indices.cpu().numpy()
        new = sorted((-(cum[base + i] + val[i, j]), i * k + j, int(idx[i, j]), base + i) for i in range(len(batch)) for j in range(k))
        for nll, _, t, p in new[:min(K, c["B"] * k)]:
            queue.append((nll, serial, t, p))
            serial += 1
    keep = sorted(sorted(range(len(cum)), key=lambda i: (-cum[i], i))[:K])
    out = torch.zeros(K, dtype=torch.float64)
    out[:len(keep)] = torch.tensor([cum[i] for i in keep], dtype=torch.float64)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "walk":
        return None
    s = prepare(case, seed)
    if kind == "draft":
        return dict(tokens=None, parent=None, cum_logp=_draft64(s), n=None)
    if kind in ("round", "forward"):
        P, first = case["P"], case.get("first", 0)
        pk, pv = (s["k"], s["v"]) if kind == "round" else (s["pk"], s["pv"])
        lg, k, v = _forward64(s["cfg"], s["w"], pk, pv, P, s["tok"].cpu().numpy(), s["par"].cpu().numpy(), first, s.get("tk"), s.get("tv"))
        if kind == "forward":
            return dict(logits=lg, tree_k=k, tree_v=v)
        return dict(logits=lg, tree_k=k, tree_v=v, path=None, tokens=None, n=None, cache_k=None, cache_v=None)
    if kind == "attn":
        T = case["T"]
        x = s["x"].double()
        q = _rope64((x @ s["wq"].double().T).view(T, -1, 128), s["pos"])
        k = _rope64((x @ s["wk"].double().T).view(T, -1, 128), s["pos"])
        v = (x @ s["wv"].double().T).view(T, -1, 128)
        o = _attend64(q, k, v, s["pk"], s["pv"], _dev(_depth_mask(s["par"].cpu().numpy())[1]))
        return dict(q=q, k=k, v=v, o=o, y=o.reshape(T, -1) @ s["wo"].double().T)
    if kind == "mlp":
        x = s["x"].double()
        gate = x @ s["wg"].double().T
        act = gate * torch.sigmoid(gate) * (x @ s["wu"].double().T)
        return dict(act=act, y=act @ s["wd"].double().T)
    if kind == "head":
        s["logits"] = s["x"].double() @ s["w"].double().T
    best = torch.cat([torch.log_softmax(r.double(), dim=1).topk(case["k"], dim=1).values for r in s["logits"].split(256)])
    best = (best + s["cum"].double()[:, None]).reshape(-1)
    score = torch.zeros(case["B"], dtype=torch.float64, device="cuda")
    n = min(case["B"], best.numel())
    score[:n] = best.topk(n).values
    out = dict(row=None, token=None, cum_logp=score, n=None)
    return dict(out, logits=s["logits"]) if kind == "head" else out
