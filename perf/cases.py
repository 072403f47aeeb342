"""What a program that decodes with this library has it do, as cases that can be timed and compared.

Six kinds of work, all through the public binding:
  step     one speculative step of one sequence: feature fusion, draft-tree expansion, tree verification, greedy walk
  verify   verification of the trees of a ragged batch and the greedy walk (no drafting)
  chain    one cycle of the batched serving loop: fusion, chain drafting, verification, greedy walk, commit
  prefill  a prompt through target and draft: both caches filled, features and logits of the last position
  accept   the acceptance walk alone on given logits, greedy or at a temperature
  ttt      self-attention of the draft layer during a training-time-test step, forward

Model shapes are the repository's own (eagle3_synth.get_shape): c1 tiny fp32, c3 LLaMA-3.1-8B, c5 LLaMA-3.3-70B; "mid" is the
small bf16 model of the tests.  `layers` cuts the target stack (a pipeline stage, or the one-layer configuration).

Weights are random, but placed so that the model has what a trained one has: a next token that is ahead of the rest by
several nats.  The embedding rows dominate the residual stream (the outputs of the attention and MLP blocks are scaled
by 1/sqrt(2 layers), as at the start of training), and the LM head's row of token successor[t] carries a share of
embedding row t.  The draft's LM head does the same for a set of contexts from which the recorded features are taken.
With purely random rows the first and the second of 128 k tokens lie 0.2 nats apart, and every last bit of an
activation would turn greedy tokens over.
"""
import math

import numpy as np
import torch

import eagle3_synth as S
import paper_2503_01840_amd as E

DEV = "cuda:0"
CONTEXTS = 256            # feature vectors that recorded features are drawn from
TOP_LOGIT = 14.0          # planted next-token logit; the others are N(0, 1.3^2): at 128 k tokens it holds ~4/5 of the mass
DRAFT_LOGIT = 19.0        # the same at the first drafted level; some 13 at the second, where the context is less clear


# ------------------------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest calls: a tiny exact-arithmetic model, where every launch counts
        dict(name="step-tiny", kind="step", model="c1", layers=4, prefix=64, n_new=2, depth=3, topk=4, nodes=16),
        # one decoder layer + LM head of the 8B model under a 60-node tree
        dict(name="step-8b-1layer", kind="step", model="c3", layers=1, prefix=2048, n_new=4, depth=6, topk=10, nodes=60),
        # the headline: a whole step of the 8B model at batch 1, four tokens accepted by the step before
        dict(name="step-8b", kind="step", model="c3", layers=32, prefix=4096, n_new=4, depth=8, topk=10, nodes=60),
        # a pipeline stage of the 70B model with its draft, at a reasoning-length context
        dict(name="step-70b-stage", kind="step", model="c5", layers=16, prefix=16384, n_new=4, depth=6, topk=10, nodes=60),
        # a handful of sequences with trees of an odd size: more than 64 rows, fewer than a full tile of the batched GEMM
        dict(name="verify-4x29", kind="verify", model="c3", layers=8, batch=4, nodes=29, lo=300, hi=3000),
        # the throughput regime: 64 ragged sequences, 8-node trees, all 32 layers
        dict(name="verify-64x8", kind="verify", model="c3", layers=32, batch=64, nodes=8, lo=512, hi=2048),
        # the serving loop at batch 64: chains of three, up to four positions accepted per sequence
        dict(name="chain-64x3", kind="chain", model="c3", layers=32, batch=64, length=3, rows=4, lo=512, hi=2048),
        # the walk at temperature 1 over the logits of 64 8-node trees
        dict(name="accept-64x8-sampled", kind="accept", vocab=128256, batch=64, nodes=8, temperature=1.0),
        # a short chat turn and an ordinary prompt
        dict(name="prefill-77", kind="prefill", model="c3", layers=32, tokens=77),
        dict(name="prefill-2048", kind="prefill", model="c3", layers=32, tokens=2048),
        # training-time test: an ordinary training length at the third step, and a ragged one of the 70B draft
        dict(name="ttt-2048", kind="ttt", dtype="bf16", tokens=2048, heads=32, kv_heads=8, dim=128, step=2),
        dict(name="ttt-517", kind="ttt", dtype="bf16", tokens=517, heads=64, kv_heads=8, dim=128, step=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "verify", "chain", "prefill", "accept", "ttt"])
    if kind == "step":
        model = rng.choice(["c1", "mid", "c3", "c3", "c5"])
        depth, topk = rng.randint(2, 8), rng.randint(2, 10)
        pool = 1 + topk + (depth - 1) * topk * topk
        return dict(kind=kind, model=model, layers=4 if model == "c1" else _log(rng, 1, 8 if model == "c5" else 16),
                    prefix=_log(rng, 48, 512 if model == "c1" else 12000), n_new=rng.randint(1, 8), depth=depth, topk=topk,
                    nodes=rng.randint(min(8, pool), min(60, pool)))
    if kind == "verify":
        batch = _log(rng, 1, 64)
        lo = _log(rng, 40, 1500)
        return dict(kind=kind, model=rng.choice(["mid", "c3", "c3"]), layers=_log(rng, 1, 8), batch=batch,
                    nodes=rng.randint(1, min(60, max(4, 640 // batch))), lo=lo, hi=rng.randint(lo, 2 * lo + 500))
    if kind == "chain":
        lo = _log(rng, 40, 1500)
        return dict(kind=kind, model=rng.choice(["mid", "c3", "c3"]), layers=_log(rng, 1, 8), batch=_log(rng, 1, 64),
                    length=rng.randint(1, 5), rows=rng.randint(1, 4), lo=lo, hi=rng.randint(lo, 2 * lo + 500))
    if kind == "prefill":
        model = rng.choice(["c1", "mid", "c3", "c3", "c3"])
        return dict(kind=kind, model=model, layers=4 if model == "c1" else _log(rng, 1, 14),
                    tokens=_log(rng, 8, 400 if model == "c1" else 4096))
    if kind == "accept":
        batch = _log(rng, 1, 64)
        return dict(kind=kind, vocab=rng.choice([32000, 128256]), batch=batch, nodes=rng.randint(1, min(60, 640 // batch)),
                    temperature=rng.choice([0.0, 0.7, 1.0]))
    heads, kv_heads = rng.choice([(32, 8), (64, 8), (8, 8), (4, 4)])
    if rng.random() < 0.2:                                        # the exact kernels, at the sizes they are meant for
        return dict(kind="ttt", dtype="fp32", tokens=_log(rng, 16, 256), heads=4, kv_heads=rng.choice([1, 2, 4]), dim=64,
                    step=rng.randint(0, 6))
    return dict(kind="ttt", dtype="bf16", tokens=_log(rng, 33, 4096), heads=heads, kv_heads=kv_heads, dim=128,
                step=rng.randint(0, 6))


# ------------------------------------------------------------------------------------------------------------ inputs
def _shape(case):
    if case["model"] == "mid":
        s = S.get_shape("c3").with_(name="mid", hidden=512, n_heads=8, n_kv_heads=2, intermediate=1024, vocab=4096,
                                    draft_vocab=2048)
    else:
        s = S.get_shape(case["model"])
    L = case["layers"]
    taps = s.taps if L == s.n_layers else (0, L // 2, L - 1)
    return s.with_(n_layers=L, taps=taps)


def _normal(gen, dims, std=1.0, mean=0.0, dtype=torch.float32):
    return torch.empty(dims, dtype=dtype, device=DEV).normal_(mean, std, generator=gen)


def _ints(gen, dims, lo, hi):
    return torch.randint(lo, hi, dims, dtype=torch.int32, device=DEV, generator=gen)


def _i32(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.int32, device=DEV)


def _layer(gen, s, fan_in, damp, dt):
    k, I = s.hidden, s.intermediate
    w = lambda n, m, std=0.02: _normal(gen, (n, m), std, 0.0, dt)  # noqa: E731
    return {"wq": w(s.q_dim, fan_in), "wk": w(s.kv_dim, fan_in), "wv": w(s.kv_dim, fan_in), "wo": w(k, s.q_dim, 0.02 * damp),
            "w_gate": w(I, k), "w_up": w(I, k), "w_down": w(k, I, 0.02 * damp),
            "norm_attn": _normal(gen, (k,), 0.02, 1.0, dt), "norm_mlp": _normal(gen, (k,), 0.02, 1.0, dt)}


def _target(gen, s, dt, own=None):
    """Target weights and the successor of every token; tokens in `own` are their own successors."""
    k, V = s.hidden, s.vocab
    damp = 1.0 / math.sqrt(2.0 * s.n_layers)
    layers = [_layer(gen, s, k, damp, dt) for _ in range(s.n_layers)]
    embed = _normal(gen, (V, k), 1.0, 0.0, dt)
    lm_head = _normal(gen, (V, k), 0.02, 0.0, dt)
    others = torch.ones(V, dtype=torch.bool, device=DEV)
    if own is not None:
        others[own] = False
    others = others.nonzero()[:, 0]
    successor = torch.arange(V, device=DEV)
    successor[others] = others[torch.randperm(others.numel(), device=DEV, generator=gen)]
    lm_head[successor] += embed * (TOP_LOGIT / (0.52 * k))           # 0.52: cosine of the final stream and the embedding
    return {"layers": layers, "embed": embed, "final_norm": _normal(gen, (k,), 0.02, 1.0, dt), "lm_head": lm_head}, successor


def _draft(gen, s, dt):
    """Draft weights, the low / mid / high features of the contexts its LM head knows, and the contexts' tokens."""
    k, Vd = s.hidden, s.draft_vocab
    layer = _layer(gen, s, 2 * k, math.sqrt(0.5), dt)
    del layer["norm_attn"]
    w_fc = _normal(gen, (k, 3 * k), 0.02, 0.0, dt)
    contexts = _normal(gen, (3, CONTEXTS, k))
    fused = torch.cat(list(contexts), 1) @ w_fc.float().t()
    fused /= fused.square().mean(1, keepdim=True).sqrt()
    lm_head = _normal(gen, (Vd, k), 0.02, 0.0, dt)
    own = torch.randperm(Vd, device=DEV, generator=gen)[:CONTEXTS]
    lm_head[own] += (fused * (DRAFT_LOGIT / (0.8 * k))).to(dt)
    d2t = torch.arange(Vd, dtype=torch.int64, device=DEV) * s.vocab // Vd
    return {"w_fc": w_fc, "layer": layer, "norm_embed": _normal(gen, (k,), 0.02, 1.0, dt),
            "norm_feat": _normal(gen, (k,), 0.02, 1.0, dt), "final_norm": _normal(gen, (k,), 0.02, 1.0, dt),
            "lm_head": lm_head, "d2t": d2t.to(torch.int32)}, contexts, d2t[own].to(torch.int32)


def _caches(gen, s, n_layers, slots, dt):
    """One tensor [layers, 2, slots, Hkv, d] and its per-layer key and value views."""
    kv = _normal(gen, (n_layers, 2, slots, s.n_kv_heads, s.head_dim), 1.0, 0.0, dt)
    return kv, [kv[l, 0] for l in range(n_layers)], [kv[l, 1] for l in range(n_layers)]


def _features(gen, contexts, rows):
    """Recorded features of `rows` positions, each near those of a context, and which context."""
    pick = torch.randint(0, CONTEXTS, (rows,), device=DEV, generator=gen)
    return (contexts[:, pick] + 0.1 * _normal(gen, (3, rows, contexts.shape[2]))).contiguous(), pick


def _trees(seed, batch, nodes, successor, vocab):
    """Random trees of at most two children per node in the order a level-by-level drafter emits; the first child of a node
    holds the target's next token in two cases of three."""
    rs = np.random.RandomState(seed % (2 ** 31 - 1))
    succ = successor.cpu().numpy()
    parent = np.empty((batch, nodes), np.int32)
    tok = rs.randint(0, vocab, (batch, nodes)).astype(np.int32)
    for b in range(batch):
        parent[b] = S.random_tree(seed, 7919 * b + 1, nodes, 8, 2)[0]
        first = set()
        for i in range(1, nodes):
            p = int(parent[b, i])
            if p not in first and rs.random_sample() < 0.67:
                tok[b, i] = succ[tok[b, p]]
            first.add(p)
    return _i32(tok), _i32(parent)


def _ragged(seed, case, extra):
    rs = np.random.RandomState((seed + 17) % (2 ** 31 - 1))
    plen = rs.randint(case["lo"], case["hi"] + 1, case["batch"])
    return plen, np.concatenate([[0], np.cumsum(plen + extra)])


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    st = {"case": dict(case)}
    if kind == "ttt":
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        T, H, G, d = case["tokens"], case["heads"], case["kv_heads"], case["dim"]
        st["q"] = _normal(gen, (T, H, d), 1.0, 0.0, dt)
        st["k"] = _normal(gen, (case["step"] + 1, T, G, d), 1.0, 0.0, dt)
        st["v"] = _normal(gen, (case["step"] + 1, T, G, d), 1.0, 0.0, dt)
        return st
    if kind == "accept":
        B, N, V = case["batch"], case["nodes"], case["vocab"]
        st["successor"] = torch.randperm(V, device=DEV, generator=gen)
        st["tok"], st["parent"] = _trees(seed, B, N, st["successor"], V)
        logits = _normal(gen, (B * N, V), 1.3)
        ahead = TOP_LOGIT + _normal(gen, (B * N,), 1.0)
        logits[torch.arange(B * N, device=DEV), st["successor"][st["tok"].reshape(-1).long()]] = ahead
        st["logits"] = logits.reshape(B, N, V)
        st["uniforms"] = torch.rand(B, 2 * N, device=DEV, generator=gen)
        st["ctx"] = E.Eagle3Context(S.get_shape("c1"), vocab=V, max_batch=B, max_nodes=N, max_depth=2, max_topk=2, max_new=1)
        return st
    s = _shape(case)
    dt = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    draft = contexts = own = None
    if kind != "verify":
        draft, contexts, own = _draft(gen, s, dt)
    target, successor = _target(gen, s, dt, own)
    if kind == "step":
        st["ctx"] = E.Eagle3Context(s, max_batch=1, max_nodes=64, max_depth=8, max_topk=10, max_new=8)
        P, N, n_new, D, K = case["prefix"], case["nodes"], case["n_new"], case["depth"], case["topk"]
        plen = _i32([P])
        _, ks, vs = _caches(gen, s, s.n_layers, P + N, dt)
        st["kv"] = E.KVCache(ks, vs, _i32([0, P + N]), plen, P)
        slots = P + n_new + (D - 1) * K
        _, dk, dv = _caches(gen, s, 1, slots, dt)
        st["dkv"] = E.KVCache(dk, dv, _i32([0, slots]), plen.clone(), P)
        st["taps"], near = _features(gen, contexts, n_new)
        st["tok_new"] = _ints(gen, (n_new,), 0, s.vocab)
        st["tok_new"][-1] = own[near[-1]]
        st["logits"] = torch.empty(1, N, s.vocab, device=DEV)
        st["taps_out"] = torch.empty(3, 1, N, s.hidden, device=DEV)
    elif kind == "verify":
        B, N = case["batch"], case["nodes"]
        st["ctx"] = E.Eagle3Context(s, max_batch=B, max_nodes=N, max_depth=4, max_topk=2, max_new=8)
        plen, indptr = _ragged(seed, case, N)
        _, ks, vs = _caches(gen, s, s.n_layers, int(indptr[-1]), dt)
        st["kv"] = E.KVCache(ks, vs, _i32(indptr), _i32(plen), int(plen.max()))
        st["tok"], st["parent"] = _trees(seed, B, N, successor, s.vocab)
        st["logits"] = torch.empty(B, N, s.vocab, device=DEV)
        st["taps_out"] = torch.empty(3, B, N, s.hidden, device=DEV)
    elif kind == "chain":
        B, rows, N = case["batch"], case["rows"], case["length"] + 1
        st["ctx"] = E.Eagle3Context(s, max_batch=B, max_nodes=max(N, rows, 8), max_depth=8, max_topk=2, max_new=64)
        plen, indptr = _ragged(seed, case, rows + N)
        _, ks, vs = _caches(gen, s, s.n_layers, int(indptr[-1]), dt)
        st["plen0"] = _i32(plen)
        st["kv"] = E.KVCache(ks, vs, _i32(indptr), st["plen0"].clone(), int(plen.max()))
        _, dk, dv = _caches(gen, s, 1, int(indptr[-1]), dt)
        st["dkv"] = E.KVCache(dk, dv, _i32(indptr), st["plen0"].clone(), int(plen.max()))
        st["taps"], near = _features(gen, contexts, B * rows)
        st["tok_new"] = _ints(gen, (B, rows), 0, s.vocab)
        st["n_new"] = _ints(gen, (B,), 1, rows + 1)
        good = torch.rand(B, rows, device=DEV, generator=gen) < 0.67
        st["tok_new"][good] = own[near].reshape(B, rows)[good]
        st["parent"] = _i32(np.tile(np.arange(-1, N - 1), (B, 1)))
        st["logits"] = torch.empty(B, N, s.vocab, device=DEV)
        st["taps_out"] = torch.empty(3, B, N, s.hidden, device=DEV)
    else:
        T = case["tokens"]
        st["ctx"] = E.Eagle3Context(s, max_batch=1, max_nodes=64, max_depth=8, max_topk=10, max_new=64)
        st["kv_all"], ks, vs = _caches(gen, s, s.n_layers, T, dt)
        st["dkv_all"], dk, dv = _caches(gen, s, 1, T - 1, dt)
        st["kv"] = E.KVCache(ks, vs, _i32([0, T]), _i32([0]), 0)
        st["dkv"] = E.KVCache(dk, dv, _i32([0, T - 1]), _i32([0]), 0)
        st["tokens"] = _ints(gen, (T,), 0, s.vocab)
    st["ctx"].set_weights(target, draft)
    return st


# -------------------------------------------------------------------------------------------------------------- run
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "ttt":
        return E.eagle3_ttt_attention(st["q"], st["k"], st["v"])
    ctx = st["ctx"]
    if kind == "accept":
        t = case["temperature"]
        return E.eagle3_accept(ctx, st["logits"], st["tok"], st["parent"], t, st["uniforms"] if t > 0 else None)
    if kind == "verify":
        logits, taps = E.eagle3_tree_verify(ctx, st["tok"], st["parent"], st["kv"], logits=st["logits"], taps=st["taps_out"])
        return logits, taps, E.eagle3_accept(ctx, logits, st["tok"], st["parent"])
    if kind == "step":
        taps = st["taps"]
        g = E.eagle3_fuse_features(ctx, taps[0], taps[1], taps[2])
        tree = E.eagle3_draft_expand(ctx, g, st["tok_new"], st["dkv"], case["depth"], case["topk"], case["nodes"])
        tok, parent = tree["tree_tok"][None], tree["parent"][None]
        logits, taps_out = E.eagle3_tree_verify(ctx, tok, parent, st["kv"], logits=st["logits"], taps=st["taps_out"])
        return g, tree, logits, taps_out, E.eagle3_accept(ctx, logits, tok, parent)
    if kind == "chain":
        B, rows, N = case["batch"], case["rows"], case["length"] + 1
        kv, dkv, taps = st["kv"], st["dkv"], st["taps"]
        kv.prefix_len.copy_(st["plen0"])                             # the same contexts on every pass
        dkv.prefix_len.copy_(st["plen0"])
        g = torch.cat([E.eagle3_fuse_features(ctx, *(taps[t, i:i + 64] for t in range(3))) for i in range(0, B * rows, 64)])
        tok, logp = E.eagle3_draft_chain(ctx, g.reshape(B, rows, -1), st["tok_new"], st["n_new"], dkv, case["length"])
        logits, taps_out = E.eagle3_tree_verify(ctx, tok, st["parent"], kv, logits=st["logits"], taps=st["taps_out"])
        walk = E.eagle3_accept(ctx, logits, tok, st["parent"])
        nxt = E.eagle3_commit(ctx, tok, walk[1], walk[0], walk[2], kv, taps_out, N, draft_kv=dkv, draft_rows=rows)
        return tok, logp, logits, taps_out, walk, nxt, kv.prefix_len
    kv, dkv = st["kv"], st["dkv"]
    kv.prefix_len.zero_()                                            # a new prompt: both caches empty
    dkv.prefix_len.zero_()
    kv.set_max_prefix_len(0)
    dkv.set_max_prefix_len(0)
    g_last, logits = E.eagle3_prefill(ctx, st["tokens"], kv, dkv)
    return g_last, logits, st["kv_all"], st["dkv_all"]


# -------------------------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "ttt":
        T, H, G, d, s = case["tokens"], case["heads"], case["kv_heads"], case["dim"], case["step"]
        b = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": T * H * d * (b + 4) + 2 * (s + 1) * T * G * d * b, "flops": 4.0 * (T * (T + 1) / 2 + s * T) * d * H}
    if kind == "accept":
        return {"bytes": 4.0 * case["batch"] * case["nodes"] * case["vocab"], "flops": 0.0}
    s = _shape(case)
    b = 2 if s.dtype == "bf16" else 4
    k, V, Vd, L = s.hidden, s.vocab, s.draft_vocab, s.n_layers
    layer, draft_layer, head, dhead, fc = s.layer_params(), s.draft_layer_params(), V * k, Vd * k, 3 * k * k
    kv_row = 2 * s.kv_dim * b
    attn = lambda rows, keys: 4.0 * rows * keys * s.q_dim  # noqa: E731

    def verify(rows, keys, pairs):
        by = b * (L * layer + head) + L * kv_row * (keys + rows) + 4 * rows * (V + 3 * k)
        return by, 2.0 * rows * (L * layer + head) + L * attn(1, pairs)

    if kind == "step":
        P, N, n_new, D, K = case["prefix"], case["nodes"], case["n_new"], case["depth"], case["topk"]
        by, fl = verify(N, P, N * P)
        # the D draft forwards depend on each other and no cache holds the draft's weights: once per forward
        by += b * (fc + D * (draft_layer + dhead)) + D * kv_row * P + 3 * 4 * n_new * k
        rows = n_new + (D - 1) * K
        fl += 2.0 * (n_new * fc + rows * (draft_layer + dhead)) + attn(rows, P)
        return {"bytes": by, "flops": fl}
    if kind == "prefill":
        T = case["tokens"]
        by = b * (L * layer + head + fc + 4 * k * s.kv_dim) + (L + 1) * kv_row * T + b * k * T
        fl = 2.0 * T * (L * layer + fc + 4 * k * s.kv_dim) + 2.0 * head + L * attn(1, T * (T + 1) / 2)
        return {"bytes": by, "flops": fl}
    B = case["batch"]
    keys = B * (case["lo"] + case["hi"]) / 2.0
    if kind == "verify":
        by, fl = verify(B * case["nodes"], keys, keys * case["nodes"])
        return {"bytes": by, "flops": fl}
    N, rows, length = case["length"] + 1, case["rows"], case["length"]
    by, fl = verify(B * N, keys, keys * N)
    by += b * (fc + length * (draft_layer + dhead)) + length * kv_row * keys + 3 * 4 * B * rows * k
    fl += 2.0 * B * (rows * (fc + draft_layer) + (length - 1) * draft_layer + length * dhead) + attn(rows + length - 1, keys)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # Four times what the present kernels differ by from themselves with their sums in another order (the same rows through the
    # few-row and the many-row products; prompts in other chunks), from fp64 where the sums are fp32: one bf16 layer 1.5e-3
    # (largest 1.2e-2), 8 layers 4.7e-3 (2.7e-2), 32 layers 6.2e-3 (3.4e-2); attention alone 1.8e-6 (2.2e-5) in bf16, which
    # carries exp(S) with 16 bits, and 2.4e-7 (2.3e-6) in fp32.
    if case["kind"] == "accept":
        return "exact"
    if case["kind"] == "ttt":
        return {"rel": 8e-6, "max": 1e-4} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    if case["model"] == "c1":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.08, "differ": 0.01} if case["layers"] <= 2 else {"rel": 2.5e-2, "max": 0.15, "differ": 0.01}
