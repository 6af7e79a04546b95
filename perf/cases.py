"""The calls that this library is timed on: verify steps with their commit, and
KV migration, over the shapes, batch and tree sizes, cache lengths and options
that a generation loop brings.

A case names a decoder shape (the Llama-3-8B and Llama-3.2-1B shapes and the
small one of the tests), a number of layers, a batch, tree sizes and committed
lengths.  Sizes of one case are fixed by its own ``sizes`` number; the seed
draws every value: weights, cached K/V, tree shapes, tokens, draft
distributions and uniforms.

Weights follow the usual initialisation (0.02, residual products over
sqrt(2 layers)) with unit embeddings, and the LM head holds a bigram: the row
of a token's successor leans towards the token's embedding.  Greedy tokens are
thereby decided by a margin, as a trained model's are, and a draft that follows
the successor is accepted.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2512_04752_amd as sv

SHAPES = {
    "tiny": dict(hidden=256, n_heads=4, n_kv_heads=2, head_dim=64, ffn=1024, vocab=1024,
                 rope_theta=1e4),
    "1b": dict(hidden=2048, n_heads=32, n_kv_heads=8, head_dim=64, ffn=8192, vocab=128256,
               rope_theta=5e5),
    "8b": dict(hidden=4096, n_heads=32, n_kv_heads=8, head_dim=128, ffn=14336, vocab=128256,
               rope_theta=5e5),
}
STD = 0.02
TOP_LOGIT = 14.0      # logit of a token's successor
FOLLOW = 0.7          # chance that a branch's next draft token is the successor
KV_VIEWS = 24         # samples whose new K/V come back one by one


def _case(name, kind="greedy", shape="8b", layers=8, batch=1, nodes=1, ragged=False, lo=128,
          median=1024, hi=8192, sizes=1, temperature=0.0):
    return dict(name=name, kind=kind, shape=shape, layers=layers, batch=batch, nodes=nodes,
                ragged=ragged, lo=lo, median=median, hi=hi, sizes=sizes, temperature=temperature)


def listed():
    return [
        # the smallest call: a two-layer decoder on four 4-node chains, all launches and latency
        _case("tiny_b4_chain4", shape="tiny", layers=2, batch=4, nodes=4, lo=128, median=128, hi=128),
        # plain decoding of the last live sample, the whole 8B model: a stream of the weights
        _case("8b_whole_b1_n1", layers=32, batch=1, nodes=1, median=1100),
        # the same sample with a draft tree
        _case("8b_b1_n16", batch=1, nodes=16, median=1100, sizes=2),
        # a few live samples with trees of about 16 nodes each
        _case("8b_b4_n16", batch=4, nodes=16, median=2048, hi=16384, sizes=3),
        # long tail of the generation stage: four samples at 16K to 32K tokens, 64-node trees
        _case("8b_tail_b4_n64", layers=4, batch=4, nodes=64, lo=16384, median=24000, hi=32768, sizes=4),
        # 1B shape (head dim 64), 32 samples, 15-node trees
        _case("1b_b32_n15", shape="1b", layers=8, batch=32, nodes=15, lo=512, median=1100, hi=2048, sizes=5),
        # middle of the generation stage: 64 samples whose trees differ in size
        _case("8b_b64_ragged12", layers=4, batch=64, nodes=12, ragged=True, median=2048, hi=16384, sizes=6),
        # a large batch without drafts: attention over the cache
        _case("8b_b256_n1", layers=4, batch=256, nodes=1, median=2048, hi=16384, sizes=7),
        # early generation, the whole 8B model: 128 samples, 8-node trees
        _case("8b_whole_b128_n8", layers=32, batch=128, nodes=8, sizes=8),
        # early generation with acceptance at temperature 1
        _case("8b_sampled_b128_n8", kind="sampled", layers=4, batch=128, nodes=8, sizes=9,
              temperature=1.0),
        # many samples with large trees: 4096 rows through every product
        _case("8b_b64_n64", layers=4, batch=64, nodes=64, sizes=10),
        # 16 samples move to another instance's pool
        _case("8b_migrate16", kind="migrate", layers=32, batch=16, sizes=11),
    ]


def draw(rng):
    def logint(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["greedy"] * 6 + ["sampled", "migrate"])
    shape = rng.choice(["8b", "8b", "8b", "1b", "tiny"])
    c = _case("", kind=kind, shape=shape, layers=rng.randint(1, 4), ragged=rng.random() < 0.5,
              median=logint(256, 8192), hi=32768, sizes=rng.randrange(1 << 30))
    del c["name"]
    if kind == "migrate":
        c.update(batch=logint(1, 64), layers=rng.randint(2, 16))
        most_kv = 400_000 // c["layers"]
    else:
        most_rows = 1024 if kind == "sampled" else 4096
        c["batch"] = logint(1, 256)
        c["nodes"] = logint(1, max(1, min(256 if rng.random() < 0.1 else 64, most_rows // c["batch"])))
        most_kv = 400_000
    if kind == "sampled":
        c["temperature"] = rng.choice([0.7, 1.0])
    c["median"] = max(128, min(c["median"], most_kv // (2 * c["batch"])))
    c["hi"] = max(c["median"], min(c["hi"], most_kv // c["batch"]))
    return c


# ---------------------------------------------------------------------------
# sizes (from the case alone)
# ---------------------------------------------------------------------------

def _config(case):
    return SimpleNamespace(n_layers=case["layers"], rms_eps=1e-5, **SHAPES[case["shape"]])


def _sizes(case):
    """(committed lengths, tree sizes) of the samples."""
    rng = np.random.default_rng(case["sizes"])
    x = np.exp(rng.normal(math.log(case["median"]), 0.8, size=case["batch"]))
    if case["lo"] > 1024:      # long tail: spread evenly
        x = rng.uniform(case["lo"], case["hi"], size=case["batch"])
    lens = np.clip(np.rint(x), min(case["lo"], case["hi"]), case["hi"]).astype(np.int32)
    n = case["nodes"]
    trees = rng.integers(max(1, n // 2), n + n // 2 + 1, size=case["batch"]) if case["ragged"] else \
        np.full(case["batch"], n)
    return lens, np.minimum(trees, sv.SPEC_MAX_TREE).astype(np.int32)


def work(case):
    cfg = _config(case)
    lens, trees = _sizes(case)
    kv_token = cfg.n_layers * 2 * cfg.n_kv_heads * cfg.head_dim * 2
    if case["kind"] == "migrate":    # into the buffer and out of it, each byte read and written
        return {"bytes": 4 * int(lens.sum()) * kv_token, "flops": 0}
    n = int(trees.sum())
    h, d = cfg.hidden, cfg.head_dim
    layer = h * (cfg.n_heads + 2 * cfg.n_kv_heads) * d + cfg.n_heads * d * h + 3 * h * cfg.ffn
    params = cfg.n_layers * layer + cfg.vocab * h
    keys = (lens.astype(np.int64) + trees)
    flops = 2 * n * params + 4 * cfg.n_layers * cfg.n_heads * d * int((keys * trees).sum())
    logits = n * cfg.vocab * 4
    nbytes = 2 * params + int(keys.sum()) * kv_token + n * h * 2 + logits
    if case["kind"] == "sampled":    # the draft rows of the nodes that can be drawn from
        nbytes += logits
    return {"bytes": int(nbytes), "flops": int(flops)}


# ---------------------------------------------------------------------------
# values (from the seed)
# ---------------------------------------------------------------------------

def _gen(seed, what):
    return torch.Generator(device="cuda").manual_seed((seed * 1_000_003 + what) % (1 << 62))


def _normal(shape, std, gen):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)


def _successor(cfg, tok):
    return (tok * 5 + 3) % cfg.vocab         # vocab sizes are not multiples of 5: a permutation


def _layer(cfg, seed, l):
    g = _gen(seed, 100 + l)
    h, q, kv = cfg.hidden, cfg.n_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim
    out = STD / math.sqrt(2 * cfg.n_layers)

    def gain():
        return torch.empty(h, device="cuda").uniform_(0.8, 1.2, generator=g).to(torch.bfloat16)

    return {"attn_norm": gain(), "wq": _normal((q, h), STD, g), "wk": _normal((kv, h), STD, g),
            "wv": _normal((kv, h), STD, g), "wo": _normal((h, q), out, g), "ffn_norm": gain(),
            "w_gate": _normal((cfg.ffn, h), STD, g), "w_up": _normal((cfg.ffn, h), STD, g),
            "w_down": _normal((h, cfg.ffn), out, g)}


def _ends(cfg, seed):
    g = _gen(seed, 1)
    embed = _normal((cfg.vocab, cfg.hidden), 1.0, g)
    head = _normal((cfg.vocab, cfg.hidden), STD, g)
    succ = _successor(cfg, torch.arange(cfg.vocab, device="cuda"))
    lean = TOP_LOGIT / (0.55 * cfg.hidden)   # 0.55: share of the embedding in the last hidden state
    for at in range(0, cfg.vocab, 16384):
        rows = succ[at:at + 16384]
        head[rows] = (head[rows].float() + lean * embed[at:at + 16384].float()).to(torch.bfloat16)
    return embed, torch.ones(cfg.hidden, dtype=torch.bfloat16, device="cuda"), head


def _prefix(cfg, seed, sample, length):
    """Committed K/V of one sample, [layers, K/V, kv heads, length, head_dim]."""
    return _normal((cfg.n_layers, 2, cfg.n_kv_heads, length, cfg.head_dim),
                   STD * math.sqrt(cfg.hidden), _gen(seed, 100_000 + sample))


def _tree(rng, n):
    """Parents of a tree of n nodes, at most 8 levels (a chain up to 4 nodes), 4 children each."""
    if n <= 4:
        return [-1] + list(range(n - 1))
    parents, depth, kids = [-1], [0], [0]
    while len(parents) < n:
        fit = [i for i in range(len(parents)) if depth[i] < 7 and kids[i] < 4]
        p = fit[-1] if len(parents) < 4 else fit[int(rng.integers(len(fit)))]
        kids[p] += 1
        parents.append(p)
        depth.append(depth[p] + 1)
        kids.append(0)
    return parents


def _drafts(case, cfg, seed):
    """Flat trees: offsets, tokens, parents (int32), and, for sampling, the draft distributions
    (each child is a draw of its parent's) and the uniforms."""
    _, trees = _sizes(case)
    rng = np.random.default_rng([seed, 7])
    offsets = np.concatenate([[0], np.cumsum(trees)]).astype(np.int32)
    n = int(offsets[-1])
    parents = np.concatenate([_tree(rng, int(t)) for t in trees]).astype(np.int32)
    tokens = rng.integers(0, cfg.vocab, size=n).astype(np.int32)
    follow = rng.random(n) < FOLLOW
    noise = None
    if case["kind"] == "sampled":
        g = _gen(seed, 2)
        noise = torch.empty(n, cfg.vocab, device="cuda").normal_(0.0, STD * math.sqrt(cfg.hidden), generator=g)
        drawn = torch.multinomial(torch.softmax(noise, -1), 4, replacement=True, generator=g).cpu().numpy()
    for b in range(len(trees)):
        born = {}
        for i in range(offsets[b] + 1, offsets[b + 1]):
            up = int(offsets[b] + parents[i])
            if follow[i]:
                tokens[i] = _successor(cfg, int(tokens[up]))
            elif noise is not None:
                tokens[i] = drawn[up, born.get(up, 0) % 4]
            born[up] = born.get(up, 0) + 1
    if noise is None:
        return (offsets, tokens, parents), None, None
    succ = _successor(cfg, torch.from_numpy(tokens.astype(np.int64)).cuda())
    noise.scatter_(1, succ[:, None], TOP_LOGIT)
    uniforms = torch.rand(n, 2, generator=g, device="cuda")
    return (offsets, tokens, parents), torch.softmax(noise, -1), uniforms


def _fill(pool, cfg, seed, lens):
    for b, s in enumerate(lens):
        kv = _prefix(cfg, seed, b, int(s))
        k, v = pool.sample_view(b)
        k[:, :, :int(s)] = kv[:, 0]
        v[:, :, :int(s)] = kv[:, 1]


# ---------------------------------------------------------------------------
# the pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    cfg = _config(case)
    lens, trees = _sizes(case)
    batch = len(lens)
    ids = np.arange(batch, dtype=np.int32)
    if case["kind"] == "migrate":
        src, dst = sv.KVPool(cfg, lens), sv.KVPool(cfg, lens)
        _fill(src, cfg, seed, lens)
        dst.buf.zero_()
        begin = np.zeros(batch, np.int32)
        nbytes = sv.spec_kv_transfer_bytes(src, begin, lens)
        buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        got = [dst.sample_view(b) for b in range(min(batch, KV_VIEWS))]
        return dict(case=case, src=src, dst=dst, ids=ids, begin=begin, end=lens, buf=buf,
                    out={"buffer": buf.view(torch.bfloat16), "kv": got})
    flat, draft, uniforms = _drafts(case, cfg, seed)
    embed, final, head = _ends(cfg, seed)
    W = {"tok_embed": embed, "final_norm": final, "lm_head": head,
         "layers": [_layer(cfg, seed, l) for l in range(cfg.n_layers)]}
    n = int(trees.sum())
    ver = sv.Verifier(cfg, W, lens + trees, batch, n, sampling=case["kind"] == "sampled")
    _fill(ver.kv, cfg, seed, lens)
    new = []
    for b in range(min(batch, KV_VIEWS)):
        k, v = ver.kv.sample_view(b)
        at = slice(int(lens[b]), int(lens[b] + trees[b]))
        new.append((k[:, :, at], v[:, :, at]))
    debug = {"logits": torch.empty(n, cfg.vocab, dtype=torch.float32, device="cuda")}
    return dict(case=case, ver=ver, ids=ids, flat=flat, lens=lens, debug=debug, draft=draft,
                uniforms=uniforms, kv=new)


def run(state):
    """A verify step and its commit: logits, acceptance, new lengths and the trees' K/V; or a
    migration: pack and unpack."""
    s = state
    if "src" in s:
        sv.spec_kv_pack(s["src"], s["ids"], s["begin"], s["end"], s["buf"])
        sv.spec_kv_unpack(s["dst"], s["ids"], s["begin"], s["end"], s["buf"])
        return s["out"]
    ver = s["ver"]
    if s["draft"] is None:
        acc, nxt, nodes = ver.verify(s["ids"], None, s["lens"], debug=s["debug"], flat=s["flat"])
    else:
        acc, nxt, nodes = ver.verify_sampled(s["ids"], None, s["lens"], s["case"]["temperature"],
                                             eos_token=2, draft_probs=s["draft"],
                                             uniforms=s["uniforms"], debug=s["debug"],
                                             flat=s["flat"])
    lens = ver.commit(s["ids"], s["lens"])
    out = {"logits": s["debug"]["logits"], "accepted_nodes": nodes, "new_lens": lens, "kv": s["kv"]}
    if s["draft"] is None:     # a sampled token lies where a sum of 128K shares passes a uniform:
        out["next"] = nxt      # the last bit of a logit moves it, so it cannot be compared
        out["accepted_len"] = acc
    return out


def tolerance(case):
    if case["kind"] == "migrate":
        return "exact"
    # Activations are rounded to bf16 at every product; a whole model passes that on through 32
    # layers.  Acceptance turns on margins, except where a uniform falls next to a threshold.
    return {"rel": 0.02 if case["layers"] > 8 else 0.01, "max": 0.2, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def exact(case, seed):
    cfg = _config(case)
    lens, trees = _sizes(case)
    f64 = torch.float64
    if case["kind"] == "migrate":
        every = [_prefix(cfg, seed, b, int(s)) for b, s in enumerate(lens)]
        buf = torch.cat([p[l, w].reshape(-1) for l in range(cfg.n_layers) for w in range(2) for p in every])
        return {"buffer": buf, "kv": [(p[:, 0], p[:, 1]) for p in every[:KV_VIEWS]]}
    (offsets, tokens, parents), _, _ = _drafts(case, cfg, seed)
    batch, n = len(lens), int(offsets[-1])
    d, half, group = cfg.head_dim, cfg.head_dim // 2, cfg.n_heads // cfg.n_kv_heads
    depth = np.zeros(n, np.int64)
    sees = []
    for b in range(batch):
        t0, t = int(offsets[b]), int(trees[b])
        m = np.eye(t, dtype=bool)
        for i in range(1, t):
            p = int(parents[t0 + i])
            depth[t0 + i] = depth[t0 + p] + 1
            m[i] |= m[p]
        sees.append(torch.from_numpy(m).cuda())
    pos = torch.from_numpy(np.repeat(lens, trees).astype(np.int64) + depth).cuda()
    freq = cfg.rope_theta ** (-2.0 * torch.arange(half, dtype=f64, device="cuda") / d)
    cos, sin = torch.cos(pos[:, None] * freq)[:, None], torch.sin(pos[:, None] * freq)[:, None]

    def norm(x, gain):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * gain.to(f64)

    def turn(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    embed, final, head = _ends(cfg, seed)
    x = embed[torch.from_numpy(tokens.astype(np.int64)).cuda()].to(f64)
    del embed
    shown = min(batch, KV_VIEWS) if case["kind"] == "greedy" else 0
    new = [([], []) for _ in range(shown)]
    # the cached K/V of a few samples at a time is enough: one layer of all of them is kept
    cached = [_prefix(cfg, seed, b, int(s)) for b, s in enumerate(lens)]
    for l in range(cfg.n_layers):
        w = _layer(cfg, seed, l)
        h = norm(x, w["attn_norm"])
        q = turn((h @ w["wq"].to(f64).T).view(n, cfg.n_heads, d))
        k = turn((h @ w["wk"].to(f64).T).view(n, cfg.n_kv_heads, d))
        v = (h @ w["wv"].to(f64).T).view(n, cfg.n_kv_heads, d)
        o = torch.empty(n, cfg.n_kv_heads, group, d, dtype=f64, device="cuda")
        for b in range(batch):
            t0, t, s = int(offsets[b]), int(trees[b]), int(lens[b])
            at = slice(t0, t0 + t)
            kb = torch.cat([cached[b][l, 0].to(f64), k[at].transpose(0, 1)], 1)
            vb = torch.cat([cached[b][l, 1].to(f64), v[at].transpose(0, 1)], 1)
            qb = q[at].view(t, cfg.n_kv_heads, group, d).permute(1, 2, 0, 3).reshape(cfg.n_kv_heads, group * t, d)
            score = torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(d)
            score.view(cfg.n_kv_heads, group, t, s + t)[..., s:].masked_fill_(~sees[b], -math.inf)
            ob = torch.matmul(torch.softmax(score, -1), vb).view(cfg.n_kv_heads, group, t, d)
            o[at] = ob.permute(2, 0, 1, 3)
            if b < shown:
                new[b][0].append(k[at].transpose(0, 1).clone())
                new[b][1].append(v[at].transpose(0, 1).clone())
        x = x + o.view(n, -1) @ w["wo"].to(f64).T
        h = norm(x, w["ffn_norm"])
        act = torch.nn.functional.silu(h @ w["w_gate"].to(f64).T) * (h @ w["w_up"].to(f64).T)
        x = x + act @ w["w_down"].to(f64).T
    del cached
    h = norm(x, final)
    logits = torch.empty(n, cfg.vocab, dtype=f64, device="cuda")
    for at in range(0, cfg.vocab, 16384):
        logits[:, at:at + 16384] = h @ head[at:at + 16384].to(f64).T
    out = {"logits": logits, "accepted_nodes": None, "new_lens": None, "kv": None}
    if case["kind"] == "greedy":
        best = logits.argmax(-1).cpu().numpy()
        kv = [(torch.stack(a), torch.stack(c)) for a, c in new]
        for b in range(shown):     # commit: row d takes the accepted branch's node at depth d
            t0 = int(offsets[b])
            ok, end = [True], 0
            for i in range(1, int(trees[b])):
                p = int(parents[t0 + i])
                ok.append(ok[p] and int(tokens[t0 + i]) == int(best[t0 + p]))
                if ok[i] and depth[t0 + i] > depth[t0 + end]:
                    end = i
            path = []
            while end != -1:
                path.append(end)
                end = int(parents[t0 + end])
            for y in kv[b]:
                y[:, :, :len(path)] = y[:, :, path[::-1]].clone()
        out.update(kv=kv, next=None, accepted_len=None)
    return out
