"""Workloads that the framework's speed is judged on.

The framework decodes one image (or a batch of images) by draft-then-verify cycles; a case is
one call of that work through the public entry points of `paper_2512_21857_amd.runtime`, at
the shapes of this repository's configurations: the tiny fp32 model, the LlamaGen-XL shape
(d 1280, 20 heads of 64, FFN 3584), and the 7B shape of Lumina and Anole (d 4096, 32 heads of
128, FFN 11008).  Models keep two to four of their layers, so that a rounding travels through
a few layers only; layer shapes, image vocabularies, prompts and tree sizes are the real ones.

Kinds
  verify   one tree-masked target forward over a drafted tree at the start of an image
  draft    one draft-head forward of the tree's root and its top-k children (a one-layer tree)
  prefill  a new session for an image and its prompt through target and draft head
  attn     tree attention of one image or of many images over their caches
  gemm     a projection of many trees' rows at once (packed weights)
  accept   sampled acceptance (exact or codebook-relaxed) of a verified tree
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2512_21857_amd import runtime as rt

MODELS = {
    #                 layers d_model heads head_dim ffn  vocab  image ids
    "tiny":     dict(layers=2, d=256, heads=4, dh=64, ffn=1024, vocab=1056, img=1024, dtype="f32", grid=16, prompt=64),
    "llamagen": dict(layers=4, d=1280, heads=20, dh=64, ffn=3584, vocab=16384, img=16384, dtype="bf16", grid=32,
                     prompt=120),
    "anole":    dict(layers=2, d=4096, heads=32, dh=128, ffn=11008, vocab=16384, img=8192, dtype="bf16", grid=32,
                     prompt=64),
    "lumina":   dict(layers=2, d=4096, heads=32, dh=128, ffn=11008, vocab=65536, img=65536, dtype="bf16", grid=48,
                     prompt=64),
}
# (N, K) of the projections of the two bf16 model shapes: QKV, O, gate and up, down, LM head
PROJECTIONS = {
    "llamagen": [(3840, 1280), (1280, 1280), (7168, 1280), (1280, 3584), (16384, 1280)],
    "7b": [(12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008), (8192, 4096)],
}


def listed():
    return [
        # the fp32 model that the parity runs decode whole images with: the smallest whole call
        dict(name="tiny_verify_17", kind="verify", model="tiny", n=17, prompt=64, guided=False),
        # LlamaGen-XL's most common cycle (a one-layer, ten-wide tree): its root's draft forward
        # with the top-k, and its 11-row verify; latency of many short launches
        dict(name="llamagen_draft_10", kind="draft", model="llamagen", k=10, prompt=120),
        dict(name="llamagen_verify_11", kind="verify", model="llamagen", n=11, prompt=120, guided=False),
        # a new image: session set-up and the prompt's 120 rows through target and draft head
        dict(name="llamagen_prefill_120", kind="prefill", model="llamagen", prompt=120),
        # the 7B draft forward at one row over the full vocabulary: plain weight streaming
        dict(name="lumina_draft_10", kind="draft", model="lumina", k=10, prompt=64),
        # a full 60-node tree of a 7B model, plain and with classifier-free guidance (122 rows)
        dict(name="anole_verify_61", kind="verify", model="anole", n=61, prompt=64, guided=False),
        dict(name="anole_guided_verify_61", kind="verify", model="anole", n=61, prompt=64, guided=True),
        # attention of one 7B layer at the end of a 2352-token image, and of sixteen images
        # somewhere in theirs: ragged trees, and the largest trees the framework takes
        dict(name="attn_image_61", kind="attn", B=1, heads=32, dh=128, n=61, lo=2340, hi=2340, cap=2560, ragged=False),
        dict(name="attn_images16_61", kind="attn", B=16, heads=32, dh=128, n=61, lo=512, hi=2400, cap=2560, ragged=True),
        dict(name="attn_images16_128", kind="attn", B=16, heads=32, dh=128, n=128, lo=512, hi=2400, cap=2560,
             ragged=False),
        # the widest and the square projection of sixteen images' 61-row trees
        dict(name="gemm_gate_up_976", kind="gemm", M=976, N=22016, K=4096),
        dict(name="gemm_o_976", kind="gemm", M=976, N=4096, K=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "draft", "prefill", "attn", "attn", "gemm", "gemm", "accept"])
    if kind == "verify":
        model = rng.choice(["tiny", "llamagen", "anole"])
        guided = model != "tiny" and rng.random() < 0.4
        return dict(kind=kind, model=model, n=_log_int(rng, 2, 61), prompt=_log_int(rng, 8, 64 if guided else 120),
                    guided=guided)
    if kind == "draft":
        return dict(kind=kind, model=rng.choice(["llamagen", "anole", "lumina"]), k=rng.randint(4, 13),
                    prompt=_log_int(rng, 8, 120))
    if kind == "prefill":
        return dict(kind=kind, model=rng.choice(["llamagen", "anole"]), prompt=_log_int(rng, 8, 120))
    if kind == "attn":
        heads, dh = rng.choice([(32, 128), (20, 64)])
        B = rng.choice([1, 1, 1, 2, 5, 8, 16])
        lo = _log_int(rng, 60, 2300)
        hi = lo if B == 1 else rng.randint(lo, 2400)
        return dict(kind=kind, B=B, heads=heads, dh=dh, n=_log_int(rng, 2, 128), lo=lo, hi=hi, cap=2560,
                    ragged=rng.random() < 0.5)
    if kind == "gemm":
        N, K = rng.choice(PROJECTIONS[rng.choice(["llamagen", "7b"])])
        return dict(kind=kind, M=_log_int(rng, 40, 976), N=N, K=K)
    return dict(kind="accept", relaxed=rng.random() < 0.5, n=_log_int(rng, 4, 61), vocab=8448, ids=8192,
                top_k=rng.choice([0, 700, 2000]))


# ------------------------------------------------------------------------------ inputs
def _rng(seed, tag):
    return np.random.default_rng([int(seed), tag])


def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000 + tag)
    return g


def _tree(rng, n, max_children=10, max_depth=9):
    """Parents of a random n-node tree in breadth-first order, and its depths."""
    parent, depth, head = [-1], [0], 0
    while len(parent) < n:
        if head >= len(parent):
            head = 0
        if depth[head] < max_depth:
            for _ in range(int(rng.integers(1, max_children + 1))):
                if len(parent) < n:
                    parent.append(head)
                    depth.append(depth[head] + 1)
        head += 1
    order = sorted(range(n), key=lambda i: depth[i])     # stable: the list's order within a depth
    new = {o: i for i, o in enumerate(order)}
    return [-1 if parent[o] < 0 else new[parent[o]] for o in order], [depth[o] for o in order]


def _visible(parent):
    """[n][n]: whether node j is on the path from the root to node i."""
    m = np.zeros((len(parent), len(parent)), dtype=bool)
    for i, p in enumerate(parent):
        if p >= 0:
            m[i] = m[p]
        m[i, i] = True
    return m


class _Config:
    """What a session needs to know of a model and an image."""

    def __init__(self, case, seed):
        d = MODELS[case["model"]]
        self.model = SimpleNamespace(n_layers=d["layers"], d_model=d["d"], n_heads=d["heads"], head_dim=d["dh"],
                                     ffn=d["ffn"], vocab=d["vocab"], dtype=d["dtype"])
        self.prefix_len = case["prompt"]
        self.grid_w = d["grid"]
        self.n_image = d["grid"] * d["grid"]
        self.img = d["img"]
        self.seed = int(seed)
        self.guidance = 3.0 if case.get("guided") else None
        k_hi = 4 if case["model"] == "tiny" else 13
        self.sched = SimpleNamespace(d_lo=1, d_hi=4, k_lo=1, k_hi=k_hi, l_d=1, l_k=1, beta=1.0, n_budget=60, d0=4,
                                     k0=4, init="horizontal", flock_delta=2, fix_d=0, fix_k=0, k_clamp="always", seed=0)
        self.accept = SimpleNamespace(mode="greedy", temperature=1.0, top_k=0, delta=0.0, knn_k=1, children=0)
        rng = _rng(seed, 1)
        self.prompt = rng.integers(0, d["vocab"], size=case["prompt"]).astype(np.int32)
        self.null_prompt = np.full(case["prompt"], d["vocab"] - 1, dtype=np.int32)
        # an image opens with a fixed token, so the tree's root does not hang on an argmax
        self.first = int(rng.integers(0, d["img"]))
        if case["kind"] == "verify":
            self.parent, self.depth = _tree(rng, case["n"])
            self.token = [self.first] + rng.integers(0, d["img"], size=case["n"] - 1).tolist()

    def allowed_table(self):
        t = np.tile(np.array([[0, self.img]], dtype=np.int32), (self.n_image, 1))
        t[0] = (self.first, self.first + 1)
        return t

    def tensor_shapes(self):
        m = self.model
        s = {"embed": (m.vocab, m.d_model), "lm_head": (m.vocab, m.d_model), "draft.fc": (m.d_model, 2 * m.d_model)}
        for pre in [f"layer{l}" for l in range(m.n_layers)] + ["draft"]:
            for w in ("wq", "wk", "wv", "wo"):
                s[f"{pre}.{w}"] = (m.d_model, m.d_model)
            s[pre + ".wg"] = s[pre + ".wu"] = (m.ffn, m.d_model)
            s[pre + ".wd"] = (m.d_model, m.ffn)
        return s


def _weights(cfg):
    """Seeded N(0, 0.02^2) weights on the GPU: every tensor is a window of one drawn pool."""
    shapes = cfg.tensor_shapes()
    size = max(a * b for a, b in shapes.values()) + 4099 * len(shapes)
    dt = torch.float32 if cfg.model.dtype == "f32" else torch.bfloat16
    pool = torch.empty(size, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=_gen(cfg.seed, 2))
    rng = random.Random(cfg.seed)
    out = {}
    for name, (a, b) in shapes.items():
        at = rng.randrange(0, size - a * b)
        out[name] = pool[at: at + a * b].view(a, b)
    return pool, out


def _device_model(cfg):
    pool, w = _weights(cfg)
    host = pool.view(torch.int16).cpu().numpy().view(np.uint16) if pool.dtype == torch.bfloat16 else pool.cpu().numpy()
    base, es = pool.data_ptr(), pool.element_size()
    arrays = {}
    for name, t in w.items():
        at = (t.data_ptr() - base) // es
        arrays[name] = host[at: at + t.numel()].reshape(tuple(t.shape))
    del pool, w
    return rt.DeviceModel(cfg, arrays)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("verify", "draft", "prefill"):
        cfg = _Config(case, seed)
        s = SimpleNamespace(case=case, cfg=cfg, model=_device_model(cfg))
        if kind == "prefill":
            m = cfg.model
            cap = ((cfg.prefix_len + cfg.n_image + 128 + 63) // 64) * 64
            s.caches = tuple(torch.zeros(m.n_layers, m.n_heads, cap, m.head_dim, dtype=torch.bfloat16, device="cuda")
                             for _ in range(2))
            return s
        s.session = rt.DeviceSession(s.model, cfg)
        s.session.prefill(cfg.prompt, cfg.null_prompt if cfg.guidance is not None else None)
        P = cfg.prefix_len
        if kind == "verify":
            s.session.set_tree(cfg.parent, cfg.token)
            t = s.session.tensors()
            n = case["n"]
            s.out = {"logits": t["logits"][:, : cfg.img], "k": s.session.k_cache[..., P: P + n, :],
                     "v": s.session.v_cache[..., P: P + n, :]}
        else:
            s.session.expand(1, case["k"], 60)
            t = s.session.tensors()
            s.out = {"logits": t["draft_logits"][0, : cfg.img], "scores": t["score"][1:]}
        return s
    if kind == "attn":
        B, H, Dh, n, cap = (case[k] for k in ("B", "heads", "dh", "n", "cap"))
        rng, g = _rng(seed, 3), _gen(seed, 4)
        nodes, parent, L = _attn_trees(case, rng)
        rnd = lambda *sh: torch.empty(*sh, dtype=torch.bfloat16, device="cuda").normal_(generator=g)  # noqa: E731
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()  # noqa: E731
        s = SimpleNamespace(case=case, q=rnd(B, n, H, Dh), k=rnd(B, H, cap, Dh), v=rnd(B, H, cap, Dh), kv_len=dev(L),
                            nodes=dev(nodes), out=torch.zeros(B, n, H, Dh, dtype=torch.bfloat16, device="cuda"))
        s.mask, _ = rt.tree_masks(dev(parent), s.nodes)
        need = rt.lib().adt_tree_attn_workspace_size(B, H, Dh, n, cap)
        s.ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
        return s
    if kind == "gemm":
        x, w = _gemm_operands(case, seed)
        need = rt.lib().adt_gemm_bf16_packed_workspace_size(case["M"], case["N"], case["K"])
        return SimpleNamespace(case=case, x=x, w=rt.pack_bf16(w),
                               out=torch.empty(case["M"], case["N"], dtype=torch.float32, device="cuda"),
                               ws=torch.empty(max(need, 256), dtype=torch.uint8, device="cuda"))
    return _accept_inputs(case, seed)


def _attn_trees(case, rng):
    """Node counts, parents and prefix lengths of the B images (odd lengths among them)."""
    B, n = case["B"], case["n"]
    nodes = rng.integers(max(1, n // 8), n + 1, size=B) if case["ragged"] and B > 1 else np.full(B, n)
    nodes[0] = n
    parent = np.full((B, n), -1, dtype=np.int32)
    for b in range(B):
        parent[b, : nodes[b]] = _tree(rng, int(nodes[b]))[0]
    return nodes.astype(np.int32), parent, rng.integers(case["lo"], case["hi"] + 1, size=B).astype(np.int32)


def _gemm_operands(case, seed):
    """Rows as a norm leaves them (unit variance), weights as initialised."""
    g = _gen(seed, 5)
    x = torch.empty(case["M"], case["K"], dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    w = torch.empty(case["N"], case["K"], dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    return x, w


def _accept_inputs(case, seed):
    """Verified logits in which most nodes favour one drafted child, as a trained pair's do."""
    rng, g = _rng(seed, 6), _gen(seed, 7)
    n, V, ids = case["n"], case["vocab"], case["ids"]
    parent, _ = _tree(rng, n, max_children=6)
    kids = [[c for c in range(n) if parent[c] == u] for u in range(n)]
    token = np.zeros(n, dtype=np.int32)
    logits = torch.empty(n, V, dtype=torch.float32, device="cuda").normal_(0.0, 1.5, generator=g)
    for u in range(n):
        if kids[u]:
            token[kids[u]] = rng.choice(ids, size=len(kids[u]), replace=False)
            if rng.random() < 0.85:
                logits[u, int(token[kids[u][0]])] += 9.0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()  # noqa: E731
    knn = None
    if case["relaxed"]:
        knn = torch.randint(0, ids, (ids, 100), generator=g, device="cuda", dtype=torch.int32)
        knn[:, 0] = torch.arange(ids, device="cuda", dtype=torch.int32)
    cfg = rt.accept_cfg("relaxed" if case["relaxed"] else "exact", 1.0, case["top_k"], 0.1 if case["relaxed"] else 0.0,
                        knn, 100 if case["relaxed"] else 1, int(seed))
    ws = torch.empty(rt.lib().adt_accept_workspace_size(V), dtype=torch.uint8, device="cuda")
    return SimpleNamespace(case=case, logits=logits, parent=dev(parent), token=dev(token),
                           allowed=dev(np.tile([0, ids], (n, 1))), n=dev([n]), cfg=cfg, ws=ws)


# ------------------------------------------------------------------------------ one pass
def run(s):
    c = s.case
    kind = c["kind"]
    if kind == "verify":
        s.session.verify()
        return s.out
    if kind == "draft":
        s.session.expand(1, c["k"], 60)
        return s.out
    if kind == "prefill":
        s.session = rt.DeviceSession(s.model, s.cfg, caches=s.caches)
        first = s.session.prefill(s.cfg.prompt)
        P = s.cfg.prefix_len
        return {"first": first, "k": s.caches[0][:, :, :P], "v": s.caches[1][:, :, :P],
                "draft_k": s.session.dk_cache[:, :P], "draft_v": s.session.dv_cache[:, :P]}
    if kind == "attn":
        return rt.tree_attn(s.q, s.k, s.v, s.kv_len, s.nodes, s.nodes, s.mask, c["cap"], out=s.out, workspace=s.ws)
    if kind == "gemm":
        return rt.gemm_bf16_packed(s.x, s.w, c["N"], out=s.out, workspace=s.ws)
    path, n_acc, bonus = rt.verify_accept(s.logits, s.parent, s.token, s.allowed, s.n, s.cfg, 1, workspace=s.ws)
    return {"path": path, "accepted": n_acc, "bonus": bonus}


# ------------------------------------------------------------------------------ what it takes
def work(case):
    kind = case["kind"]
    if kind in ("verify", "draft", "prefill"):
        m = MODELS[case["model"]]
        es = 4 if m["dtype"] == "f32" else 2
        d, layer = m["d"], 4 * m["d"] ** 2 + 3 * m["d"] * m["ffn"]
        P, nb = case["prompt"], 2 if case.get("guided") else 1
        if kind == "verify":
            rows, weights, cols, layers, keys = nb * case["n"], m["layers"] * layer, m["img"], m["layers"], P
        elif kind == "draft":
            rows, weights, cols, layers, keys = 1, layer + 2 * d * d, m["img"], 1, P
        else:
            rows, weights, cols, layers, keys = P, (m["layers"] + 1) * layer + 2 * d * d, 16, m["layers"] + 1, 0
        out_rows = 1 if kind == "prefill" else rows
        attn = layers * 4 * rows * (keys + rows / nb) * d
        return {"bytes": es * (weights + cols * d + nb * layers * 2 * keys * d + rows * d * (1 + 2 * layers))
                + 4 * out_rows * cols,
                "flops": 2 * rows * weights + 2 * out_rows * cols * d + attn}
    if kind == "attn":
        B, H, Dh, n = case["B"], case["heads"], case["dh"], case["n"]
        L = B * (case["lo"] + case["hi"]) / 2
        rows = B * n if not case["ragged"] or B == 1 else n + (B - 1) * (n // 8 + n) / 2
        return {"bytes": 2 * (2 * (L + rows) * H * Dh + 2 * rows * H * Dh) + 16 * rows,
                "flops": 4 * rows * (L / B + n / 2) * H * Dh}
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * K + N * K) + 4 * M * N, "flops": 2 * M * N * K}
    # the rows of the accepted path: about half the depth of a tree of n nodes
    rows = 2
    return {"bytes": rows * 4 * case["ids"], "flops": rows * 20 * case["ids"]}


def tolerance(case):
    """About four times each path's measured distance from exact(): fp32 sums 2e-7 to 7e-7; attention, whose
    probabilities and output are bf16, 2e-3; two to four bf16 layers 4e-3 to 9e-3, the draft head 7e-3 to 15e-3."""
    kind = case["kind"]
    if kind == "accept":
        return "exact"
    if kind == "gemm":
        return {"rel": 3e-6, "max": 1e-4}
    if kind == "attn":
        return {"rel": 8e-3, "max": 0.1}
    if case["model"] == "tiny":
        return {"rel": 2e-6, "max": 1e-4}
    return {"rel": 0.02 if kind == "verify" else 0.03, "max": 0.2}


# ------------------------------------------------------------------------------ in 64 bits
def _norm(x):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-5)


def _rope(x, pos):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * 10000.0 ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _layer(cfg, w, pre, h, pos, see):
    """One decoder layer over all rows at once; see[i][j]: row i attends to row j."""
    m = cfg.model
    f = lambda t: w[f"{pre}.{t}"].double().t()  # noqa: E731
    split = lambda x: x.view(-1, m.n_heads, m.head_dim)  # noqa: E731
    a = _norm(h)
    q, k, v = _rope(split(a @ f("wq")), pos), _rope(split(a @ f("wk")), pos), split(a @ f("wv"))
    s = torch.matmul(q.transpose(0, 1), k.permute(1, 2, 0).contiguous()) / math.sqrt(m.head_dim)
    p = torch.softmax(s.masked_fill(~see, -math.inf), -1)
    o = torch.matmul(p, v.transpose(0, 1).contiguous()).transpose(0, 1).reshape(h.shape[0], -1)
    h = h + o @ f("wo")
    b = _norm(h)
    return h + (torch.nn.functional.silu(b @ f("wg")) * (b @ f("wu"))) @ f("wd"), k.transpose(0, 1), v.transpose(0, 1)


def _target(cfg, w, tok, pos, see):
    h, ks, vs = w["embed"][tok].double(), [], []
    for l in range(cfg.model.n_layers):
        h, k, v = _layer(cfg, w, f"layer{l}", h, pos, see)
        ks.append(k)
        vs.append(v)
    return _norm(h), torch.stack(ks), torch.stack(vs)


def exact(case, seed):
    kind = case["kind"]
    if kind == "accept":
        return None
    if kind == "gemm":
        x, w = _gemm_operands(case, seed)
        return x.double() @ w.double().t()
    if kind == "attn":
        return _exact_attn(case, seed)
    cfg = _Config(case, seed)
    _, w = _weights(cfg)
    P, dev = cfg.prefix_len, "cuda"
    head = w["lm_head"][: cfg.img]
    causal = torch.ones(P + 1, P + 1, dtype=torch.bool, device=dev).tril()
    if kind == "verify":
        n = case["n"]
        see = torch.zeros(P + n, P + n, dtype=torch.bool, device=dev)
        see[:P, :P] = causal[:P, :P]
        see[P:, :P] = True
        see[P:, P:] = torch.from_numpy(_visible(cfg.parent)).to(dev)
        pos = torch.tensor(list(range(P)) + [P + d for d in cfg.depth], device=dev)
        logits, ks, vs = [], [], []
        for prompt in [cfg.prompt] + ([cfg.null_prompt] if cfg.guidance is not None else []):
            f, k, v = _target(cfg, w, torch.tensor(prompt.tolist() + cfg.token, device=dev), pos, see)
            logits.append(f[P:] @ head.double().t())
            ks.append(k[:, :, P:])
            vs.append(v[:, :, P:])
        if cfg.guidance is None:
            return {"logits": logits[0], "k": ks[0], "v": vs[0]}
        return {"logits": logits[1] + cfg.guidance * (logits[0] - logits[1]), "k": torch.stack(ks), "v": torch.stack(vs)}
    # the prompt through the target, then prompt and root through the draft head
    tok = torch.tensor(cfg.prompt.tolist() + [cfg.first], device=dev)
    pos = torch.arange(P + 1, device=dev)
    feat, k, v = _target(cfg, w, tok[:P], pos[:P], causal[:P, :P])
    before = torch.cat([torch.zeros_like(feat[:1]), feat])
    h = torch.cat([w["embed"][tok].double(), before], 1) @ w["draft.fc"].double().t()
    h, dk, dv = _layer(cfg, w, "draft", h, pos, causal)
    if kind == "prefill":
        return {"first": None, "k": k, "v": v, "draft_k": dk[:, :P], "draft_v": dv[:, :P]}
    logits = _norm(h[P:])[0] @ head.double().t()
    return {"logits": logits, "scores": torch.topk(torch.log_softmax(logits, -1), case["k"]).values}


def _exact_attn(case, seed):
    B, H, Dh, n, cap = (case[k] for k in ("B", "heads", "dh", "n", "cap"))
    nodes, parent, L = _attn_trees(case, _rng(seed, 3))
    g = _gen(seed, 4)
    q, k, v = (torch.empty(*sh, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
               for sh in ((B, n, H, Dh), (B, H, cap, Dh), (B, H, cap, Dh)))
    out = torch.zeros(B, n, H, Dh, dtype=torch.float64, device="cuda")
    for b in range(B):
        m, l = int(nodes[b]), int(L[b])
        see = torch.ones(m, l + m, dtype=torch.bool, device="cuda")
        see[:, l:] = torch.from_numpy(_visible(parent[b, :m].tolist())).cuda()
        s = torch.matmul(q[b, :m].double().transpose(0, 1).contiguous(), k[b, :, : l + m].double().transpose(1, 2).contiguous())
        p = torch.softmax((s / math.sqrt(Dh)).masked_fill(~see, -math.inf), -1)
        out[b, :m] = torch.matmul(p, v[b, :, : l + m].double().contiguous()).transpose(0, 1)
    return out
