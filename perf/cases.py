"""Workloads on which the speculative verify-and-commit path is measured.

A case is one context (model shape, depth, vocabulary, draft, sequences) and one
pass through the public calls on it:

  verify   one verify of [pending, d_1..d_K] of every sequence and its commit
           (K = 0: one step of plain greedy decoding)
  round    a whole speculative round: the draft's K proposals, the verify of
           given drafts and the commit
  open     a scene from its prompt K/V: opening the context on weights and
           workspace that the program keeps, then its first round

Depths are cut to a few layers, which repeat in a full model: rounding in one
layer travels through all that follow, so that at full depth two correct bf16
implementations agree no better than the format does.  Widths, vocabularies,
row counts and prompt lengths are those of the repository's workloads.

The embedding (and so the tied LM head) is drawn wider than the other weights:
a row's own token then clearly wins its argmax, as a trained model's prediction
does, and the committed tokens are not a matter of rounding.
"""
import math

import torch

import workloads as W
from paper_2606_31160_amd import binding as B
from paper_2606_31160_amd.harness import Session

SHAPES = {
    # 7B-class backbone and its shard under 4-way tensor parallelism
    "7b": (W.ModelShape(1, 3584, 28, 4, 128, 18944, (16, 24, 24)), 152064, 64.0),
    "tp4": (W.ModelShape(1, 3584, 7, 1, 128, 4736, (16, 24, 24)), 38016, 64.0),
    # the paper's own backbone: interleaved axis assignment, blocks of K = 16
    "paper": (W.ModelShape(1, 4096, 32, 8, 128, 12288, (24, 20, 20), True), 151936, 64.0),
    "tiny": (W.ModelShape(1, 256, 4, 2, 64, 688, (8, 12, 12)), 1024, 4.0),
}


def _case(name, do, shape, layers, K, prompts, vocab=0, draft="none", draft_layers=2, rowmajor=False, accept=0):
    """prompts: the sequences' prompt lengths, space-separated; vocab 0: the shape's own; accept: leading proposals
    of every second sequence that the target accepts."""
    c = {"do": do, "shape": shape, "layers": layers, "K": K, "prompts": prompts, "vocab": vocab, "draft": draft,
         "draft_layers": draft_layers if draft != "none" else 0, "rowmajor": rowmajor, "accept": accept}
    return dict(c, name=name) if name else c


# sixteen driving scenes of 2048 to 8192 tokens (workload C5's own draw)
SCENES_16 = " ".join(str(s.prefix_len) for s in W.get("C5").seqs)


def listed():
    return [
        # the smallest call in use: launches and latency are all of it
        _case("tiny round", "round", "tiny", 2, 4, "320", draft="chain", draft_layers=1),
        # one decoder layer of the 7B target, 9 rows, under a small head: the layer kernels by themselves
        _case("7b layer verify", "verify", "7b", 1, 8, "3328", vocab=1024),
        # the headline verify: 9 rows through target layers and the full head, half of the rows' first proposal right
        _case("7b verify", "verify", "7b", 4, 8, "4096", accept=1),
        # plain greedy decoding of one scene: one row
        _case("7b greedy step", "verify", "7b", 4, 0, "2753"),
        # a speculative round as an application runs it: 8 chained draft steps, then the verify
        _case("7b round", "round", "7b", 2, 8, "4096", draft="chain", accept=1),
        # the same round with the proposals made in one forward (block-diffusion draft)
        _case("7b block round", "round", "7b", 2, 8, "4096", draft="block"),
        # the paper's backbone at its verification width: 17 rows
        _case("paper verify", "verify", "paper", 4, 16, "4096"),
        # a few ragged scenes together: 45 rows
        _case("5 scenes verify", "verify", "7b", 4, 8, "517 1290 2311 3071 4444", accept=1),
        # sixteen scenes together: 144 rows
        _case("16 scenes verify", "verify", "7b", 4, 8, SCENES_16),
        # ... and their whole round, the largest call
        _case("16 scenes round", "round", "7b", 4, 8, SCENES_16, draft="chain", accept=1),
        # without the second, tile-packed copy of the weights
        _case("row-major verify", "verify", "7b", 4, 8, "4096", rowmajor=True),
        # a new scene on weights that stay: opening the context and its first round
        _case("open scene", "open", "7b", 4, 8, "4096", draft="chain"),
    ]


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        shape = rng.choice(["tiny", "7b", "7b", "tp4", "paper"])
        do = rng.choice(["verify", "verify", "round", "round", "open"])
        K = rng.choice([0, 1, 2, 3, 4, 5, 7, 8, 8, 11, 16]) if do == "verify" else rng.choice([2, 4, 5, 8, 8, 16])
        batch = min(16, 160 // (K + 1), rng.choice([1, 1, 1, 2, 3, 4, 6, 9, 12, 16]))
        if do == "open":
            batch = min(batch, 2)
        prompts = " ".join(str(int(round(2.0 ** rng.uniform(6, 13)))) for _ in range(batch))
        vocab = 0 if rng.random() < 0.7 else 32 * rng.randint(32, 1000)
        draft = "none" if do == "verify" else rng.choice(["chain", "chain", "block", "cond"])
        rowmajor = rng.random() < 0.15 and batch * (K + 1) <= 64
        c = _case("", do, shape, rng.randint(1, 4), K, prompts, vocab, draft, rng.randint(1, 2), rowmajor,
                  rng.randint(0, 1) if K else 0)
        if draft == "cond" and batch * (K + 1) > 24:
            continue   # the feature fusion holds this many rows at every shape here
        if work(c)["bytes"] <= most:
            return c


def _prompts(case):
    return [int(p) for p in case["prompts"].split()]


def _workload(case, seed):
    shape, vocab, _ = SHAPES[case["shape"]]
    # prompts with room for four camera grids are vision-dominated, shorter ones text
    seqs = tuple(W.c5_layout(p) if p >= 256 else W.SeqLayout(p) for p in _prompts(case))
    target = W.ModelShape(**{**shape.__dict__, "layers": case["layers"]})
    draft = (W.ModelShape(**{**shape.__dict__, "layers": case["draft_layers"], "interleaved": False})
             if case["draft"] != "none" else None)
    return W.Workload("case", target, draft, vocab=case["vocab"] or vocab, K=case["K"], seqs=seqs,
                      p_accept=(0.75,) * len(seqs), max_new_tokens=_budget(case), seed=int(seed))


def _budget(case):
    """Tokens a context is opened for: a scene's own few where each pass opens one, else enough for a long run of
    passes (a program that goes on past it opens the next scene)."""
    if case["do"] == "open":
        return 20
    return 6144 if case["shape"] == "tiny" or case["layers"] == 1 else 2048


class _Weights(W.DeviceWeights):
    """Seeded device weights with the embedding scaled by a power of two."""

    def __init__(self, w, scale):
        super().__init__(w)
        self.scale = scale

    def tensor(self, model, layer, name):
        t = super().tensor(model, layer, name)
        if name == "embed" and not getattr(t, "_scaled", False):
            t.mul_(self.scale)
            t._scaled = True
        return t


class _Scene(Session):
    """A session that keeps its prompt K/V, so that its context can be opened again."""

    def __init__(self, *a, **kw):
        self.prompt_kv = []
        super().__init__(*a, **kw)

    def _prefix(self, *a):
        t = super()._prefix(*a)
        self.prompt_kv.append(t)
        return t

    def reopen(self):
        self.close()
        self.ctx = B.spec_init(self.cfg, self.embed.data_ptr(), self.tgt_struct,
                               self.drf_struct if self.has_draft else None, self.seqs, self.ws.data_ptr(),
                               self.ws_bytes, self.stream.cuda_stream)


def _drafts(case, w):
    """Given proposals: uniform tokens, the first `accept` of every second sequence being the token the target
    repeats."""
    g = torch.Generator().manual_seed(w.seed + 17)
    d = torch.randint(0, w.vocab, (w.batch, max(1, w.K)), generator=g, dtype=torch.int32)
    for b in range(w.batch):
        pending = W.first_pending_token(w, b)
        d[b][d[b] == pending] = (pending + 1) % w.vocab
        if b % 2 == 0:
            d[b, :case["accept"]] = pending
    return d


def prepare(case, seed):
    w = _workload(case, seed)
    flags = (B.SPEC_FLAG_ROWMAJOR if case["rowmajor"] else 0) | (B.SPEC_FLAG_BLOCK_DRAFT if case["draft"] == "block" else 0)
    cond = (0, case["layers"] // 2, case["layers"] - 1) if case["draft"] == "cond" else None
    s = _Scene(w, source="device", provider=_Weights(w, SHAPES[case["shape"]][2]), flags=flags, cond_layers=cond,
               page_seed=5 if w.batch > 1 else None)
    return {"do": case["do"], "scene": s, "drafts": _drafts(case, w).to("cuda"), "left": w.max_new_tokens,
            "most": case["accept"] + 1}


def run(state):
    s = state["scene"]
    if state["do"] == "open":
        s.reopen()
    else:
        if state["left"] <= state["most"]:
            s.reopen()
            state["left"] = s.w.max_new_tokens
        state["left"] -= state["most"]
    if s.has_draft:
        B.draft_steps(s.ctx, s.K, s.dtok.data_ptr())
    B.spec_verify(s.ctx, state["drafts"].data_ptr() if s.K else 0, s.logits.data_ptr())
    B.spec_commit(s.ctx, s.acc.data_ptr(), s.com.data_ptr(), s.ncom.data_ptr(), s.fin.data_ptr())
    return {"logits": s.logits, "accepted": s.acc, "committed": s.com, "count": s.ncom, "finished": s.fin,
            "proposed": s.dtok if s.has_draft else None}


def _layer_params(s):
    return s.hidden * (s.q_heads + 2 * s.kv_heads) * s.head_dim + s.q_heads * s.head_dim * s.hidden + 3 * s.hidden * s.ffn


def work(case):
    """Weights once per pass over them (each chained draft step is one), every prompt's K/V once per pass over it, new
    K/V rows and logits written."""
    s, vocab, _ = SHAPES[case["shape"]]
    V = case["vocab"] or vocab
    prompts, K = _prompts(case), case["K"]
    batch, R = len(prompts), case["K"] + 1
    row = s.kv_heads * s.head_dim * 2 * 2   # bytes of one slot's K and V in one layer
    P, head = _layer_params(s), s.hidden * V

    def stack(layers, rows, head_rows):   # one pass over every sequence
        attn = 4 * s.q_heads * s.head_dim * sum(prompts) * rows
        return (layers * (2 * P + (sum(prompts) + batch * rows) * row) + 2 * head,
                layers * (2 * P * batch * rows + attn) + 2 * head * batch * head_rows)

    nbytes, flops = stack(case["layers"], R, R)
    nbytes += 2 * batch * R * V
    L = case["draft_layers"]
    if case["draft"] in ("chain", "cond"):
        b, f = stack(L, 1, 1)
        nbytes, flops = nbytes + K * b, flops + K * f
        if case["draft"] == "cond":
            nbytes, flops = nbytes + 2 * (3 + 2 * K) * s.hidden ** 2, flops + 2 * (3 * R + 2 * K) * batch * s.hidden ** 2
    elif case["draft"] == "block":
        b, f = stack(L, R, K)
        nbytes, flops = nbytes + b, flops + f
    if case["do"] == "open":   # every prompt slot read once and written once to the caches
        nbytes += 2 * (case["layers"] + L) * sum(prompts) * row
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # The tile-packed and the row-major path form the same sums in other orders.  Their logits differ by 1.2e-3 (2-norm;
    # 8e-3 at most) after one layer, 3.0e-3 (1.4e-2) after two and 4.4e-3 to 5.1e-3 (2.6e-2) after four; four times that.
    return {"rel": 0.005 * case["layers"], "max": 0.03 * case["layers"]}


def _rope(x, pos3, s):
    """Rotates adjacent pairs of x [N, heads, D] at positions pos3 [3, N]."""
    half = s.head_dim // 2
    d = torch.arange(half, device=x.device)
    sec = s.mrope_section
    axis = d % 3 if s.interleaved else (d >= sec[0]).long() + (d >= sec[0] + sec[1]).long()
    theta = s.rope_base ** (-2.0 * d.double() / s.head_dim)
    ang = pos3[axis].double().T * theta             # [N, half]
    c, n = ang.cos()[:, None], ang.sin()[:, None]
    e, o = x[..., 0::2], x[..., 1::2]
    return torch.stack([e * c - o * n, e * n + o * c], dim=-1).flatten(-2)


def exact(case, seed):
    w = _workload(case, seed)
    src, s, V = _Weights(w, SHAPES[case["shape"]][2]), w.target, w.vocab
    get = lambda model, li, name: src.tensor(model, li, name).double()
    dr = _drafts(case, w)
    E = src.tensor("global", -1, "embed")
    R, D, nq, nkv = w.K + 1, s.head_dim, s.q_heads, s.kv_heads
    toks = torch.tensor([[W.first_pending_token(w, b)] + dr[b, :w.K].tolist() for b in range(w.batch)])
    x = E[toks.flatten().to(E.device)].double()      # [B R, H]
    inv = lambda v: 1.0 / torch.sqrt((v * v).mean(-1, keepdim=True) + s.rms_eps)
    for li in range(s.layers):
        h = x * inv(x) * get("target", li, "attn_norm")
        q, k, v = (h @ get("target", li, n).T for n in ("wq", "wk", "wv"))
        out = torch.empty_like(q)
        for b, lay in enumerate(w.seqs):
            P = lay.prefix_len
            pos = torch.arange(P + R).repeat(3, 1)
            for g in lay.blocks:
                i = torch.arange(g.ntok)
                pos[:, g.start:g.start + g.ntok] = g.start + torch.stack([i // (g.h * g.w), i // g.w % g.h, i % g.w])
            pos = pos.to(x.device)
            rows = slice(b * R, (b + 1) * R)
            kp, vp = (W.prefix_kv_device(w, b, "target", li, c).double() for c in "kv")
            kk = _rope(torch.cat([kp, k[rows].view(R, nkv, D)]), pos, s)
            vv = torch.cat([vp, v[rows].view(R, nkv, D)])
            qq = _rope(q[rows].view(R, nq, D), pos[:, P:], s).view(R, nkv, nq // nkv, D)
            mask = torch.arange(P + R, device=x.device)[None] > P + torch.arange(R, device=x.device)[:, None]
            for n in range(nkv):
                sc = (qq[:, n].reshape(-1, D) @ kk[:, n].T).view(R, -1, P + R) / math.sqrt(D)
                pr = sc.masked_fill(mask[:, None], -math.inf).softmax(-1).view(-1, P + R)
                out[rows].view(R, nkv, -1, D)[:, n] = (pr @ vv[:, n]).view(R, -1, D)
        x = x + out @ get("target", li, "wo").T
        h = x * inv(x) * get("target", li, "ffn_norm")
        gate, up = (h @ get("target", li, n).T for n in ("w_gate", "w_up"))
        x = x + (torch.nn.functional.silu(gate) * up) @ get("target", li, "w_down").T
    h = x * inv(x) * get("target", -1, "final_norm")
    z = torch.cat([h @ E[i:i + 16384].double().T for i in range(0, V, 16384)], dim=1)
    return {"logits": z.view(w.batch, R, V), "accepted": None, "committed": None, "count": None, "finished": None,
            "proposed": None}
