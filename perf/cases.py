"""What the speed of this framework is measured on: calls of its public entry points (`SwiftModel`) as a decoding
program makes them, at the model shapes of `synthetic_inputs.py`.

A case is one call (or the short sequence of calls that one decoding step is) on a context whose cache holds the
tokens before it.  Models of the full 7B depth stand for whole passes; the others are a few layers of the named
width, so that a call is dominated by single attention and MLP sublayers of that size.

Weights are drawn, not trained: matrices N(0, 0.02^2), gains around 1, the sublayers' output projections scaled so
that all branches together weigh about as much in the residual stream as the token's embedding, and an LM head that
carries a share of the embedding of each token's successor.  Logits then look like a trained model's -- one token
clearly ahead, confidences well inside (0, 1), a layer-skipping draft that mostly agrees -- and no arg-max hangs on
the last bits of a sum.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2410_06916_amd as P
import synthetic_inputs as si

TEMPERATURE, TOP_P = 0.6, 0.95  # the sampled runs of the paper
SHAPES = {"tiny": si.TINY, "7b": si.LLAMA2_7B, "13b": si.LLAMA2_13B, "70b": si.LLAMA2_70B}


# ------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------
# kind      the call                                                         sizes
# step      draft_step(k) and verify of the k + 1 rows                       k, ctx
# decode    verify of the pending token alone: plain decoding                ctx
# draft     draft_step(k) under a skip mask                                  k, ctx
# verify    verify of a chain block                                          rows, ctx
# tree      verify_tree: three levels of candidates                          rows, ctx
# prefill   prefill of a prompt                                              n
# eval      eval_mask: a candidate draft model over the last gamma tokens    gamma, ctx
# sample    draft_step_sample(k) and verify_sample                           k, ctx
# ctx: tokens in the cache before the call; cap: cache capacity; skip: skipped sublayers of the mask.
def listed():
    return [
        # the smallest model (fp32): a decoding step and a prompt are nothing but launches and latency
        dict(name="tiny-step", kind="step", model="tiny", layers=4, ctx=48, cap=101, k=4, skip=2),
        dict(name="tiny-prefill", kind="prefill", model="tiny", layers=4, n=32, cap=101),
        # the headline workload (7B, prompt 512, 256 new tokens): plain decoding, drafting, chain verification,
        # dynamic verification, candidate evaluation, prompt
        dict(name="7b-decode", kind="decode", model="7b", layers=32, ctx=640, cap=777),
        dict(name="7b-draft", kind="draft", model="7b", layers=32, ctx=600, cap=777, k=8, skip=32),
        dict(name="7b-verify", kind="verify", model="7b", layers=32, ctx=611, cap=777, rows=9),
        dict(name="7b-tree", kind="tree", model="7b", layers=32, ctx=611, cap=777, rows=31),
        dict(name="7b-eval", kind="eval", model="7b", layers=32, ctx=700, cap=777, gamma=32, skip=32),
        dict(name="7b-prefill", kind="prefill", model="7b", layers=32, n=512, cap=777),
        # long contexts: a verification over 8 000 tokens, a long prompt that is not a multiple of any block
        dict(name="7b-long-verify", kind="verify", model="7b", layers=8, ctx=8150, cap=8329, rows=9),
        dict(name="7b-long-prefill", kind="prefill", model="7b", layers=4, n=3990, cap=8329),
        # a short ragged prompt at the 13B width
        dict(name="13b-prefill", kind="prefill", model="13b", layers=8, n=205, cap=1293),
        # speculative sampling at the grouped-query 70B width
        dict(name="70b-sample", kind="sample", model="70b", layers=4, ctx=2048, cap=2185, k=4, skip=3),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "decode", "draft", "verify", "tree", "prefill", "prefill", "eval", "sample"])
    model = rng.choice(["tiny", "7b", "7b", "13b", "70b"])
    layers = rng.randint(2, 4) if model == "tiny" else rng.randint(2, 5)
    c = dict(kind=kind, model=model, layers=layers)
    if kind == "prefill":
        c["n"] = _log_int(rng, 1, 200) if model == "tiny" else _log_int(rng, 1, 1000 if model == "70b" else 3000)
        c["cap"] = c["n"] + rng.randint(2, 1500)
        return c
    c["ctx"] = _log_int(rng, 8, 300) if model == "tiny" else _log_int(rng, 16, 8000)
    c["cap"] = c["ctx"] + rng.randint(40, 1500)
    if kind in ("step", "draft", "sample"):
        c["k"] = rng.randint(1, 8)
    if kind == "verify":
        c["rows"] = rng.randint(2, 32)
    if kind == "tree":
        c["rows"] = rng.randint(4, 31)
    if kind == "eval":
        c["gamma"] = min(c["ctx"], _log_int(rng, 1, 128))
    if kind in ("step", "draft", "sample", "eval"):
        c["skip"] = rng.randint(0, layers)
    return c


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _shape(case):
    return SHAPES[case["model"]].with_layers(case["layers"])


def _seed(seed, what):
    return (int(seed) * 1000003 + what * 7919 + 12345) % (1 << 62)


def _weights(shape, seed):
    """(name, tensor) on the GPU, one after the other."""
    gen = torch.Generator(device="cuda")
    dt = torch.float32 if shape.dtype == "fp32" else torch.bfloat16
    H = shape.hidden
    branch = 0.75 / math.sqrt(2 * shape.n_layers)
    embed = None
    for i, (name, dims, kind) in enumerate(si.tensor_specs(shape)):
        gen.manual_seed(_seed(seed, i))
        if kind == "gain":
            yield name, torch.empty(dims, dtype=torch.float32, device="cuda").normal_(1.0, 0.1, generator=gen)
            continue
        std = 1.0 if name == "embed" else 0.02 * branch if name.endswith((".wo", ".wd")) else 0.02
        w = torch.empty(dims, dtype=dt, device="cuda").normal_(0.0, std, generator=gen)
        if name == "embed":
            embed = w
        elif name == "lm_head":
            V = shape.vocab
            nxt = (torch.arange(V, device="cuda") * 7919 + int(seed) % V) % V  # the successor of each token
            w[nxt] += embed * (16.0 / H)
        yield name, w


def _ids(shape, seed, what, n):
    return si.uniform_ids(_seed(seed, 1000 + what), n, shape.vocab)


def _mask(case):
    """The skipped sublayers: drawn among all but the outer layers where there are enough, else among all."""
    L, skip = case["layers"], case.get("skip", 0)
    return si.random_mask(L, skip, 2) if skip <= 2 * (L - 4) else si.random_mask(L, skip, 2, 0, L - 1)


def _levels(case):
    """Widths of a tree of `rows` rows: the pending token and up to three levels of at most ten candidates."""
    left, n = case["rows"] - 1, 3
    return [left // n + (1 if i < left % n else 0) for i in range(n)]


def _calls(case, seed):
    """Everything a call is given besides the weights."""
    shape = _shape(case)
    n = case.get("n", case.get("ctx"))
    u = np.random.default_rng(_seed(seed, 3000)).random(64).astype(np.float32)
    return dict(prompt=_ids(shape, seed, 0, n), more=_ids(shape, seed, 1, 64), mask=_mask(case), u=u)


class State:
    def __init__(self, case, seed):
        self.case, self.shape = case, _shape(case)
        self.__dict__.update(_calls(case, seed))
        self.g = P.SwiftModel(self.shape, case["cap"])
        self.g.load_weights(_weights(self.shape, seed))
        if case["kind"] != "prefill":
            self.g.prefill(self.prompt)  # the tokens before the call
            self.n, self.pending = self.g.cache_len, self.g.pending

    def __del__(self):
        self.g.close()


def _padded(tokens, n):
    """A step emits as many tokens as it accepts: -1 past them."""
    return np.append(tokens, np.full(n - len(tokens), -1)).astype(np.int32)


def prepare(case, seed):
    return State(case, seed)


def run(s):
    c, g, kind = s.case, s.g, s.case["kind"]
    if kind == "prefill":
        tok = g.prefill(s.prompt)
        return dict(token=tok, logits=g.read_logits((c["n"] - 1) % (64 if s.shape.dtype == "bf16" else 32)))
    if kind == "decode":
        tgt, lg = g.verify([s.pending], True)
        return dict(targets=tgt, logits=lg)
    if kind == "draft":
        tok, conf = g.draft_step(s.mask, c["k"], 0.0)
        return dict(tokens=tok, conf=conf, logits=g.read_logits(0))
    if kind == "step":
        tok, conf = g.draft_step(s.mask, c["k"], 0.0)
        tgt, lg = g.verify(np.concatenate([[s.pending], tok]), True)
        return dict(tokens=tok, conf=conf, targets=tgt, logits=lg)
    if kind == "verify":
        tgt, lg = g.verify(np.concatenate([[s.pending], s.more[:c["rows"] - 1]]), True)
        return dict(targets=tgt, logits=lg)
    if kind == "tree":
        at, levels = 0, []
        for w in _levels(c):
            levels.append(s.more[at:at + w])
            at += w
        tgt, lg = g.verify_tree(levels, True)
        return dict(targets=tgt, logits=lg)
    if kind == "eval":
        gamma = c["gamma"]
        pred, match = g.eval_mask(s.mask, np.concatenate([s.prompt[-gamma:], [s.pending]]))
        return dict(predicted=pred, match=match, logits=g.read_logits((gamma - 1) % 64))
    assert kind == "sample"
    k = c["k"]
    tok, conf = g.draft_step_sample(s.mask, k, 0.0, TEMPERATURE, TOP_P, s.u[:k])
    out, probs = g.verify_sample(np.concatenate([[s.pending], tok]), TEMPERATURE, TOP_P, s.u[16:16 + k], float(s.u[40]), True)
    g.rollback(s.n, s.pending)  # the next pass decodes the same position
    return dict(tokens=tok, conf=conf, emitted=_padded(out, k + 1), probs=probs)


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def _pass(shape, mask, ctx, rows, logit_rows, write=True):
    """(bytes, flops) of one pass of `rows` rows over ctx cached tokens: the weights of the sublayers that run and the
    LM head once, keys and values once, logits out."""
    eb = shape.elem_bytes()
    kv = 2 * shape.kv_dim * eb
    by = logit_rows and (shape.vocab * shape.hidden * eb + logit_rows * shape.vocab * 4)
    fl = 2.0 * logit_rows * shape.vocab * shape.hidden
    by += rows * shape.hidden * eb
    for l in range(shape.n_layers):
        if mask is None or not mask[2 * l]:
            q_only = 0 if write else 2 * shape.kv_dim * shape.hidden
            by += (shape.attn_sublayer_elems() - q_only) * eb + kv * (ctx + (rows if write else 0))
            fl += 2.0 * rows * (shape.attn_sublayer_elems() - q_only) + 4.0 * shape.q_dim * rows * (ctx + (rows + 1) / 2)
        if mask is None or not mask[2 * l + 1]:
            by += shape.mlp_sublayer_elems() * eb
            fl += 2.0 * rows * shape.mlp_sublayer_elems()
    return np.array([by, fl], np.float64)


def work(case):
    shape, kind = _shape(case), case["kind"]
    mask, ctx = _mask(case), case.get("ctx", 0)
    drafts = lambda: sum(_pass(shape, mask, ctx + j, 1, 1) for j in range(case["k"]))  # noqa: E731
    if kind == "prefill":
        w = _pass(shape, None, 0, case["n"], 1)
    elif kind == "decode":
        w = _pass(shape, None, ctx, 1, 1)
    elif kind == "draft":
        w = drafts()
    elif kind in ("step", "sample"):
        w = drafts() + _pass(shape, None, ctx, case["k"] + 1, case["k"] + 1)
    elif kind == "eval":
        w = _pass(shape, mask, ctx - case["gamma"], case["gamma"], case["gamma"], write=False)
    else:
        w = _pass(shape, None, ctx, case["rows"], case["rows"])
    return {"bytes": float(w[0]), "flops": float(w[1])}


def tolerance(case):
    # fp32 models: sums in another order.  bf16 models: every accumulation is fp32, but keys and values are rounded to
    # bf16 where they enter the cache, and a sum in another order moves some of them by one rounding step.  About four
    # times the distance from 64-bit sums: 1.2e-7 for the fp32 model; for the others up to 9e-4 in logits, 1.2e-3 in
    # confidences (exponentials of logits) and 2.3e-3 in the sampled runs' probabilities (exponentials at 1 / 0.6).
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if case["kind"] == "sample":
        return {"rel": 1e-2, "max": 0.05, "differ": 0.0}
    if case["kind"] in ("draft", "step"):
        return {"rel": 5e-3, "max": 0.02, "differ": 0.0}
    return {"rel": 3e-3, "max": 0.02, "differ": 0.0}


# ------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------
class _Exact:
    """The model in float64; keys and values are rounded to the cache's storage type, as the cache holds them."""

    def __init__(self, case, seed):
        self.shape = s = _shape(case)
        self.w = dict(_weights(s, seed))
        self.__dict__.update(_calls(case, seed))
        self.k = [torch.zeros(s.n_kv_heads, case["cap"], s.head_dim, dtype=torch.float64, device="cuda") for _ in range(s.n_layers)]
        self.v = [torch.zeros_like(x) for x in self.k]

    def mat(self, name, x):
        w = self.w[name]
        return torch.cat([x @ part.double().t() for part in w.split(8192)], 1)

    def norm(self, x, gain):
        return x / torch.sqrt((x * x).mean(1, keepdim=True) + self.shape.rms_eps) * self.w[gain].double()

    def stored(self, x):
        return x.float().to(torch.float32 if self.shape.dtype == "fp32" else torch.bfloat16).double()

    def rotate(self, x, pos):
        d = self.shape.head_dim
        ang = pos.double()[:, None] * self.shape.rope_theta ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d)
        c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
        a, b = x[..., : d // 2], x[..., d // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    def forward(self, tokens, pos, sees, slots, mask=None, logit_rows=None):
        """Rows `tokens` at positions `pos`; their keys and values go to `slots` (None: nowhere); row i attends the slots
        that sees[i] marks.  Logits of logit_rows (default: all)."""
        s = self.shape
        pos = torch.as_tensor(np.asarray(pos), device="cuda")
        R, d, nq, nkv = len(tokens), s.head_dim, s.n_q_heads, s.n_kv_heads
        S = sees.shape[1]
        x = self.w["embed"][torch.as_tensor(np.asarray(tokens, np.int64), device="cuda")].double()
        for l in range(s.n_layers):
            if mask is None or not mask[2 * l]:
                h = self.norm(x, f"l{l}.attn_norm")
                q = self.rotate(self.mat(f"l{l}.wq", h).view(R, nq, d), pos)
                if slots is not None:
                    self.k[l][:, slots] = self.stored(self.rotate(self.mat(f"l{l}.wk", h).view(R, nkv, d), pos)).transpose(0, 1)
                    self.v[l][:, slots] = self.stored(self.mat(f"l{l}.wv", h).view(R, nkv, d)).transpose(0, 1)
                y = torch.empty(R, nq, d, dtype=torch.float64, device="cuda")
                for hq in range(nq):
                    g = hq // (nq // nkv)
                    sc = (q[:, hq] @ self.k[l][g, :S].t()) / math.sqrt(d)
                    y[:, hq] = torch.softmax(sc.masked_fill_(~sees, -math.inf), 1) @ self.v[l][g, :S]
                x = x + self.mat(f"l{l}.wo", y.view(R, nq * d))
            if mask is None or not mask[2 * l + 1]:
                h = self.norm(x, f"l{l}.mlp_norm")
                gate = self.mat(f"l{l}.wg", h)
                x = x + self.mat(f"l{l}.wd", gate * torch.sigmoid(gate) * self.mat(f"l{l}.wu", h))
        x = x if logit_rows is None else x[logit_rows]
        return self.mat("lm_head", self.norm(x, "final_norm"))

    def chain(self, tokens, pos0, mask=None, logit_rows=None, write=True):
        n = len(tokens)
        at = torch.arange(pos0, pos0 + n, device="cuda")
        sees = torch.arange(pos0 + n, device="cuda")[None] <= at[:, None]
        return self.forward(tokens, np.arange(pos0, pos0 + n), sees, at if write else None, mask, logit_rows)

    def warped(self, logits):
        p = torch.softmax(logits / TEMPERATURE, 1)
        srt = p.sort(1, descending=True).values
        t = srt.gather(1, (srt.cumsum(1) < TOP_P).sum(1, keepdim=True).clamp(max=p.shape[1] - 1))
        p = torch.where(p >= t, p, torch.zeros_like(p))
        return p / p.sum(1, keepdim=True)

    @staticmethod
    def drawn(p, u):
        c = p.cumsum(0)
        return int((c > float(u) * c[-1]).nonzero()[0])


def _host(t, dtype=np.float64):
    return t.cpu().numpy().astype(dtype)


@torch.no_grad()
def exact(case, seed):
    kind, e = case["kind"], _Exact(case, seed)
    n = len(e.prompt)
    last = e.chain(e.prompt, 0, logit_rows=[n - 1])
    pending = int(last[0].argmax())
    if kind == "prefill":
        return dict(token=pending, logits=_host(last[0]))
    if kind in ("decode", "verify"):
        lg = e.chain([pending] + list(e.more[:case.get("rows", 1) - 1]), n)
        return dict(targets=_host(lg.argmax(1), np.int32), logits=_host(lg))
    if kind == "eval":
        gamma = case["gamma"]
        lg = e.chain(list(e.prompt[-gamma:]), n - gamma, e.mask, write=False)
        pred = _host(lg.argmax(1), np.int32)
        want = np.append(e.prompt[-gamma:][1:], pending)
        return dict(predicted=pred, match=int((pred == want).sum()), logits=_host(lg[-1]))
    if kind == "tree":
        rows, depth, path = case["rows"], [0], []
        for j, w in enumerate(_levels(case)):
            path.append(len(depth))
            depth += [j + 1] * w
        sees = torch.zeros(rows, n + rows, dtype=torch.bool, device="cuda")
        sees[:, :n + 1] = True
        for r in range(rows):
            for j in range(depth[r] - 1):
                sees[r, n + path[j]] = True
            sees[r, n + r] = True
        lg = e.forward([pending] + list(e.more[:rows - 1]), n + np.array(depth), sees, torch.arange(n, n + rows, device="cuda"))
        return dict(targets=_host(lg.argmax(1), np.int32), logits=_host(lg))
    toks, conf, q = [pending], [], []
    for j in range(case["k"]):
        lg = e.chain([toks[-1]], n + j, e.mask)
        conf.append(float(torch.softmax(lg[0], 0).max()))
        q.append(e.warped(lg)[0] if kind == "sample" else None)
        toks.append(e.drawn(q[-1], e.u[j]) if kind == "sample" else int(lg[0].argmax()))
    drafted, conf = np.array(toks[1:], np.int32), np.array(conf)
    if kind == "draft":
        return dict(tokens=drafted, conf=conf, logits=_host(lg[0]))
    lg = e.chain(toks, n)
    if kind == "step":
        return dict(tokens=drafted, conf=conf, targets=_host(lg.argmax(1), np.int32), logits=_host(lg))
    p, out = e.warped(lg), []
    for i, t in enumerate(drafted):
        if not float(e.u[16 + i]) * float(q[i][t]) < float(p[i][t]):
            rest = (p[i] - q[i]).clamp(min=0)
            out.append(e.drawn(rest if float(rest.sum()) > 0 else p[i], e.u[40]))
            break
        out.append(int(t))
    else:
        out.append(e.drawn(p[-1], e.u[40]))
    return dict(tokens=drafted, conf=conf, emitted=_padded(out, case["k"] + 1), probs=_host(p))
