"""What a user of this framework has it do, as measurable cases.

Five kinds of work, each through the public entry points:
  verify    one round of the speculative loop: ad_verify_step over a drafted block (a chain,
            or a draft tree), the commit, and, for a model with linear draft heads, the
            next draft block (ad_draft_heads)
  draft     one audio-conditioned draft step: ad_draft_input and the one-layer draft block
  prefill   the encoder K/V of a batch of utterances (ad_cross_kv_prefill)
  loss      the AnchorDraft objective with its three gradients (ad_anchordraft_loss)
  kv        a committed prefix restored and saved again (ad_kv_import, ad_kv_export)

Weights, encoder states and committed prefixes follow the distributions of the package's
seeded inputs (N(0, 0.02) weights, unit-variance encoder states, a prefix with the spread
of the model's own keys and values), drawn on the GPU from the case's seed.
"""
import math

import numpy as np
import torch

from paper_2608_12703_amd import ad
from paper_2608_12703_amd.configs import Config
from paper_2608_12703_amd.harness import Session
from paper_2608_12703_amd.synth import param_specs

LARGE = dict(d=1280, ffn=5120, vocab=51866, dtype="bf16")
SMALL = dict(d=768, ffn=3072, vocab=51865, dtype="bf16")
TINY = dict(d=384, ffn=1536, vocab=51865, dtype="f32")
# the 11-node candidate tree of the package's tests and benchmark (depth 4)
TREE = [-1, 0, 0, 0, 1, 1, 2, 4, 4, 6, 7]


def listed():
    return [
        # a 64-token decode of the tiny float32 model at batch 1, drafts from four linear
        # heads: one round in the middle of it (verify, commit, draft)
        dict(name="tiny_f32_round_b1", kind="verify", layers=4, **TINY, batch=1, k_min=4, k=4, n_min=40, n=40,
             mix=0, frames_min=1500, frames=1500, packed=False, tree=False, heads=4),
        # the tiny model's setup for a new utterance
        dict(name="tiny_f32_prefill_1", kind="prefill", layers=4, **TINY, batch=1, mix=0, frames_min=1500, frames=1500),
        # the small bf16 model at its configured batch
        dict(name="small_verify_b16", kind="verify", layers=12, **SMALL, batch=16, k_min=4, k=4, n_min=0, n=224,
             mix=0, frames_min=1500, frames=1500, packed=False, tree=False, heads=0),
        # the large-v3 shape for a single live stream (the paper times batch 1)
        dict(name="large_verify_b1", kind="verify", layers=32, **LARGE, batch=1, k_min=6, k=6, n_min=220, n=220,
             mix=0, frames_min=1500, frames=1500, packed=False, tree=False, heads=0),
        # the benchmark's step: 32 sequences, 7 rows each
        dict(name="large_verify_b32", kind="verify", layers=32, **LARGE, batch=32, k_min=6, k=6, n_min=0, n=441,
             mix=0, frames_min=1500, frames=1500, packed=False, tree=False, heads=0),
        # ragged serving batch in the packed layout (eight layers of the stack)
        dict(name="large_ragged_b64", kind="verify", layers=8, **LARGE, batch=64, k_min=2, k=8, n_min=0, n=439,
             mix=0, frames_min=200, frames=1500, packed=True, tree=False, heads=0),
        # an 11-node draft tree per sequence and its commit (eight layers of the stack)
        dict(name="large_tree_b32", kind="verify", layers=8, **LARGE, batch=32, k_min=10, k=10, n_min=0, n=437,
             mix=0, frames_min=1500, frames=1500, packed=False, tree=True, heads=0),
        # one audio-conditioned draft step, the first of a round (it reads the target's taps)
        dict(name="large_draft_b32", kind="draft", d=1280, ffn=2560, vocab=51866, dtype="bf16", batch=32, k=6,
             mix=0, frames_min=1500, frames=1500, first=True),
        # a new utterance joins a live large-v3 session
        dict(name="large_prefill_1", kind="prefill", layers=32, **LARGE, batch=1, mix=0, frames_min=1500, frames=1500),
        # a ragged batch of utterances starts together
        dict(name="large_prefill_16", kind="prefill", layers=32, **LARGE, batch=16, mix=0, frames_min=200, frames=1500),
        # the training objective at the paper's batch of 12 utterances, forward and backward
        dict(name="large_loss_b12", kind="loss", d=1280, ffn=2560, vocab=51866, dtype="bf16", batch=12, rows=128,
             mix=0, frames_min=1500, frames=1500),
        # a sequence's decode state restored from a snapshot and saved again
        dict(name="large_kv_snapshot", kind="kv", layers=32, **LARGE, batch=4, n=220),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify"] * 5 + ["draft", "prefill", "prefill", "loss", "kv"])
    dtype = "f32" if kind in ("verify", "prefill", "draft") and rng.random() < 0.3 else "bf16"
    d = 64 * (_log(rng, 2, 8) if dtype == "f32" else _log(rng, 2, 24))
    ffn = d * (2 if kind in ("draft", "loss") else rng.choice([2, 4]))
    vocab = _log(rng, 997, 51866)
    hi = _log(rng, 33, 1500)
    case = dict(kind=kind, d=d, ffn=ffn, vocab=vocab, dtype=dtype, mix=rng.randint(0, 10**6),
                frames_min=rng.choice([hi, max(1, hi // rng.randint(2, 8))]), frames=hi)
    if kind == "verify":
        k = rng.randint(0, 12)
        tree = rng.random() < 0.2
        k = 10 if tree else k
        n = _log(rng, 1, 448 - 1 - k)
        batch = _log(rng, 1, 6 if dtype == "f32" else 64)
        k_min = k if tree else rng.choice([k, rng.randint(0, k)])
        # (the padded layout leaves the rows past a sequence's own undefined, so blocks of
        # several lengths are packed)
        case.update(layers=rng.randint(1, 4), batch=batch, k_min=k_min, k=k, n_min=rng.choice([n, 0]), n=n,
                    packed=k_min < k or rng.random() < 0.25, tree=tree,
                    heads=k if not tree and 1 <= k <= 4 and batch <= 16 and rng.random() < 0.4 else 0)
    elif kind == "draft":
        case.update(batch=_log(rng, 1, 64), k=rng.randint(1, 8), first=rng.random() < 0.5)
    elif kind == "prefill":
        case.update(layers=rng.randint(1, 4) if dtype == "f32" else rng.randint(1, 16),
                    batch=_log(rng, 1, 2 if dtype == "f32" else 16))
    elif kind == "loss":
        case.update(batch=_log(rng, 1, 12), rows=_log(rng, 5, 128))
    else:
        case.update(layers=rng.randint(1, 32), batch=rng.randint(1, 4), n=_log(rng, 1, 448))
    return case


# ---------------------------------------------------------------------------- inputs

def _rng(seed, what):
    return np.random.default_rng([seed, what])


class _Draw:
    """Normal draws on the GPU from one seed, in call order."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def __call__(self, *shape, scale=1.0, dtype=torch.float32):
        return (torch.randn(*shape, generator=self.g, device="cuda") * scale).to(dtype)


def _config(case, layers):
    return Config(name=case["kind"], n_layers=layers, d_model=case["d"], n_heads=case["d"] // 64,
                  d_ffn=case["ffn"], vocab=case["vocab"], dtype=case["dtype"], batch=case["batch"], k=case.get("k", 0))


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _params(case, layers, draw_):
    d, out = case["d"], []
    for name, shape in param_specs(_config(case, layers)):
        x = draw_(*shape, scale=0.02)
        base = name.split(".")[-1]
        if base.endswith("_g"):
            x += 1.0
        if base == "b_qkv":
            x[d: 2 * d] = 0.0        # keys carry no bias
        if base == "b_xkv":
            x[:d] = 0.0
        out.append(x.to(_dtype(case)))
    return out


def _sizes(case, what, lo, hi):
    """The batch's lengths: the case's own (its `mix`), the same for every seed."""
    return [int(t) for t in _rng(case["mix"], what).integers(lo, hi + 1, size=case["batch"])]


def _frames(case):
    return _sizes(case, 1, case["frames_min"], case["frames"])


def _encoder(case, frames, draw_):
    return [draw_(t, case["d"], dtype=_dtype(case)) for t in frames]


def _verify_inputs(case, seed):
    """Shapes, tokens, weights, encoder states and committed prefixes of a verify round."""
    r, draw_ = _rng(seed, 2), _Draw(seed)
    L, H = case["layers"], case["d"] // 64
    frames = _frames(case)
    ks = _sizes(case, 5, case["k_min"], case["k"])
    ns = _sizes(case, 6, case["n_min"], case["n"])
    blocks = [r.integers(0, case["vocab"], size=k + 1) for k in ks]
    params = _params(case, L, draw_)
    heads = draw_(case["heads"], case["vocab"], case["d"], scale=0.02, dtype=_dtype(case)) if case["heads"] else None
    encs = _encoder(case, frames, draw_)
    prefix = lambda n: draw_(L, 2, n, H, 64, scale=0.02 * math.sqrt(case["d"]), dtype=_dtype(case))
    return frames, ks, ns, blocks, params, heads, encs, prefix


def _path(b):
    """The accepted tree path of sequence b that the commit moves: 1 to 4 nodes deep."""
    return [[0, 2], [0, 2, 6], [0, 1, 4, 7], [0, 1, 4, 7, 10], [0, 2, 6, 9]][b % 5]


def _session(case, params, frames, k, layers, **kw):
    return Session(_config(case, layers), params, case["batch"], k, frames, **kw)


def _fill_encoder(s, encs):
    enc = torch.zeros(s.frames_cap, s.cfg.d_model, dtype=s.dt, device="cuda")
    for off, e in zip(s.enc_off.tolist(), encs):
        enc[off: off + len(e)] = e
    return enc


def prepare(case, seed):
    return {"verify": _prepare_verify, "draft": _prepare_draft, "prefill": _prepare_prefill, "loss": _prepare_loss,
            "kv": _prepare_kv}[case["kind"]](case, seed)


def _prepare_verify(case, seed):
    frames, ks, ns, blocks, params, heads, encs, prefix = _verify_inputs(case, seed)
    s = _session(case, params, frames, case["k"], case["layers"], packed_encoder=case["packed"], want_logits=True,
                 layout=ad.AD_PACKED if case["packed"] else ad.AD_PADDED)
    s.pool.zero_()
    s.cross.zero_()
    ad.cross_kv_prefill(s.model, _fill_encoder(s, encs), s.cross_struct())
    for b, n in enumerate(ns):
        if n:
            ad.kv_import(s.model, s.kv_struct(), b, prefix(n), n, s.err_flag)
    s.prepare(blocks, parents=[TREE] * case["batch"] if case["tree"] else None)
    st = dict(case=case, s=s, n0=torch.tensor(ns, dtype=torch.int32, device="cuda"), heads=heads)
    if case["tree"]:
        acc = [len(_path(b)) - 1 for b in range(case["batch"])]
        path = [_path(b) + [-1] * (case["k"] + 1 - len(_path(b))) for b in range(case["batch"])]
        st["acc"] = torch.tensor(acc, dtype=torch.int32, device="cuda")
        st["path"] = torch.tensor(path, dtype=torch.int32, device="cuda")
    if heads is not None:
        st["next"] = torch.zeros(case["batch"], case["heads"] + 1, dtype=torch.int32, device="cuda")
        st["ws"] = torch.empty(s.model.draft_heads_workspace_size(case["heads"], case["batch"]), dtype=torch.uint8,
                               device="cuda")
    return st


def _prepare_draft(case, seed):
    r, draw_ = _rng(seed, 3), _Draw(seed)
    B, d, k = case["batch"], case["d"], case["k"]
    frames = _frames(case)
    params = _params(case, 1, draw_)
    s = _session(case, params, frames, 0, 1, page_seed=None, want_logits=True)
    s.pool.zero_()
    s.cross.zero_()
    ad.cross_kv_prefill(s.model, _fill_encoder(s, _encoder(case, frames, draw_)), s.cross_struct())
    dt, i32 = _dtype(case), dict(dtype=torch.int32, device="cuda")
    rows = B * (k + 1)
    st = dict(case=case, s=s, fuse=[draw_(d, 4 * d, scale=0.02, dtype=dt), draw_(d, scale=0.02, dtype=dt),
                                    draw_(d, 2 * d, scale=0.02, dtype=dt), draw_(d, scale=0.02, dtype=dt)],
              taps=draw_(3, rows, d), hidden=draw_(rows, d), feature=draw_(B, d), rows=rows,
              accept=torch.tensor(r.integers(0, k + 1, size=B), **i32),
              tokens=torch.tensor(r.integers(0, case["vocab"], size=(B, k + 1)), **i32),
              anchor=torch.tensor([int(r.integers(0, t)) for t in frames], **i32),
              ws=torch.empty(ad.draft_input_workspace_size(s.model, B), dtype=torch.uint8, device="cuda"))
    s.in_rows = torch.zeros(B, d, dtype=torch.float32, device="cuda")
    s.cross_window = torch.zeros(B, 2, **i32)
    lo = [max(0, int(a) - 20) for a in st["anchor"].tolist()]
    s.cross_window.copy_(torch.tensor([[l, min(t, int(a) + 21)] for l, a, t in zip(lo, st["anchor"].tolist(), frames)]))
    s.prepare([np.zeros(1, np.int64)] * B)
    return st


def _prepare_prefill(case, seed):
    draw_ = _Draw(seed)
    frames = _frames(case)
    s = _session(case, _params(case, case["layers"], draw_), frames, 0, case["layers"], packed_encoder=True)
    s.cross.zero_()
    return dict(case=case, s=s, enc=_fill_encoder(s, _encoder(case, frames, draw_)))


def _loss_inputs(case, seed):
    r, draw_ = _rng(seed, 4), _Draw(seed)
    B, R, d = case["batch"], case["rows"], case["d"]
    M, frames = B * R, _frames(case)
    center = np.concatenate([r.integers(0, t, R) for t in frames])
    center[r.random(M) < 0.2] = -1
    targets = r.integers(0, case["vocab"], M)
    targets[r.random(M) < 0.2] = -1
    params = _params(case, 1, draw_)
    encs = _encoder(case, frames, draw_)
    return (frames, center, targets, params, encs, draw_(M, d, scale=0.7), draw_(M, case["vocab"], scale=1.5),
            draw_(M, d, scale=1.5), draw_(M, d))


def _prepare_loss(case, seed):
    frames, center, targets, params, encs, xq, logits, feat, feat_target = _loss_inputs(case, seed)
    B, R, d = case["batch"], case["rows"], case["d"]
    s = _session(case, params, frames, 0, 1)
    s.cross.zero_()
    ad.cross_kv_prefill(s.model, _fill_encoder(s, encs), s.cross_struct())
    i32 = dict(dtype=torch.int32, device="cuda")
    z = lambda *sh: torch.zeros(*sh, dtype=torch.float32, device="cuda")
    return dict(case=case, s=s, xq=xq, logits=logits, feat=feat, feat_target=feat_target,
                center=torch.tensor(center, **i32), targets=torch.tensor(targets, **i32),
                out=dict(terms=z(4), row=z(B * R), dxq=z(B * R, d), dlogits=z(B * R, case["vocab"]), dfeat=z(B * R, d)),
                ws=torch.empty(ad.anchordraft_loss_workspace_size(s.model, B, R), dtype=torch.uint8, device="cuda"))


def _prepare_kv(case, seed):
    draw_ = _Draw(seed)
    cfg = _config(dict(case, ffn=64, vocab=2), case["layers"])
    # the cache of a serving process; its model only carries the shapes here
    s = Session(cfg, _params(dict(case, ffn=64, vocab=2), case["layers"], draw_), case["batch"], 0, [32] * case["batch"],
                pack_weights=False, page_seed=seed % 1000)
    s.pool.zero_()
    src = draw_(case["layers"], 2, case["n"], case["d"] // 64, 64, scale=0.02 * math.sqrt(case["d"]), dtype=_dtype(case))
    return dict(case=case, s=s, src=src, dst=torch.zeros_like(src), b=seed % case["batch"])


# ------------------------------------------------------------------------------- run

def run(st):
    case, s = st["case"], st["s"]
    kind = case["kind"]
    if kind == "verify":
        s.kv_len.copy_(st["n0"])
        s.run()
        out = dict(logits=s.out_logits[: s.rows], hidden=s.out_hidden[: s.rows], margin=s.out_margin[: s.rows],
                   greedy=s.out_greedy[: s.rows], accept=s.accept_len, tokens=s.out_tokens, kv_len=s.kv_len,
                   pool=s.pool, err=s.err_flag)
        if case["tree"]:
            ad.kv_commit_tree(s.model, s.kv_struct(), st["acc"], st["path"], case["k"] + 1, case["batch"])
            out["path"] = s.out_path
        else:
            s.commit()
        if st["heads"] is not None:
            ad.draft_heads(s.model, st["heads"], case["heads"], s.out_hidden, s.layout, s.k_max, s.cu_rows,
                           s.accept_len, s.out_tokens, case["batch"], st["next"], st["ws"])
            out["next"] = st["next"]
        return out
    if kind == "draft":
        f, k = st["fuse"], case["k"]
        if case["first"]:
            ad.draft_input(s.model, *f, case["batch"], st["taps"], st["hidden"], ad.AD_PADDED, k, None, st["accept"],
                           st["rows"], None, st["tokens"], k + 1, st["accept"], st["anchor"], s.enc_len, 20,
                           s.cross_window, s.in_rows, st["ws"])
        else:
            ad.draft_input(s.model, *f, case["batch"], None, None, ad.AD_PADDED, k, None, None, st["rows"],
                           st["feature"], st["tokens"], k + 1, None, None, None, 0, None, s.in_rows, st["ws"])
        s.run()
        return dict(in_rows=s.in_rows, window=s.cross_window, logits=s.out_logits, hidden=s.out_hidden,
                    greedy=s.out_greedy, pool=s.pool, err=s.err_flag)
    if kind == "prefill":
        ad.cross_kv_prefill(s.model, st["enc"], s.cross_struct())
        return s.cross
    if kind == "loss":
        o = st["out"]
        ad.anchordraft_loss(s.model, s.cross_struct(), 0, case["batch"], case["rows"], st["xq"], st["center"], 5.0, 0.1,
                            st["logits"], st["targets"], st["feat"], st["feat_target"], o["terms"], o["row"], o["dxq"],
                            o["dlogits"], o["dfeat"], s.err_flag, st["ws"])
        return dict(o, err=s.err_flag)
    ad.kv_import(s.model, s.kv_struct(), st["b"], st["src"], case["n"], s.err_flag)
    ad.kv_export(s.model, s.kv_struct(), st["b"], st["dst"], case["n"], s.err_flag)
    return dict(saved=st["dst"], pool=s.pool, err=s.err_flag)


# ------------------------------------------------------------------------------ work

def _size(case):
    return 2 if case["dtype"] == "bf16" else 4


def work(case):
    """(Lengths and frames of a ragged batch by their means.)"""
    e, d, V, B = _size(case), case["d"], case["vocab"], case["batch"]
    F, L, kind = case["ffn"], case.get("layers", 1), case["kind"]
    T = (case["frames_min"] + case["frames"]) / 2 if "frames" in case else 0
    layer = 6 * d * d + 2 * d * F              # projection weights of one layer that a step reads
    if kind == "verify":
        rows = B * ((case["k_min"] + case["k"]) / 2 + 1)
        n = (case["n_min"] + case["n"]) / 2
        b = e * (L * layer + V * d + L * B * 2 * d * (T + n)) + 4 * rows * (V + d) + e * L * rows * 2 * d
        f = 2 * rows * (L * layer + V * d) + L * 4 * rows * d * (T + n)
        if case["heads"]:
            b += e * case["heads"] * V * d
            f += 2 * B * case["heads"] * V * d
        return dict(bytes=b, flops=f)
    if kind == "draft":
        win = min(41, T)
        fuse = (6 if case["first"] else 2) * d * d
        b = e * (fuse + layer + V * d + B * 2 * d * win) + 4 * B * ((4 if case["first"] else 1) * d + V + 2 * d)
        return dict(bytes=b, flops=2 * B * (fuse + layer + V * d) + 4 * B * d * win)
    if kind == "prefill":
        return dict(bytes=e * (B * T * d + L * (2 * d * d + B * T * 2 * d)), flops=L * 2 * B * T * d * 2 * d)
    if kind == "loss":
        M = B * case["rows"]
        return dict(bytes=4 * M * (2 * V + 5 * d) + e * B * T * d, flops=M * T * d * 2 * 3)
    return dict(bytes=4 * e * L * 2 * case["n"] * d, flops=0)


# Relative errors: about four times what these outputs were measured off their 64-bit values.
# bf16 models keep activations in 32 bits and enter the products as pairs of bf16 values
# (16 significant bits), and a key or value near a rounding boundary of its bf16 cache slot
# may fall on either side of it (one ulp, at most 2^-7 of the value), which the following
# layers carry on: hidden rows and logits 1e-5 to 6e-5, top-2 margins (a difference of two
# logits) up to 2.2e-4.  Whole values may differ at near ties of the logits.
def tolerance(case):
    if case["kind"] == "kv":
        return "exact"
    if case["kind"] == "prefill":              # 3.5e-7 (float32), 2.6e-5 (bf16)
        return dict(rel=2e-6, max=2e-4) if case["dtype"] == "f32" else dict(rel=1e-4, max=1.6e-2)
    if case["dtype"] == "f32":                 # logits 1.2e-6, margins 1.3e-5
        return dict(rel=5e-5, max=2e-3, differ=0.01)
    if case["kind"] == "loss":                 # the query gradient 3.5e-5
        return dict(rel=1.5e-4, max=1.6e-2)
    return dict(rel=1e-3, max=4e-2, differ=0.01)


# ----------------------------------------------------------------------------- exact

def exact(case, seed):
    if case["kind"] == "verify":
        return _exact_verify(case, seed)
    if case["kind"] == "draft":
        return _exact_draft(case, seed)
    if case["kind"] == "prefill":
        return _exact_prefill(case, seed)
    if case["kind"] == "loss":
        return _exact_loss(case, seed)
    return None


def _ln(x, g, b):
    return (x - x.mean(-1, keepdim=True)) / torch.sqrt(x.var(-1, unbiased=False, keepdim=True) + 1e-5) * g + b


def _gelu(u):
    return 0.5 * u * (1 + torch.erf(u / math.sqrt(2.0)))


def _attend(q, K, V, see):
    """q [r, H, 64], K and V [n, H, 64], see [r, n] or None."""
    s = torch.matmul(q.transpose(0, 1), K.permute(1, 2, 0).contiguous()) / 8
    if see is not None:
        s = s.masked_fill(~see, -math.inf)
    return torch.matmul(torch.softmax(s, -1), V.transpose(0, 1).contiguous()).transpose(0, 1).reshape(len(q), -1)


def _store(case, x):
    """What the caches hold: keys and values rounded to the model's type."""
    return x.to(_dtype(case)).double()


def _decoder(case, params, layers, xs, pres, encs, sees, windows=None):
    """The pre-LN decoder over the rows xs[b] of every sequence, in 64 bits.  pres[b](l):
    the committed keys and values; returns the final rows and every layer's new ones."""
    d, H = case["d"], case["d"] // 64
    new = [[] for _ in xs]
    for l in range(layers):
        (g1, b1, wqkv, bqkv, wo, bo, g2, b2, wxq, bxq, wxkv, bxkv, wxo, bxo, g3, b3, w1, c1, w2, c2) = [
            p.double() for p in params[4 + 20 * l: 24 + 20 * l]]
        for b, x in enumerate(xs):
            r = len(x)
            q, k, v = (_ln(x, g1, b1) @ wqkv.T + bqkv).split(d, -1)
            k, v = _store(case, k).view(r, H, 64), _store(case, v).view(r, H, 64)
            new[b].append((k, v))
            pk, pv = pres[b](l)
            x = x + _attend(q.view(r, H, 64), torch.cat([pk, k]), torch.cat([pv, v]), sees[b]) @ wo.T + bo
            e = encs[b].double()
            if windows is not None:
                e = e[windows[b][0]: windows[b][1]]
            ck, cv = (e @ wxkv.T + bxkv).split(d, -1)
            q = _ln(x, g2, b2) @ wxq.T + bxq
            x = x + _attend(q.view(r, H, 64), _store(case, ck).view(-1, H, 64), _store(case, cv).view(-1, H, 64),
                            None) @ wxo.T + bxo
            xs[b] = x + _gelu(_ln(x, g3, b3) @ w1.T + c1) @ w2.T + c2
    return [_ln(x, params[2].double(), params[3].double()) for x in xs], new


def _exact_verify(case, seed):
    frames, ks, ns, blocks, params, heads, encs, prefix = _verify_inputs(case, seed)
    B = case["batch"]
    pre = [prefix(n) if n else torch.zeros(case["layers"], 2, 0, case["d"] // 64, 64, device="cuda") for n in ns]
    depth = [0] * len(TREE)
    mask = torch.zeros(len(TREE), len(TREE), dtype=torch.bool)
    for i, p in enumerate(TREE):
        if p >= 0:
            depth[i] = depth[p] + 1
            mask[i] = mask[p]
        mask[i, i] = True
    tok, pos = params[0].double(), params[1].double()
    xs, sees = [], []
    for b in range(B):
        r = ks[b] + 1
        at = torch.tensor(depth if case["tree"] else list(range(r)), device="cuda") + ns[b]
        xs.append(tok[torch.tensor(blocks[b], device="cuda")] + pos[at])
        m = mask if case["tree"] else torch.ones(r, r, dtype=torch.bool).tril()
        sees.append(torch.cat([torch.ones(r, ns[b], dtype=torch.bool), m], 1).cuda())
    hid, new = _decoder(case, params, case["layers"], xs, [lambda l, p=p: (p[l, 0].double(), p[l, 1].double()) for p in pre],
                        encs, sees)
    hid = torch.cat(hid)
    logits = hid @ tok.T
    top = logits.topk(2, -1).values
    out = dict(logits=logits, hidden=hid, margin=top[:, 0] - top[:, 1], greedy=None, accept=None, tokens=None,
               kv_len=None, pool=None, err=None)
    if case["tree"]:
        out["path"] = None
    if heads is not None:
        out["next"] = None
    return out


def _exact_draft(case, seed):
    r, draw_ = _rng(seed, 3), _Draw(seed)
    B, d, k = case["batch"], case["d"], case["k"]
    frames = _frames(case)
    params = _params(case, 1, draw_)
    encs = _encoder(case, frames, draw_)
    dt, rows = _dtype(case), case["batch"] * (case["k"] + 1)
    wf, bf, wi, bi = (w.double() for w in (draw_(d, 4 * d, scale=0.02, dtype=dt), draw_(d, scale=0.02, dtype=dt),
                                           draw_(d, 2 * d, scale=0.02, dtype=dt), draw_(d, scale=0.02, dtype=dt)))
    taps, hidden, feature = draw_(3, rows, d).double(), draw_(rows, d).double(), draw_(B, d).double()
    acc = torch.tensor(r.integers(0, k + 1, size=B), device="cuda")
    tokens = torch.tensor(r.integers(0, case["vocab"], size=(B, k + 1)), device="cuda")
    anchor = [int(r.integers(0, t)) for t in frames]
    at = torch.arange(B, device="cuda")
    if case["first"]:
        row = at * (k + 1) + acc
        f = torch.cat([taps[0][row], taps[1][row], taps[2][row], hidden[row]], -1) @ wf.T + bf
        t = tokens[at, acc]
    else:
        f, t = feature, tokens[:, 0]
    tok = params[0].double()
    u = torch.cat([f, tok[t]], -1) @ wi.T + bi
    empty = torch.zeros(0, d // 64, 64, dtype=torch.float64, device="cuda")
    win = [(max(0, c - 20), min(T, c + 21)) for c, T in zip(anchor, frames)]
    hid, _ = _decoder(case, params, 1, [u[b: b + 1] + params[1].double()[:1] for b in range(B)],
                      [lambda l: (empty, empty)] * B, encs, [None] * B, win)
    hid = torch.cat(hid)
    return dict(in_rows=u, window=None, logits=hid @ tok.T, hidden=hid, greedy=None, pool=None, err=None)


def _exact_prefill(case, seed):
    draw_ = _Draw(seed)
    frames, d, H, L = _frames(case), case["d"], case["d"] // 64, case["layers"]
    slots = [(t + 31) // 32 * 32 for t in frames]
    if L * 2 * d * sum(slots) > 2_000_000_000:    # 16 GB of values in 64 bits
        return None
    params = _params(case, L, draw_)
    enc = torch.zeros(sum(slots), d, dtype=torch.float64, device="cuda")
    off = 0
    for e, sl in zip(_encoder(case, frames, draw_), slots):
        enc[off: off + len(e)] = e.double()
        off += sl
    out = torch.empty(L, H, len(enc) // 32, 2, 2048, dtype=torch.float64, device="cuda")
    # the cache's order inside a 32-frame block: frame t, lane j
    t, j = torch.arange(32, device="cuda")[:, None], torch.arange(64, device="cuda")[None, :]
    at_k = (((t // 4 % 2) * 2 + (j // 8) % 2) * 64 + (j // 16) * 16 + 4 * (t // 8) + t % 4) * 8 + j % 8
    at_v = ((j // 16) * 64 + (t // 8) * 16 + j % 16) * 8 + t % 8
    for l in range(L):
        w, bias = params[4 + 20 * l + 10].double(), params[4 + 20 * l + 11].double()
        kv = (enc @ w.T + bias).view(len(enc) // 32, 32, 2, H, 64)
        if case["dtype"] == "bf16":
            kv = _store(case, kv)
        for which, at in ((0, at_k), (1, at_v)):
            out[l, :, :, which][..., at.reshape(-1)] = kv[:, :, which].permute(2, 0, 1, 3).reshape(H, -1, 2048)
    return out.reshape(-1)


def _exact_loss(case, seed):
    frames, center, targets, params, encs, xq, logits, feat, feat_target = _loss_inputs(case, seed)
    B, R, d, H = case["batch"], case["rows"], case["d"], case["d"] // 64
    w = params[4 + 10].double()
    center, targets = torch.tensor(center, device="cuda"), torch.tensor(targets, device="cuda")
    aligned, has = center >= 0, targets >= 0
    nv, nt = max(1, int(aligned.sum())), max(1, int(has.sum()))
    row, dxq = torch.zeros(B * R, dtype=torch.float64, device="cuda"), torch.zeros(B * R, d, dtype=torch.float64, device="cuda")
    for b, T in enumerate(frames):
        K = _store(case, encs[b].double() @ w[:d].T).view(T, H, 64).transpose(0, 1).contiguous()
        x = xq[b * R: (b + 1) * R].double().view(R, H, 64).transpose(0, 1).contiguous().requires_grad_()
        c = center[b * R: (b + 1) * R]
        q = torch.exp(-(torch.arange(T, device="cuda").double() - c[:, None]) ** 2 / 50.0)
        q = q / q.sum(-1, keepdim=True)
        abar = torch.softmax(torch.matmul(x, K.transpose(1, 2).contiguous()) / 8, -1).mean(0)
        ell = -(q * abar.log()).sum(-1) * (c >= 0)
        (0.1 / nv * ell.sum()).backward()
        row[b * R: (b + 1) * R] = ell.detach()
        dxq[b * R: (b + 1) * R] = x.grad.transpose(0, 1).reshape(R, d)
    z = logits.double()
    y = targets.clamp(min=0)[:, None]
    tok = (torch.logsumexp(z, -1) - z.gather(1, y)[:, 0]) * has
    dlogits = torch.softmax(z, -1)
    dlogits.scatter_add_(1, y, torch.full_like(y, -1, dtype=torch.float64))
    dlogits *= (has / nt)[:, None]
    e = feat.double() - feat_target.double()
    ft = torch.where(e.abs() < 1, 0.5 * e * e, e.abs() - 0.5).sum(-1) * has
    dfeat = e.clamp(-1, 1) * (0.5 / (nt * d)) * has[:, None]
    la, lt, lf = row.sum() / nv, tok.sum() / nt, ft.sum() / (nt * d)
    return dict(terms=torch.stack([lt + 0.5 * lf + 0.1 * la, lt, lf, la]), row=row, dxq=dxq, dlogits=dlogits,
                dfeat=dfeat, err=None)
