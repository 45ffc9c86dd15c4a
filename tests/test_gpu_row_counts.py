"""The projections and the LM head at the row counts where the launch changes kernel or tile.

A launch with few 16 x 16 output tiles runs the register-direct product (one to eight tiles
per wave), a larger one the LDS product.  The LM head runs the register-direct product at 1, 2,
3, 5 and 6 row tiles where the LDS product would take a second round of workgroups (33001
columns are 258 tiles of 128; three row tiles from width 768 on), and at one row tile of tiled
weights up to width 768; the other vocabularies here take the LDS product otherwise.
One row per sequence: the same sequences in batches of every size must give the same bits
(the order of a row's sums never depends on the launch), and the rows must match the oracle.
The float32 product changes its tile by the number of 16 x 16 output tiles (the vocabulary of
33001 columns reaches its larger ones at every row count).  Widths: 192 (not a multiple of the 128-column weight tile, odd vocabulary) and 1280 (the
two-row-tile waves).  Tolerance against the oracle: the logit bar of the parity tests.
"""
import numpy as np
import pytest
import torch

from oracle import decoder as od
from paper_2608_12703_amd import ad, synth
from paper_2608_12703_amd.configs import Config
from paper_2608_12703_amd.harness import Session, upload_params

from gpu_common import LOGIT_TOL

pytestmark = pytest.mark.gpu

FRAMES = 33


def _run(cfg, plist, encs, tokens, pack):
    s = Session(cfg, plist, len(tokens), 0, [FRAMES] * len(tokens), want_logits=True, pack_weights=pack)
    s.prefill_encoder(encs[: len(tokens)])
    s.step([[t] for t in tokens])
    r = s.results()
    assert r["err"] == 0
    return r


@pytest.mark.parametrize("dtype,d,ffn,vocab,rows,pack", [
    ("bf16", 192, 384, 1003, (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 81, 96, 97, 112), True),
    ("bf16", 192, 384, 1003, (1, 33, 81), False),
    ("bf16", 1280, 5120, 517, (16, 17, 49, 80, 81, 112), True),
    # the register-direct LM head at every row tile count that it takes
    ("bf16", 768, 128, 33001, (1, 16, 17, 32, 33, 48, 49, 65, 80, 81, 96, 97), True),
    ("bf16", 768, 128, 33001, (16, 32, 48, 96), False),
    # the 256-column LM head: 12 and 16 row tiles per workgroup, one and two row chunks (33001
    # columns x 385 rows stay with 128-column workgroups)
    ("bf16", 128, 128, 51865, (272, 385), True),
    ("bf16", 128, 128, 33001, (97, 112, 192, 193, 272, 385), True),
    ("bf16", 128, 128, 33001, (97, 272), False),
    ("f32", 192, 384, 33001, (1, 16, 17, 32, 33, 49), False),
    ("f32", 64, 64, 1003, (1, 17, 33), False),
    # LayerNorm inside the product and as a launch of its own (the widest fused row; the up
    # product of 257 rows and the QKV product of 400 have more than 2048 tiles)
    ("f32", 512, 2048, 515, (1, 17, 256, 257), False),
])
def test_rows_do_not_depend_on_the_launch(dtype, d, ffn, vocab, rows, pack):
    top = 400 if max(rows) > 200 else 200 if dtype == "bf16" else 70    # 25, 13 and 5 row tiles
    cfg = Config(name="rows", n_layers=1, d_model=d, n_heads=d // 64, d_ffn=ffn, vocab=vocab, dtype=dtype,
                 batch=top, k=0, frames=FRAMES, seed=21)
    params = synth.make_params(cfg)
    plist = upload_params(cfg, params)
    encs = [synth.make_encoder(cfg, b, FRAMES) for b in range(top)]
    tokens = [int(t) for t in np.random.default_rng(4).integers(0, vocab, top)]
    full = _run(cfg, plist, encs, tokens, pack)
    model = od.Model(cfg, params)
    for b in (0, 16, top - 1):
        ref = od.verify(model, od.new_state(model, od.cross_kv(model, encs[b]), tokens[b]), np.zeros(0, np.int64))
        assert float(np.max(np.abs(full["logits"][b] - ref.logits[0]))) <= LOGIT_TOL[dtype]
    for n in rows:
        got = _run(cfg, plist, encs, tokens[:n], pack)
        for key in ("hidden", "logits", "margin"):
            np.testing.assert_array_equal(got[key].view(np.uint32), full[key][:n].view(np.uint32),
                                          err_msg=f"{key} at {n} rows")
        np.testing.assert_array_equal(got["greedy"], full["greedy"][:n])
        torch.cuda.synchronize()


@pytest.mark.parametrize("batch,n_heads", [(1, 4), (17, 2), (33, 1)])
def test_bf16_draft_heads_pick_the_largest_logit(batch, n_heads):
    """Drafts of bf16 heads against the float64 products (a draft may differ only where the
    float64 logits tie within 1e-5, far above the float32 sums' error of ~1e-6)."""
    d, vocab, k = 192, 5003, 2
    cfg = Config(name="heads", n_layers=1, d_model=d, n_heads=3, d_ffn=64, vocab=vocab, dtype="bf16", batch=batch,
                 k=k, frames=32, seed=8)
    s = Session(cfg, synth.make_params(cfg), batch, k, [32] * batch)
    g = torch.Generator(device="cuda").manual_seed(1)
    w = (torch.randn(n_heads, vocab, d, generator=g, device="cuda") * 0.02).bfloat16()
    hidden = torch.randn(batch * (k + 1), d, generator=g, device="cuda")
    r = np.random.default_rng(2)
    acc = torch.tensor(r.integers(0, k + 1, batch), dtype=torch.int32, device="cuda")
    toks = torch.tensor(r.integers(0, vocab, (batch, k + 1)), dtype=torch.int32, device="cuda")
    nxt = torch.zeros(batch, n_heads + 1, dtype=torch.int32, device="cuda")
    ws = torch.empty(s.model.draft_heads_workspace_size(n_heads, batch), dtype=torch.uint8, device="cuda")
    ad.draft_heads(s.model, w, n_heads, hidden, ad.AD_PADDED, k, None, acc, toks, batch, nxt, ws)
    row = torch.arange(batch, device="cuda") * (k + 1) + acc
    for i in range(n_heads):
        z = hidden[row].double() @ w[i].double().T
        assert torch.all(z.gather(1, nxt[:, 1 + i: 2 + i].long())[:, 0] >= z.max(-1).values - 1e-5)
    assert torch.equal(nxt[:, 0], toks[torch.arange(batch), acc.long()])
