"""The projections and the LM head at the row counts where the launch changes kernel or tile.

A launch with few 16 x 16 output tiles runs the register-direct product (one to eight tiles
per wave), a larger one the LDS product, and the LM head switches at 1, 2, 3, 5-6 row tiles.
One row per sequence: the same sequences in batches of every size must give the same bits
(the order of a row's sums never depends on the launch), and the rows must match the oracle.
Widths: 192 (not a multiple of the 128-column weight tile, odd vocabulary) and 1280 (the
two-row-tile waves).  Tolerance against the oracle: the logit bar of the parity tests.
"""
import numpy as np
import pytest
import torch

from oracle import decoder as od
from paper_2608_12703_amd import synth
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


@pytest.mark.parametrize("d,ffn,vocab,rows,pack", [
    (192, 384, 1003, (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 81, 96, 97, 112), True),
    (192, 384, 1003, (1, 33, 81), False),
    (1280, 5120, 517, (16, 17, 49, 80, 81, 112), True),
])
def test_rows_do_not_depend_on_the_launch(d, ffn, vocab, rows, pack):
    top = 200    # 13 row tiles
    cfg = Config(name="rows", n_layers=1, d_model=d, n_heads=d // 64, d_ffn=ffn, vocab=vocab, dtype="bf16",
                 batch=top, k=0, frames=FRAMES, seed=21)
    params = synth.make_params(cfg)
    plist = upload_params(cfg, params)
    encs = [synth.make_encoder(cfg, b, FRAMES) for b in range(top)]
    tokens = [int(t) for t in np.random.default_rng(4).integers(0, vocab, top)]
    full = _run(cfg, plist, encs, tokens, pack)
    model = od.Model(cfg, params)
    for b in (0, 16, 111):
        ref = od.verify(model, od.new_state(model, od.cross_kv(model, encs[b]), tokens[b]), np.zeros(0, np.int64))
        assert float(np.max(np.abs(full["logits"][b] - ref.logits[0]))) <= LOGIT_TOL["bf16"]
    for n in rows:
        got = _run(cfg, plist, encs, tokens[:n], pack)
        for key in ("hidden", "logits", "margin"):
            np.testing.assert_array_equal(got[key].view(np.uint32), full[key][:n].view(np.uint32),
                                          err_msg=f"{key} at {n} rows")
        np.testing.assert_array_equal(got["greedy"], full["greedy"][:n])
        torch.cuda.synchronize()
