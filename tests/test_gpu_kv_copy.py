"""ad_kv_import / ad_kv_export byte for byte: every element against the cache's tile layout
(keys token-major, values lane-major in 16-token tiles), at tile edges and remainders, for an
aligned and a misaligned linear array (the two copy kernels), slots past the prefix left alone,
and a page index outside the pool."""
import numpy as np
import pytest
import torch

from paper_2608_12703_amd import ad, synth
from paper_2608_12703_amd.configs import Config
from paper_2608_12703_amd.harness import Session

pytestmark = pytest.mark.gpu


def _session(dtype, heads):
    cfg = Config(name="kvcopy", n_layers=2, d_model=64 * heads, n_heads=heads, d_ffn=64, vocab=10, dtype=dtype,
                 batch=2, k=1, frames=32, seed=3)
    return cfg, Session(cfg, synth.make_params(cfg), 2, 1, [32, 32], page_seed=7)


def _slots(s, cfg, b, n):
    """Pool index of every element of the logical array [L][2][n][H][64]."""
    H = cfg.n_heads
    pages = s.block_table.cpu().numpy()[b]
    l, kv, p, h, j = np.meshgrid(np.arange(cfg.n_layers), np.arange(2), np.arange(n), np.arange(H), np.arange(64),
                                 indexing="ij")
    base = (((l * 2 + kv) * s.num_pages + pages[p // 16]) * H + h) * 1024
    return base + np.where(kv == 0, (p % 16) * 64 + j, j * 16 + p % 16)


@pytest.mark.parametrize("dtype,heads", [("bf16", 3), ("f32", 5)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 37, 448])
@pytest.mark.parametrize("shift", [0, 1])
def test_copies_are_exact(dtype, heads, n, shift):
    cfg, s = _session(dtype, heads)
    b, size = 1, cfg.n_layers * 2 * n * heads * 64
    g = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(size + 8, generator=g, device="cuda").to(s.dt)
    src = buf[shift: shift + size]           # shift 1: not 16-byte aligned
    s.pool.copy_(torch.randn(s.pool.numel(), generator=g, device="cuda"))
    want = s.pool.clone()
    idx = torch.tensor(_slots(s, cfg, b, n).reshape(-1), device="cuda")
    want[idx] = src
    ad.kv_import(s.model, s.kv_struct(), b, src, n, s.err_flag)
    assert torch.equal(s.pool, want)
    out = torch.zeros(size + 8, dtype=s.dt, device="cuda")
    ad.kv_export(s.model, s.kv_struct(), b, out[shift: shift + size], n, s.err_flag)
    assert torch.equal(out[shift: shift + size], src)
    assert not torch.any(out[:shift]) and not torch.any(out[shift + size:])
    assert int(s.err_flag.item()) == 0


def test_page_outside_the_pool_sets_the_flag_and_writes_nothing():
    cfg, s = _session("bf16", 3)
    s.block_table[0, 0] = s.num_pages
    s.pool.zero_()
    src = torch.ones(cfg.n_layers, 2, 16, 3, 64, dtype=s.dt, device="cuda")
    ad.kv_import(s.model, s.kv_struct(), 0, src, 16, s.err_flag)
    assert int(s.err_flag.item()) == ad.AD_ERR_PAGE and not torch.any(s.pool)
