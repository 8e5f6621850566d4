"""Tree attention (GPU) over more K/V heads than a launch has workgroups along one of its axes: one row per sequence on
no cached key or one, every sequence against the two-key formula in 64 bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,heads,kv_heads", [(65541, 8, 8), (131100, 8, 4), (1 << 18, 2, 1)])
def test_more_kv_heads_than_a_grid_axis(batch, heads, kv_heads):
    import paper_2401_12522_amd as bita
    hd = 64
    g = torch.Generator(device="cuda").manual_seed(heads)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    q, kc, vc, kt, vt = rnd(batch, 1, heads, hd), *(rnd(batch, kv_heads, 1, hd) for _ in range(4))
    lens = torch.arange(batch, dtype=torch.int32, device="cuda") % 2
    tmpl = bita.TreeTemplate(np.array([-1], np.int32), np.zeros(1, np.uint8), 1, 4)
    hi, lo = bita.tree_attention(tmpl, q, kc, vc, kt, vt, None, None, lens, 1, two_plane_out=True)
    worst = 0.0
    for at in range(0, batch, 16384):
        s = slice(at, at + 16384)
        keys = torch.cat([kc[s], kt[s]], 2).double().repeat_interleave(heads // kv_heads, 1)      # [b][heads][2][hd]
        vals = torch.cat([vc[s], vt[s]], 2).double().repeat_interleave(heads // kv_heads, 1)
        score = (keys * q[s].double().view(-1, heads, 1, hd)).sum(-1) / 8.0
        score[..., 0].masked_fill_(lens[s, None] == 0, float("-inf"))
        ref = (torch.softmax(score, -1)[..., None] * vals).sum(2)
        out = (hi[s].double() + lo[s].double()).view(-1, heads, hd)
        worst = max(worst, float((out - ref).abs().max()))
    assert worst < 1e-4, worst                                   # the kernel tests' two-plane regression bound
