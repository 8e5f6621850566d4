"""Tree attention (GPU): the exponent of a row's largest score is zero, whatever the score's size, so that a
row that sees a single key returns that key's value, exactly."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv_heads,hd", [(4, 4, 64), (4, 2, 64), (4, 4, 128), (4, 2, 128), (6, 2, 128)])
@pytest.mark.parametrize("size", [1.0, 3000.0])
def test_a_single_visible_key_returns_its_value(heads, kv_heads, hd, size):
    import paper_2401_12522_amd as bita
    B, parent = 5, synth.star_tree(9)
    R = len(parent)
    tmpl = bita.TreeTemplate(parent, np.zeros(R, np.uint8), R, 4)
    g = torch.Generator(device="cuda").manual_seed(heads * hd)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")                      # noqa: E731
    kt = rnd(B, kv_heads, R, hd).to(torch.bfloat16)
    v = rnd(B, kv_heads, R, hd)
    vt = v.to(torch.bfloat16)
    vt_lo = (v - vt.float()).to(torch.bfloat16)
    q = (kt.repeat_interleave(heads // kv_heads, 1).transpose(1, 2).float() * size).to(torch.bfloat16).contiguous()
    cache = torch.zeros(B, kv_heads, 8, hd, dtype=torch.bfloat16, device="cuda")
    hi, lo = bita.tree_attention(tmpl, q, cache, cache, kt, vt, None, None, torch.zeros(B, dtype=torch.int32, device="cuda"), 0,
                                 v_tree_lo=vt_lo, two_plane_out=True)
    root = (hi.double() + lo.double()).view(B, R, heads, hd)[:, 0]                   # no context, no prefix: the root sees itself
    want = (vt.double() + vt_lo.double())[:, :, 0].repeat_interleave(heads // kv_heads, 1)
    assert torch.equal(root, want), (root - want).abs().max().item()
