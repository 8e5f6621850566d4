"""Tree attention (GPU) where several query heads of a K/V head share a tile of 16 queries, and where none do: every number
of heads per K/V head that shares tiles differently, at row counts around a tile's rows, with few workgroups and with many, and
with the keys split between workgroups."""
import math

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv_heads,hd", [(4, 4, 64), (4, 4, 128), (4, 2, 64), (8, 2, 64), (6, 1, 128), (8, 2, 128), (8, 1, 128), (24, 2, 64), (12, 1, 128), (16, 1, 128),
                                               (32, 1, 64)])
@pytest.mark.parametrize("rows,batch,longest", [(1, 1, 2100), (2, 2, 40), (3, 70, 33), (5, 3, 300), (17, 2, 64), (33, 40, 31)])
def test_heads_that_share_a_tile(heads, kv_heads, hd, rows, batch, longest):
    import paper_2401_12522_amd as bita
    tin = synth.attach_mask_groups(synth.random_tree(rows, 4, rows), [0], 4) if rows > 1 else None
    parent, is_mask, n_tree = (tin.parent, tin.is_mask, tin.n_tree) if tin else (np.array([-1], np.int32), np.zeros(1, np.uint8), 1)
    tmpl = bita.TreeTemplate(parent, is_mask, n_tree, 4)
    R, P, lens = len(parent), 5, [longest - i % (longest + 1) for i in range(batch)]
    g = torch.Generator(device="cuda").manual_seed(heads * 100 + rows)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")                      # noqa: E731
    b16 = lambda x: x.to(torch.bfloat16)                                             # noqa: E731
    q, kc, vc = b16(rnd(batch, R, heads, hd)), b16(rnd(batch, kv_heads, longest, hd)), b16(rnd(batch, kv_heads, longest, hd))
    kt, vt, pk, pv = b16(rnd(batch, kv_heads, R, hd)), b16(rnd(batch, kv_heads, R, hd)), b16(rnd(kv_heads, P, hd)), b16(rnd(kv_heads, P, hd))
    hi, lo = bita.tree_attention(tmpl, q, kc, vc, kt, vt, pk, pv, torch.tensor(lens, dtype=torch.int32, device="cuda"), longest,
                                 two_plane_out=True)
    out = (hi.double() + lo.double()).view(batch, R, heads, hd)
    inside = np.zeros((R, R), bool)
    for i, p in enumerate(parent):
        if p >= 0:
            inside[i] = inside[p]
        inside[i, i] = True
    inside, masks = torch.tensor(inside, device="cuda"), torch.tensor(np.asarray(is_mask).astype(bool), device="cuda")
    for b in sorted({0, batch // 2, batch - 1}):
        n = lens[b]
        seen = torch.cat([masks[:, None].expand(R, P), torch.ones(R, n, dtype=torch.bool, device="cuda"), inside], 1)
        for h in range(heads):
            kv = h * kv_heads // heads
            keys = torch.cat([pk[kv], kc[b, kv, :n], kt[b, kv]]).double()
            vals = torch.cat([pv[kv], vc[b, kv, :n], vt[b, kv]]).double()
            p = torch.softmax(((q[b, :, h].double() @ keys.T) / math.sqrt(hd)).masked_fill(~seen, -math.inf), -1)
            err = float((out[b, :, h] - p @ vals).abs().max())
            assert err < 1e-4, (b, n, h, err)                                        # the kernel tests' two-plane regression bound
