"""Tree attention (GPU) where the running maximum moves in almost every chunk, or only in the last one,
or scores are far below the first chunk's, at chunk and wave edges of the context, one and two query
heads per workgroup, both head dimensions."""
import math

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv_heads,hd", [(4, 4, 64), (4, 2, 64), (4, 4, 128), (4, 2, 128), (6, 2, 128)])
@pytest.mark.parametrize("growth", [4.0, 0.25])
def test_running_maximum_moves(heads, kv_heads, hd, growth):
    import paper_2401_12522_amd as bita
    lens = [0, 1, 31, 33, 256, 300, 777]
    B, P, tin = len(lens), 8, synth.attach_mask_groups(synth.random_tree(21, 4, 5), [0], 4)
    R, smax = tin.rows, max(lens) + 3
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, 4)
    g = torch.Generator(device="cuda").manual_seed(heads * hd + int(growth * 8))
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")                      # noqa: E731
    b16 = lambda x: x.to(torch.bfloat16)                                             # noqa: E731
    ramp = growth ** (torch.arange(smax, device="cuda") / smax)                      # key norms grow (or shrink) by `growth`
    q, kc, vc = b16(rnd(B, R, heads, hd)), b16(rnd(B, kv_heads, smax, hd) * ramp[:, None]), b16(rnd(B, kv_heads, smax, hd))
    kc[:, :, -1] = float("nan")                                                      # slots past every context are never read into a result
    kt, vt, pk, pv = b16(rnd(B, kv_heads, R, hd) * growth), b16(rnd(B, kv_heads, R, hd)), b16(rnd(kv_heads, P, hd)), b16(rnd(kv_heads, P, hd))
    hi, lo = bita.tree_attention(tmpl, q, kc, vc, kt, vt, pk, pv, torch.tensor(lens, dtype=torch.int32, device="cuda"), max(lens),
                                 two_plane_out=True)
    out = hi.double().view(B, R, heads, hd) + lo.double().view(B, R, heads, hd)
    inside = np.zeros((R, R), bool)
    for i, p in enumerate(tin.parent):
        if p >= 0:
            inside[i] = inside[p]
        inside[i, i] = True
    inside, masks = torch.tensor(inside, device="cuda"), torch.tensor(tin.is_mask.astype(bool), device="cuda")
    for b, n in enumerate(lens):
        seen = torch.cat([masks[:, None].expand(R, P), torch.ones(R, n, dtype=torch.bool, device="cuda"), inside], 1)
        for h in range(heads):
            kv = h * kv_heads // heads
            keys = torch.cat([pk[kv], kc[b, kv, :n], kt[b, kv]]).double()
            vals = torch.cat([pv[kv], vc[b, kv, :n], vt[b, kv]]).double()
            p = torch.softmax(((q[b, :, h].double() @ keys.T) / math.sqrt(hd)).masked_fill(~seen, -math.inf), -1)
            err = float((out[b, :, h] - p @ vals).abs().max())
            assert err < 1e-4, (b, n, h, err)                                        # the kernel tests' two-plane regression bound
