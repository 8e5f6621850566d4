"""Tree attention (GPU) over a sequence that goes on past slot 2^23, where the kernel changes from buffer
descriptors, whose offsets have 32 bits, to 64-bit addresses.  The keys on both sides of that slot carry
the softmax, so that a chunk lost or read from elsewhere shows."""
import math

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,hd,n", [(1, 64, (1 << 23) + 77), (2, 64, (1 << 23) + 77), (1, 128, (1 << 23) + 77), (2, 128, 1 << 23)])
def test_slots_on_both_sides_of_two_to_the_23(heads, hd, n):
    import paper_2401_12522_amd as bita
    P, tin = 8, synth.attach_mask_groups(synth.star_tree(3), [0], 4)
    R = tin.rows
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, 4)
    g = torch.Generator(device="cuda").manual_seed(heads * hd)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    q, kc, vc, kt, vt, pk, pv = rnd(1, R, heads, hd), rnd(1, 1, n, hd), rnd(1, 1, n, hd), rnd(1, 1, R, hd), rnd(1, 1, R, hd), rnd(1, P, hd), rnd(1, P, hd)
    kc[:, :, (1 << 23) - 64:] *= 12                      # scores of deviation 12: e^25 and more against 2^23 keys of e^0.5
    hi, lo = bita.tree_attention(tmpl, q, kc, vc, kt, vt, pk, pv, torch.tensor([n], dtype=torch.int32, device="cuda"), n, two_plane_out=True)
    out = hi.double().view(R, heads, hd) + lo.double().view(R, heads, hd)
    inside = np.zeros((R, R), bool)
    for i, p in enumerate(tin.parent):
        if p >= 0:
            inside[i] = inside[p]
        inside[i, i] = True
    masks = torch.tensor(tin.is_mask.astype(bool), device="cuda")
    seen = torch.cat([masks[:, None].expand(R, P), torch.ones(R, n, dtype=torch.bool, device="cuda"), torch.tensor(inside, device="cuda")], 1)
    keys, vals = torch.cat([pk[0], kc[0, 0], kt[0, 0]]).double(), torch.cat([pv[0], vc[0, 0], vt[0, 0]]).double()
    for h in range(heads):
        p = torch.softmax(((q[0, :, h].double() @ keys.T) / math.sqrt(hd)).masked_fill(~seen, -math.inf), -1)
        assert float(p[:, P + (1 << 23) - 64:].sum(-1).min()) > 0.5
        err = float((out[:, h] - p @ vals).abs().max())
        assert err < 1e-4, (h, err)                      # the kernel tests' two-plane regression bound
