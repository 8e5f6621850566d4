"""Tree attention (GPU) of several sequences of unequal lengths with grouped heads and more workgroups than the CUs hold at
once: a sequence's output does not depend on its place in the batch or on the others' lengths."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("rows,lens", [(130, [40, 300]), (130, [77, 77]), (90, [5, 0, 400]), (70, [64, 64, 63, 65]), (41, [31, 500, 0, 500, 32, 33, 1]),
                                       (33, [1, 2, 3, 4, 5, 6, 7, 300]), (33, [300] * 8), (33, [9, 200, 8, 200, 7, 100, 200, 0])])
def test_a_sequence_in_any_place_of_the_batch(rows, lens, hd):
    import paper_2401_12522_amd as bita
    heads, kv_heads, B, smax, P = 64, 8, len(lens), max(lens) + 1, 5
    tin = synth.attach_mask_groups(synth.random_tree(rows, 4, rows), [0], 4)
    R = tin.rows
    plan = bita.binding.attention_plan_info(B, R, heads, kv_heads, hd, max(lens), P)
    assert plan["workgroups"] > 512 and plan["waves"] == 4 and plan["heads"] > 1, plan
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, 4)
    g = torch.Generator(device="cuda").manual_seed(rows + hd)
    b16 = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    q, kt, vt = b16(B, R, heads, hd), b16(B, kv_heads, R, hd), b16(B, kv_heads, R, hd)
    kc, vc, pk, pv = b16(B, kv_heads, smax, hd), b16(B, kv_heads, smax, hd), b16(kv_heads, P, hd), b16(kv_heads, P, hd)
    lens = torch.tensor(lens, dtype=torch.int32, device="cuda")

    def planes(at, hint):
        take = lambda t: t[at].contiguous()                                           # noqa: E731
        hi, lo = bita.tree_attention(tmpl, take(q), take(kc), take(vc), take(kt), take(vt), pk, pv, take(lens), hint, two_plane_out=True)
        return hi, lo
    here = planes(torch.arange(B), int(lens.max()))
    for perm in (torch.arange(B).flip(0), torch.tensor(np.random.default_rng(B).permutation(B))):
        there = planes(perm, int(lens.max()))
        for a, b in zip(here, there):
            assert torch.equal(a[perm], b)
    for b in range(B):                                   # and is what the sequence alone gives (other waves, other order of sums)
        hi, lo = planes(torch.tensor([b]), int(lens.max()))
        err = (here[0][b].double() + here[1][b].double() - hi[0].double() - lo[0].double()).abs().max()
        assert float(err) < 1e-4, (b, float(err))        # the kernel tests' two-plane regression bound
