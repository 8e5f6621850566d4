"""Vocabulary selection (GPU) where the k winners of a row come from one thread or one wave, where
rows fit the registers exactly, by one more, or not at all, and where most values are equal."""
import numpy as np
import pytest
import torch

import synth
from oracle.model import argmax_low, topk_desc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,kmax", [(16, 16), (1024, 5), (4096, 64), (32000, 4), (32768, 64), (32784, 64), (70000, 7)])
def test_select_matches_the_oracle_exactly(vocab, kmax):
    import paper_2401_12522_amd as bita
    rng = np.random.default_rng(vocab + kmax)
    tin = synth.attach_mask_groups(synth.star_tree(3), [0], 4)
    tmpl = bita.TreeTemplate(tin.parent, tin.is_mask, tin.n_tree, 4)
    x = rng.normal(size=(2, tmpl.rows, vocab)).astype(np.float32)
    x[0, 0] = rng.integers(0, 3, size=vocab)                     # ties everywhere
    x[0, 1] = -0.0
    x[0, 3] = rng.integers(-1, 1, size=vocab)
    x[0, 4, 4 * 7 % vocab::4096] += 50.0                         # the entries of one thread's share win
    x[0, 5, : min(vocab, 256)] += 50.0                           # ... of one wave's
    x[0, 6, -16:] = np.float32(3e38)                             # ... the row's end
    x[1, 2] = -3e38
    x[1, 3] = -np.arange(vocab)
    am, ids, val = (v.cpu().numpy() for v in bita.select(tmpl, torch.tensor(x, device="cuda"), kmax))
    for b in range(2):
        for r in range(tin.n_tree):
            assert am[b, r] == argmax_low(x[b, r])
        for m in range(4):
            want, want_val = topk_desc(x[b, tin.n_tree + m] + np.float32(0), kmax)
            assert ids[b, m].tolist() == want.tolist(), (b, m)
            assert val[b, m].tolist() == want_val.tolist(), (b, m)
