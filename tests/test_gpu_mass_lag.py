"""Batches on both sides of the distance at which the residual workgroups of an
element follow its statistics: all of them after the stream, the last element
alone among it, and several.  The ragged call agrees with the plain calls on
each element's own drafts, element by element (same rows, so the same decisions
but for roundings that no uniform of these seeds lies near)."""
import numpy as np
import pytest
import torch

from paper_2406_11016_amd import binding

pytestmark = pytest.mark.gpu

GAMMA, V = 7, 131073                 # an odd row of 512 KiB + 4 B; a ragged unit counts as gamma + 1 rows
LAG = -(-42_000_000 // ((GAMMA + 1) * V * 4))


@pytest.mark.parametrize("batch", [LAG - 1, LAG, LAG + 1, LAG + 10])
def test_ragged_batches_around_the_lag(batch):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(batch)
    draft = torch.randn(batch, GAMMA, V, generator=gen, device=dev) * 2
    target = torch.randn(batch, GAMMA + 1, V, generator=gen, device=dev)
    target[:, :GAMMA] += draft
    tokens = torch.randint(V, (batch, GAMMA), generator=gen, device=dev, dtype=torch.int32)
    tokens[:, ::2] = (draft + torch.randn(draft.shape, generator=gen, device=dev)).argmax(-1).int()[:, ::2]
    uniforms = torch.rand(batch, GAMMA + 1, generator=gen, device=dev) * 0.999
    gammas = torch.randint(1, GAMMA + 1, (batch,), generator=gen, device=dev, dtype=torch.int32)
    gammas[3] = 0                    # out of range: a sentinel
    gammas[batch - 2] = GAMMA + 1
    ws = binding.new_workspace(batch, GAMMA, V, torch.float32, dev)
    acc, nxt = binding.verify(draft, target, tokens, uniforms, gammas=gammas, workspace=ws)
    again = binding.verify(draft, target, tokens, uniforms, gammas=gammas, workspace=ws)
    assert not ws.any() and torch.equal(acc, again[0]) and torch.equal(nxt, again[1])
    want_l, want_n = torch.full_like(acc, -1), torch.full_like(nxt, -1)
    for g in range(1, GAMMA + 1):
        own = (gammas == g).nonzero().flatten()
        if own.numel():
            l, n = binding.verify(draft[own, :g].contiguous(), target[own, :g + 1].contiguous(),
                                  tokens[own, :g].contiguous(), uniforms[own, :g + 1].contiguous())
            want_l[own], want_n[own] = l, n
    assert np.array_equal(acc.cpu().numpy(), want_l.cpu().numpy())
    assert np.array_equal(nxt.cpu().numpy(), want_n.cpu().numpy())
    assert (want_l < gammas).any() and (want_l >= 0).sum() == batch - 2
