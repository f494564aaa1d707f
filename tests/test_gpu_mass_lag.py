"""Batches on both sides of the distance at which the residual workgroups of an
element follow its statistics: all of them after the stream, the last element
alone among it, and several.  The ragged call, with numbers of drafts of every
kind, all of them full, and at most one, agrees with the oracle and with the
plain calls on each element's own drafts, element by element (same rows, so the
same decisions but for roundings that no uniform of these seeds lies near)."""
import os
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2406_11016_amd import binding, build

pytestmark = pytest.mark.gpu

V = 131073                           # an odd row of 512 KiB + 4 B


def lag(gamma):
    """The distance in elements (plan.hpp): a fixed number of bytes of stream, 2 gamma rows an element."""
    with open(os.path.join(build.CSRC, "plan.hpp")) as f:
        nbytes = int(re.search(r"kLagStreamBytes = (\d+);", f.read()).group(1))
    return -(-nbytes // (2 * gamma * V * 4))


@pytest.mark.parametrize("gamma,full,beyond", [(7, False, -1), (7, False, 0), (7, False, 1), (7, False, 10),
                                               (7, True, 1), (1, True, 0), (1, True, 1)])
def test_ragged_batches_around_the_lag(gamma, full, beyond):
    batch = lag(gamma) + beyond
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(batch)
    draft = torch.randn(batch, gamma, V, generator=gen, device=dev) * 2
    target = torch.randn(batch, gamma + 1, V, generator=gen, device=dev)
    target[:, :gamma] += draft
    tokens = torch.randint(V, (batch, gamma), generator=gen, device=dev, dtype=torch.int32)
    likely = (draft + torch.randn(draft.shape, generator=gen, device=dev)).argmax(-1).int()
    if gamma > 1:
        tokens[:, ::2] = likely[:, ::2]
    else:
        tokens[::2] = likely[::2]
    uniforms = torch.rand(batch, gamma + 1, generator=gen, device=dev) * 0.999
    if full:
        gammas = torch.full((batch,), gamma, dtype=torch.int32, device=dev)
    else:
        gammas = torch.randint(1, gamma + 1, (batch,), generator=gen, device=dev, dtype=torch.int32)
    gammas[3] = 0                    # out of range: a sentinel
    gammas[batch - 2] = gamma + 1
    ws = binding.new_workspace(batch, gamma, V, torch.float32, dev)
    acc, nxt = binding.verify(draft, target, tokens, uniforms, gammas=gammas, workspace=ws)
    again = binding.verify(draft, target, tokens, uniforms, gammas=gammas, workspace=ws)
    assert not ws.any() and torch.equal(acc, again[0]) and torch.equal(nxt, again[1])
    want_l, want_n = torch.full_like(acc, -1), torch.full_like(nxt, -1)
    for g in range(1, gamma + 1):
        own = (gammas == g).nonzero().flatten()
        if own.numel():
            l, n = binding.verify(draft[own, :g].contiguous(), target[own, :g + 1].contiguous(),
                                  tokens[own, :g].contiguous(), uniforms[own, :g + 1].contiguous())
            want_l[own], want_n[own] = l, n
    assert np.array_equal(acc.cpu().numpy(), want_l.cpu().numpy())
    assert np.array_equal(nxt.cpu().numpy(), want_n.cpu().numpy())
    assert (want_l < gammas).any() and (want_l >= 0).sum() == batch - 2
    # the oracle on the elements around the lag and at the ends
    some = sorted({0, 1, 2, 3, 4, lag(gamma) - 2, batch - 2, batch - 1})
    with np.errstate(all="ignore"):
        o = oracle.verify_ragged(*(t[some].cpu().numpy() for t in (draft, target, tokens, uniforms, gammas)), dtype="f32")
    ok = ~o.flagged(1e-6)
    assert ok.sum() >= len(some) - 1
    assert np.array_equal(acc.cpu().numpy()[some][ok], o.accepted_len[ok])
    assert np.array_equal(nxt.cpu().numpy()[some][ok], o.next_token[ok])
