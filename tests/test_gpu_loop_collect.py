"""The native loop's collection of a step's results: one workgroup stores the
outputs, the error flag and then the done word that the host polls.  Batches on
both sides of the workgroup's 256 threads, ordinary and pinned host_out, direct
launches and graphs, and work on the stream that outlasts the poll."""
import numpy as np
import pytest
import torch

from paper_2406_11016_amd import binding
from paper_2406_11016_amd.decode_loop import next_gamma

pytestmark = pytest.mark.gpu

SENTINEL = -77


@pytest.mark.parametrize("pinned", [True, False])
@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("batch", [1, 255, 256, 257, 600])
def test_collected_results_are_the_steps_own(batch, graphs, pinned):
    gmax, V, steps = 3, 67, 24
    gen = torch.Generator().manual_seed(batch)
    dev = torch.device("cuda")
    draft = torch.empty(batch * gmax * V, device=dev)
    target = torch.empty(batch * (gmax + 1) * V, device=dev)
    tokens = torch.empty(batch * gmax, dtype=torch.int32, device=dev)
    uniforms = torch.empty(batch * (gmax + 1), device=dev)
    acc, nxt = (torch.empty(batch, dtype=torch.int32, device=dev) for _ in range(2))
    # host_out in the middle of an allocation, with guards on both sides
    host = torch.full((2 * batch + 14,), SENTINEL, dtype=torch.int32, pin_memory=pinned)
    need = max(binding.workspace_bytes(batch, g, V, torch.float32) for g in range(1, gmax + 1))
    ws = torch.zeros(need, dtype=torch.uint8, device=dev)
    stream = torch.cuda.Stream()
    desc = binding.LoopDesc(
        mode=0, dtype=binding.DTYPE_CODES[torch.float32], batch=batch, gamma_max=gmax, vocab=V, temperature=1.0,
        alpha=-1e3, beta=1e3, draft=draft.data_ptr(), target=target.data_ptr(), tokens=tokens.data_ptr(),
        uniforms=uniforms.data_ptr(), accepted_len=acc.data_ptr(), next_token=nxt.data_ptr(),
        host_out=host.data_ptr() + 7 * 4, workspace=ws.data_ptr(), workspace_bytes=ws.numel(),
        stream=stream.cuda_stream, use_graphs=int(graphs), early_exit=0)
    torch.cuda.synchronize()
    loop = binding.loop_create(desc)
    big = torch.empty(1 << 28, dtype=torch.uint8, device=dev)
    try:
        for i in range(steps):
            g = 1 + i % gmax
            d = torch.randn(batch, g, V, generator=gen)
            t = torch.randn(batch, g + 1, V, generator=gen) * 0.3
            t[:, :g] += d
            tok = torch.randint(V, (batch, g), generator=gen, dtype=torch.int32)
            u = torch.rand(batch, g + 1, generator=gen)
            with torch.cuda.stream(stream):
                draft[:d.numel()].copy_(d.flatten())
                target[:t.numel()].copy_(t.flatten())
                tokens[:tok.numel()].copy_(tok.flatten())
                uniforms[:u.numel()].copy_(u.flatten())
                if i % 4 == 3:  # several fills of 256 MiB: longer than the poll lasts
                    for _ in range(12):
                        big.fill_(i)
            got_gamma = binding.loop_step(loop, g)
            h = host.numpy().copy()
            want_l, want_n = binding.verify(d.to(dev), t.to(dev), tok.to(dev), u.to(dev), mode="exact")[:2]
            assert np.array_equal(h[7:7 + batch], want_l.cpu().numpy()), i
            assert np.array_equal(h[7 + batch:7 + 2 * batch], want_n.cpu().numpy()), i
            assert (h[:7] == SENTINEL).all() and (h[7 + 2 * batch:] == SENTINEL).all()
            assert got_gamma == next_gamma(g, h[7:7 + batch], gmax)
    finally:
        binding.loop_destroy(loop)
    torch.cuda.synchronize()
    assert not ws.any()
