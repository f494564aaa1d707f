"""The weights and mass probes of a bonus draw, written by the whole workgroup
with 16-byte loads: rows shorter than a vector, partial vectors, rows that start
off a 16- and a 4-byte boundary, and rows of several passes."""
import pytest
import torch

from paper_2406_11016_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16], ids=["f32", "f16", "bf16"])
@pytest.mark.parametrize("vocab", [1, 3, 9, 257, 2049, 8191, 51865, 131077])
@pytest.mark.parametrize("mode", ["exact", "sigmoid"])
def test_bonus_weights(mode, vocab, dtype):
    B, g = 3, 2
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(vocab)
    target = (torch.randn(B, g + 1, vocab, generator=gen, device=dev) * 2).clamp_(-8, 8).to(dtype)
    draft = target[:, :g].clone()
    tokens = torch.randint(vocab, (B, g), generator=gen, device=dev, dtype=torch.int32)
    uniforms = torch.zeros(B, g + 1, device=dev)          # r = 0: every draft is accepted
    uniforms[:, g] = torch.rand(B, generator=gen, device=dev) * 0.999
    acc, nxt, pr = binding.verify(draft, target, tokens, uniforms, mode=mode, alpha=-20.0, beta=20.0, probe=True)
    assert (acc == g).all() and (nxt >= 0).all() and (nxt < vocab).all()
    z = target[:, g].double()
    want = torch.softmax(z, -1) if mode == "exact" else torch.sigmoid((z + 20.0) / 40.0)
    got = pr.weights.double()
    # fp32 weights.  Exact: 2^(z c - K) and its scale, |z c| <= 12 and |log2 sum| <= 29, each argument
    # rounded at 2^-24 of its size, so (12 + 29) 2^-24 ln 2 = 1.7e-6 relative, and a few roundings of the
    # result.  Sigmoid: arguments within (0.3, 0.7), a few roundings.
    assert torch.allclose(got, want, rtol=2.5e-6, atol=0.0), ((got - want).abs() / want).max()
    total = want.sum(-1)
    assert torch.allclose(pr.mass, total, rtol=2.5e-6, atol=0.0)
