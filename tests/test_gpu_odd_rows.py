"""16-bit rows of odd length start off a 4-byte boundary every other row, rows of
even length in a tensor that starts at an odd element all do, and both are read
with 128-bit loads all the same, in every role that reads rows.

Expected values: the oracle's decisions (bit for bit outside its flagged
cases), and for a tensor moved by one element the outputs and probes of the
tensor that was not, bit for bit.  The rows of an odd-V batch alternate between the two alignments, so a
target row equal to the draft row on the other alignment must still give tau =
1 exactly (the element assignment does not depend on the address)."""
import numpy as np
import pytest
import torch

from paper_2406_11016_amd import binding
from paper_2406_11016_amd import workloads as W
from tests.gpu_util import run_gpu, run_oracle
from tests.test_gpu_early_exit import _check, _gate

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    binding.load_library()
    torch.cuda.init()


# (B, gamma, V): rows shorter than a vector and just past one, one vector per
# lane, the ends of the short streams' chunks, and a long stream with whole
# and partial last vectors
SHAPES = [(3, 2, 7), (3, 2, 9), (2, 3, 511), (2, 3, 2049), (5, 3, 8193), (4, 5, 51865), (40, 6, 65537)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,gamma,V", SHAPES, ids=[f"B{s[0]}-g{s[1]}-V{s[2]}" for s in SHAPES])
def test_odd_rows_match_the_oracle(B, gamma, V, dtype):
    x = W.small_case(B, gamma, V, dtype, seed=700 + V, noise_scale=0.5)
    n = min(B, 6)
    sub = W.Inputs(x.draft[:n], x.target[:n], x.tokens[:n], x.uniforms[:n], x.dtype, x.mode, x.temperature, x.alpha,
                   x.beta)
    for mode in ("exact", "sigmoid"):
        x.mode = sub.mode = mode
        acc, nxt = run_gpu(x, probe=False)
        o = run_oracle(sub)
        ok = ~o.flagged(1e-6)
        assert np.array_equal(acc[:n][ok], o.accepted_len[ok]), (mode, acc[:n], o.accepted_len)
        assert np.array_equal(nxt[:n][ok], o.next_token[ok]), (mode, nxt[:n], o.next_token)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_equal_rows_on_both_alignments_accept_every_draft(dtype):
    x = W.small_case(7, 4, 20011, dtype, seed=5)
    x.draft[:] = x.target[:, :4]
    x.uniforms[:, :4] = W.UNIFORM_MAX
    acc, _ = run_gpu(x, probe=False)
    assert np.all(acc == 4), acc


@pytest.mark.parametrize("gamma,batch,vocab,dtype", [(5, 28, 128257, "bf16"), (33, 10, 50001, "f16")])
@pytest.mark.parametrize("noise", [0.05, 1.0])
def test_odd_rows_in_the_gated_stages(gamma, batch, vocab, dtype, noise):
    # rows of several chunks of the early exit, which runs its staged kernel here
    assert _gate(batch, vocab, dtype) < gamma
    x = W.small_case(batch, gamma, vocab, dtype, seed=40 + gamma, noise_scale=noise)
    _check(x, f"odd rows noise={noise}", oracle_sample=4, seed=gamma)


def _from_element_1(t):
    flat = torch.empty(t.numel() + 2, dtype=t.dtype, device=t.device)
    flat[0] = flat[-1] = float("nan")
    moved = flat[1:-1].view(t.shape)
    moved.copy_(t)
    assert moved.data_ptr() % 4 == 2
    return moved


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,gamma,V", [(3, 2, 8), (2, 3, 2050), (3, 2, 9), (5, 3, 8193), (28, 5, 128256), (4, 5, 51865)])
def test_tensors_that_start_at_an_odd_element(B, gamma, V, dtype):
    x = W.small_case(B, gamma, V, dtype, seed=900 + V, noise_scale=0.5, alpha=-1e3, beta=1e3)
    d, t, tok, u = binding.to_device(x, "cuda")
    md, mt = _from_element_1(d), _from_element_1(t)
    gammas = torch.arange(B, dtype=torch.int32, device="cuda") % gamma + 1
    for kw in (dict(mode="exact", probe=True), dict(mode="sigmoid", probe=True, alpha=x.alpha, beta=x.beta),
               dict(mode="exact"), dict(mode="sigmoid", alpha=x.alpha, beta=x.beta),
               dict(mode="exact", gammas=gammas), dict(mode="exact", early_exit=True)):
        want, got = binding.verify(d, t, tok, u, **kw), binding.verify(md, mt, tok, u, **kw)
        assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1]), kw
        if len(want) > 2:
            for name in ("tau", "weights", "mass", "lognorm"):
                a, b = getattr(want[2], name), getattr(got[2], name)
                assert a is None or torch.equal(a.nan_to_num(nan=-1.0), b.nan_to_num(nan=-1.0)), (kw, name)
    n = min(B, 4)
    sub = W.Inputs(x.draft[:n], x.target[:n], x.tokens[:n], x.uniforms[:n], x.dtype, "exact", x.temperature, x.alpha,
                   x.beta)
    o = run_oracle(sub)
    ok = ~o.flagged(1e-6)
    acc, nxt = (r[:n].cpu().numpy() for r in binding.verify(md, mt, tok, u))
    assert np.array_equal(acc[ok], o.accepted_len[ok]) and np.array_equal(nxt[ok], o.next_token[ok])
