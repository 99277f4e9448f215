"""GPU: the fp32 matrix-core attention kernels at the edges of their 32-row
blocks, against the oracles, and rows that are not finite (an infinity or NaN
reaches only the outputs that read it)."""
import numpy as np
import pytest

from tests.gpu_helpers import log
from tests.test_gpu_train import test_train_forward_backward as check_train

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G,B,Hkv,n,w", [
    (64, 1, 1, 1, 31, 5), (64, 1, 1, 2, 32, 5), (128, 1, 1, 1, 33, 5),
    (128, 8, 1, 1, 129, 12), (64, 4, 2, 1, 161, 31), (128, 2, 1, 1, 193, 12),
])
def test_train_blocks(torch_cuda, d, G, B, Hkv, n, w):
    check_train(torch_cuda, ("fp32", d, G, B, Hkv, n, w, 5.0, 0.1, [3.0, 1.0][:Hkv], "lead", True))


@pytest.mark.parametrize("d,G", [(64, 1), (128, 4)])
def test_train_nonfinite_rows(torch_cuda, d, G):
    import torch
    import paper_2403_09636_amd as P
    log(f"case nonfinite d={d} G={G}")
    n, w, s, r = 77, 4, 40, 20
    gen = torch.Generator().manual_seed(7 + d)
    q, k, v, dout = (torch.randn((1, n, h, d), generator=gen).cuda() for h in (G, 1, 1, G))
    noise = torch.zeros((1, n, 1), device="cuda")
    tr = P.DMCTrainer(P.make_train_config(1, n, G, 1, d, "fp32", decision_bias=0.0, temperature=1.0,
                                          window=w))

    def run(v, dout):
        out = tr.forward(q, k, v, noise)
        return (out, *tr.backward(q, k, v, noise, out, dout))

    ref = run(v, dout)
    bad_v = v.clone()
    bad_v[0, s, 0, 5] = float("inf")
    out, dq, _, _ = run(bad_v, dout)
    # queries before token s do not read it (rounding may differ: another path); dq[0] comes
    # through omega from the states' gradients, which every later query feeds
    for got, want in ((out, ref[0]), (dq[..., 1:], ref[1][..., 1:])):
        assert torch.isfinite(got[0, :s]).all()
        torch.testing.assert_close(got[0, :s], want[0, :s], rtol=1e-4, atol=1e-5)
    assert not torch.isfinite(out[0, s]).all()
    bad_do = dout.clone()
    bad_do[0, r, 0, 3] = float("nan")
    _, _, dk, dv = run(v, bad_do)
    # states (and tokens) after row r do not feed it; dk[0] of token r + 1 holds state r's mask
    # gradient, so the decision neuron is left out
    for got, want in ((dk[..., 1:], ref[2][..., 1:]), (dv, ref[3])):
        assert torch.isfinite(got[0, r + 1:]).all()
        torch.testing.assert_close(got[0, r + 1:], want[0, r + 1:], rtol=1e-4, atol=1e-4)
    assert torch.isnan(dv[0, r]).any()


@pytest.mark.parametrize("d,G", [(64, 1), (128, 4)])
def test_train_infinite_last_row(torch_cuda, d, G):
    """An infinite gradient element of the last token reaches every token's dV as an
    infinity: the last block's padding (n G no multiple of 32) adds nothing."""
    import torch
    import paper_2403_09636_amd as P
    log(f"case infinite last row d={d} G={G}")
    n, w = 109, 4
    gen = torch.Generator().manual_seed(17 + d)
    q, k, v, dout = (torch.randn((1, n, h, d), generator=gen).cuda() for h in (G, 1, 1, G))
    dout[0, n - 1, 0, 3], dout[0, n - 1, G - 1, 6] = float("inf"), -float("inf")
    noise = torch.zeros((1, n, 1), device="cuda")
    tr = P.DMCTrainer(P.make_train_config(1, n, G, 1, d, "fp32", decision_bias=0.0, temperature=1.0,
                                          window=w))
    out = tr.forward(q, k, v, noise)
    dv = tr.backward(q, k, v, noise, out, dout)[2][0, :, 0]
    assert (dv[:, 3] == float("inf")).all() and (dv[:, 6] == -float("inf")).all()
    rest = [e for e in range(d) if e not in (3, 6)]
    assert torch.isfinite(dv[:, rest]).all()


@pytest.mark.parametrize("d,G,w", [(64, 2, 0), (128, 1, 0), (128, 4, 5)])
def test_prompt_nonfinite_rows(torch_cuda, d, G, w):
    import torch
    import paper_2403_09636_amd as P
    log(f"case prompt nonfinite d={d} G={G} w={w}")
    n, s, Hkv = 150, 83, 2
    gen = torch.Generator().manual_seed(d + G)
    q, k, v = (torch.randn((1, n, h, d), generator=gen).cuda() for h in (G * Hkv, Hkv, Hkv))
    cache = P.DMCCache(P.make_config(1, 1, G * Hkv, Hkv, d, "fp32", page_size=16, max_slots_per_seq=n,
                                     window=w))

    def run(v):
        cache.reset()
        return cache.prefill_attend(0, k, v, q)

    ref = run(v)
    bad = v.clone()
    bad[0, s, :, 5] = float("nan")
    bad[0, s + 1, :, 7] = float("inf")
    out = run(bad)
    # tokens before s do not read row s (rounding may differ: another path)
    assert torch.isfinite(out[0, :s]).all()
    torch.testing.assert_close(out[0, :s], ref[0, :s], rtol=1e-4, atol=1e-5)
    assert torch.isnan(out[0, s:, :, 5]).all()


def _low_scores(d, Hq, Hkv, n, size):
    """Every score of every query is -size^2 / sqrt(d), and the softmax uniform (size a power
    of two: scaled scores are exact, where a rounding of 2^80 would decide the softmax)."""
    import torch
    q, k = torch.zeros((1, n, Hq, d)), torch.zeros((1, n, Hkv, d))
    q[..., 1], k[..., 1], k[..., 0] = size, -size, -9.0   # (every token opens a slot)
    v = torch.randn((1, n, Hkv, d), generator=torch.Generator().manual_seed(d))
    mean = v.double().cumsum(1) / torch.arange(1, n + 1)[None, :, None, None]
    return q.cuda(), k.cuda(), v.cuda(), mean.repeat_interleave(Hq // Hkv, 2)


@pytest.mark.parametrize("d,G,w", [(64, 1, 0), (128, 4, 0), (64, 8, 5)])
def test_prompt_lowest_scores(torch_cuda, d, G, w):
    """Scores far below -1e30 still make a softmax; one of -infinity by itself is the token's own."""
    import torch
    import paper_2403_09636_amd as P
    log(f"case prompt lowest scores d={d} G={G} w={w}")
    n = 150
    cache = P.DMCCache(P.make_config(1, 1, 2 * G, 2, d, "fp32", max_slots_per_seq=n, omega_src="uniform",
                                     window=w))
    for size, upto in ((2.0 ** 57, n), (2.0 ** 83, 1)):
        q, k, v, mean = _low_scores(d, 2 * G, 2, n, size)
        cache.reset()
        out = cache.prefill_attend(0, k, v, q).cpu().double()
        torch.testing.assert_close(out[:, :upto], mean[:, :upto], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("d,G", [(64, 1), (128, 4), (64, 8)])
def test_train_lowest_scores(torch_cuda, d, G):
    import torch
    import paper_2403_09636_amd as P
    log(f"case train lowest scores d={d} G={G}")
    n = 109
    q, k, v, mean = _low_scores(d, 2 * G, 2, n, 2.0 ** 57)
    tr = P.DMCTrainer(P.make_train_config(1, n, 2 * G, 2, d, "fp32", decision_bias=0.0, temperature=1.0,
                                          window=1, omega_src="uniform"))
    out = tr.forward(q, k, v, torch.zeros((1, n, 2), device="cuda")).cpu().double()
    # (the mask entries are lost in scores of this size)
    torch.testing.assert_close(out, mean, rtol=1e-5, atol=1e-5)
