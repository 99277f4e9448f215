"""GPU: distance of the decode outputs from the 64-bit values.  What rounding the
output to bf16 gives by itself is the bound, within a tenth, however a unit's
slots are cut: the probabilities of the value product carry more than 16 bits.
fp32 outputs: the rounding of the sums."""
import math

import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


def exact(q, k, v, K, V, lens, G):
    """Attention of q [B, Hq, d] over the first lens slots and the appended (k, v), in 64 bits."""
    import torch
    B, Hkv, cap, d = K.shape
    q64, out = q.double().reshape(B, Hkv, G, d).clone(), torch.empty((B, Hkv, G, d), dtype=torch.float64)
    q64[..., 0] = 0
    for b in range(B):
        for h in range(Hkv):
            n = int(lens[b, h])
            keys = torch.cat([K[b, h, :n], k[b, h][None]]).double()
            keys[:, 0] = 0
            p = torch.softmax(q64[b, h] @ keys.T / math.sqrt(d), -1)
            out[b, h] = p @ torch.cat([V[b, h, :n], v[b, h][None]]).double()
    return out.reshape(q.shape)


# one workgroup per unit, pieces of one unit, equal ranges (forced), whole units per wave
@pytest.mark.parametrize("B,Hkv,G,d,cap,split", [
    (4, 4, 8, 128, 500, 0), (4, 4, 4, 64, 900, 0), (3, 4, 8, 128, 2100, 0), (5, 4, 4, 64, 4200, 0),
    (3, 4, 4, 128, 2100, 300), (130, 8, 8, 128, 1100, 0), (4, 4, 2, 128, 900, 0),
])
def test_error_is_the_outputs_rounding(torch_cuda, B, Hkv, G, d, cap, split):
    import torch
    import paper_2403_09636_amd as P
    log(f"case decode precision B={B} Hkv={Hkv} G={G} d={d} cap={cap} split={split}")
    gen = torch.Generator().manual_seed(cap + G)

    def rnd(*shape):
        return torch.randn(shape, generator=gen).to(torch.bfloat16)

    K, V = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d)
    K[..., 0] = 0
    lens = torch.randint(cap // 2, cap, (B, Hkv), generator=gen, dtype=torch.int32)
    if B > 100:
        lens[:] = cap - 3
    q, k, v = rnd(B, Hkv * G, d), rnd(B, Hkv, d), rnd(B, Hkv, d)
    k[..., 0] = -4   # append
    cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, "bf16", max_slots_per_seq=cap, split_tile=split))
    cache.import_(0, K.cuda(), V.cuda(), lens.cuda(), torch.ones((B, Hkv), device="cuda"))
    got = cache.decode_step(0, q.cuda(), k.cuda(), v.cuda()).cpu().double()
    cache.check()
    rows = slice(0, 5)
    want = exact(q[rows], k[rows], v[rows], K[rows], V[rows], lens[rows], G)
    rounding = (want.to(torch.bfloat16).double() - want).norm()
    err = (got[rows] - want).norm()
    log(f"error {err / want.norm():.5f}, rounding alone {rounding / want.norm():.5f}")
    assert err <= 1.1 * rounding


def test_infinite_values_stay_infinite(torch_cuda):
    """An infinite value element makes its output element infinite (not NaN) in every
    query head that weighs its slot; the other elements stay finite."""
    import torch
    import paper_2403_09636_amd as P
    B, Hkv, G, d, cap = 2, 4, 8, 128, 700
    gen = torch.Generator().manual_seed(3)

    def rnd(*shape):
        return torch.randn(shape, generator=gen).to(torch.bfloat16)

    K, V = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d)
    V[0, 1, 7, 5], V[1, 2, 333, 127] = math.inf, -math.inf
    lens = torch.full((B, Hkv), cap - 2, dtype=torch.int32)
    for split in (0, 100):
        cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, "bf16", max_slots_per_seq=cap, split_tile=split))
        cache.import_(0, K.cuda(), V.cuda(), lens.cuda(), torch.ones((B, Hkv), device="cuda"))
        k = rnd(B, Hkv, d)
        k[..., 0] = -4
        out = cache.decode_step(0, rnd(B, Hkv * G, d).cuda(), k.cuda(), rnd(B, Hkv, d).cuda()).cpu().float()
        want = torch.zeros_like(out)
        want[0, G:2 * G, 5], want[1, 2 * G:3 * G, 127] = math.inf, -math.inf
        assert torch.equal(torch.where(out.isinf(), out, 0), want) and not out.isnan().any()


def test_vanished_probability_adds_nothing(torch_cuda):
    """A slot whose probability is 0 in 32 bits (a score thousands below the largest)
    adds nothing, however large its value."""
    import torch
    import paper_2403_09636_amd as P
    B, Hkv, G, d, cap = 2, 4, 8, 128, 700
    gen = torch.Generator().manual_seed(5)

    def rnd(*shape):
        return torch.randn(shape, generator=gen).to(torch.bfloat16)

    K, V, q, k, v = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d), rnd(B, Hkv * G, d), rnd(B, Hkv, d), rnd(B, Hkv, d)
    K[..., 0], k[..., 0] = 0, -4
    q[..., 1] = 200
    K[:, :, 9, 1], V[:, :, 9] = -200, 1e38
    lens = torch.full((B, Hkv), cap - 2, dtype=torch.int32)
    want = exact(q, k, v, K, V, lens, G)
    assert want.abs().max() < 100
    for split in (0, 100):
        cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, "bf16", max_slots_per_seq=cap, split_tile=split))
        cache.import_(0, K.cuda(), V.cuda(), lens.cuda(), torch.ones((B, Hkv), device="cuda"))
        out = cache.decode_step(0, q.cuda(), k.cuda(), v.cuda()).cpu().double()
        torch.testing.assert_close(out, want, rtol=1e-2, atol=2e-2)


# Equal ranges of short and of split units, one workgroup per unit.  Limits (in 2^-24, inputs and
# kernels repeat exactly): between what chunks summed by themselves give (2.43, 2.69, 2.65, 2.46)
# and chains over a whole piece (2.66, 2.88, 2.92, 2.76).
@pytest.mark.parametrize("B,Hkv,G,d,cap,slots,limit", [
    (60, 8, 1, 128, 200, 100, 2.55), (20, 8, 2, 128, 1200, 400, 2.8), (12, 4, 8, 128, 250, 240, 2.8),
    (8, 4, 1, 64, 500, 480, 2.6),
])
def test_fp32_error(torch_cuda, B, Hkv, G, d, cap, slots, limit):
    import torch
    import paper_2403_09636_amd as P
    log(f"case fp32 decode precision B={B} Hkv={Hkv} G={G} d={d} slots={slots}")
    gen = torch.Generator().manual_seed(cap + G)

    def rnd(*shape):
        return torch.randn(shape, generator=gen)

    K, V = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d)
    K[..., 0] = 0
    lens = torch.randint(slots // 2, slots, (B, Hkv), generator=gen, dtype=torch.int32)
    q, k, v = rnd(B, Hkv * G, d), rnd(B, Hkv, d), rnd(B, Hkv, d)
    k[..., 0] = -4   # append
    cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, "fp32", max_slots_per_seq=cap))
    cache.import_(0, K.cuda(), V.cuda(), lens.cuda(), torch.ones((B, Hkv), device="cuda"))
    got = cache.decode_step(0, q.cuda(), k.cuda(), v.cuda()).cpu().double()
    cache.check()
    want = exact(q, k, v, K, V, lens, G)
    err = float((got - want).norm() / want.norm()) * 2 ** 24
    log(f"error {err:.3f} x 2^-24")
    assert err <= limit
