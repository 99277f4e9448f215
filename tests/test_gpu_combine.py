"""GPU: the split-K combine at its batch edges: units cut into 1 .. 70 pieces by
forced split sizes, few heads (a workgroup per head) and many (a wave each),
against the same layer with another split."""
import pytest

from tests.gpu_helpers import TOL, log, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,Hkv,G,d", [
    ("fp32", 2, 4, 1, 64), ("bf16", 3, 4, 2, 128), ("bf16", 2, 3, 8, 128), ("fp32", 300, 2, 2, 64),
])
def test_combine_piece_counts(torch_cuda, dtype, B, Hkv, G, d):
    import torch
    import paper_2403_09636_amd as P
    log(f"case combine {dtype} B={B} Hkv={Hkv} G={G} d={d}")
    cap, dt = 1120, torch_dtype(dtype)
    gen = torch.Generator(device="cuda").manual_seed(B)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(dt)

    K, V = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d)
    K[..., 0] = 0
    base = [cap - 2, 15, 40, 80, 130, 250, 260, 300, 500, 1030]
    lens = torch.tensor([base[i % len(base)] for i in range(B * Hkv)], dtype=torch.int32).reshape(B, Hkv).cuda()
    z = torch.ones((B, Hkv), device="cuda")
    q, k, v = rnd(B, Hkv * G, d), rnd(B, Hkv, d), rnd(B, Hkv, d)
    outs = []
    for split in (16, 32, 64, 300, 1 << 20):   # up to 70 pieces per unit .. the equal shares
        cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, dtype, max_slots_per_seq=cap,
                                         split_tile=split))
        cache.import_(0, K, V, lens, z)
        outs.append(cache.decode_step(0, q, k, v).float())
        cache.check()
    atol, rtol = TOL[dtype]
    for o in outs[1:]:
        torch.testing.assert_close(o, outs[0], rtol=rtol, atol=atol)
