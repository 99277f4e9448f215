"""GPU: matrix-core decode with whole-chunk pieces of one unit per wave (layers
with fewer units than waves) against the equal slot ranges (a split_tile no
range reaches): uniform and uneven lengths, chunk edges, empty units, windows."""
import pytest

from tests.gpu_helpers import TOL, log

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 128, 700, 1023, 1024, 1025, 1500, 2046, 2047, 2048]


@pytest.mark.parametrize("B,Hkv,G,d,window,lens", [
    (5, 4, 8, 128, 0, EDGES), (5, 4, 4, 64, 0, EDGES), (3, 8, 4, 128, 0, [2040, 2041, 2047, 2048]),
    (64, 8, 8, 128, 0, [2000, 2010, 2020, 1990]), (40, 8, 4, 64, 0, [600, 640, 2000, 100]),
    (3, 4, 4, 128, 12, None), (26, 4, 8, 64, 5, None),
])
def test_pieces_match_ranges(torch_cuda, B, Hkv, G, d, window, lens):
    import torch
    import paper_2403_09636_amd as P
    log(f"case pieces B={B} Hkv={Hkv} G={G} d={d} w={window}")
    cap = 2052
    gen = torch.Generator(device="cuda").manual_seed(B + d)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)

    U = B * Hkv
    K, V = rnd(B, Hkv, 2048, d), rnd(B, Hkv, 2048, d)
    K[..., 0] = 0
    if lens:
        ln = torch.tensor([lens[i % len(lens)] for i in range(U)], dtype=torch.int32).reshape(B, Hkv).cuda()
    steps = [(rnd(B, Hkv * G, d), rnd(B, Hkv, d), rnd(B, Hkv, d)) for _ in range(3)]
    got = []
    for split in (0, 1 << 20):
        cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, "bf16", max_slots_per_seq=cap,
                                         split_tile=split, window=window))
        if lens:
            cache.import_(0, K, V, ln, torch.ones((B, Hkv), device="cuda"))
        else:   # a windowed cache comes from a prompt
            kp = K[:, :, :1500].transpose(1, 2).contiguous()
            kp[..., 0] = V[:, :, :1500, 0].transpose(1, 2)   # decisions
            cache.prefill(0, kp, V[:, :, :1500].transpose(1, 2).contiguous(), steps[0][0][:, None, :, 0]
                          .expand(B, 1500, Hkv * G).contiguous())
        outs = []
        for q, k, v in steps:
            slot = torch.empty((B, Hkv), dtype=torch.int32, device="cuda")
            outs.append((cache.decode_step(0, q, k, v, slot_index=slot), slot, cache.lengths(0)))
        cache.check()
        got.append((outs, cache.export(0)))
    atol, rtol = TOL["bf16"]
    for (a, sa, la), (b, sb, lb) in zip(got[0][0], got[1][0]):
        assert (sa == sb).all() and (la == lb).all()
        torch.testing.assert_close(a.float(), b.float(), rtol=rtol, atol=atol)
    for a, b in zip(got[0][1], got[1][1]):
        assert torch.equal(a, b)
