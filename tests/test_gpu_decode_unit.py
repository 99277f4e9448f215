"""GPU: decode of short caches (one workgroup per unit) against the general
path (a slot-space split, chosen by a split_tile no range reaches) at unit
lengths around the chunk and page edges and at the slot capacity."""
import pytest

from tests.gpu_helpers import TOL, log, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,G,page,cap", [
    ("fp32", 64, 1, 32, 260), ("fp32", 128, 8, 8, 130), ("bf16", 128, 1, 32, 512),
    ("bf16", 64, 2, 16, 300), ("bf16", 128, 8, 32, 259), ("bf16", 64, 4, 32, 1024),
    ("bf16", 128, 4, 64, 200),
    ("bf16", 128, 8, 32, 1000), ("bf16", 128, 4, 32, 1024),   # (80 units: the wider limit)
    ("bf16", 128, 4, 16, 256), ("bf16", 64, 8, 64, 768),      # (vector ALUs at their limits)
])
def test_unit_decode_matches_general(torch_cuda, dtype, d, G, page, cap):
    import torch
    import paper_2403_09636_amd as P
    log(f"case unit decode {dtype} d={d} G={G} page={page} cap={cap}")
    dt, Hkv = torch_dtype(dtype), 4
    lens = [0, 1, 2, 16, 17, 18, 31, 32, 33, 34, 64, 65, 66, 100, 127, 128, 129, cap - 2, cap - 1, cap]
    lens = [x for x in lens if x <= cap]
    lens += [cap // 2] * (-len(lens) % Hkv)
    lens *= 4 if cap * d > 1 << 16 else 1
    B = len(lens) // Hkv
    gen = torch.Generator().manual_seed(cap)

    def rnd(*shape):
        return torch.randn(shape, generator=gen).to(dt).cuda()

    K, V = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d)
    K[..., 0] = 0
    ln = torch.tensor(lens, dtype=torch.int32).reshape(B, Hkv).cuda()
    z = torch.rand((B, Hkv), generator=gen).cuda() + 0.5
    steps = [(rnd(B, Hkv * G, d), rnd(B, Hkv, d), rnd(B, Hkv, d)) for _ in range(3)]
    got = []
    for split in (0, 1 << 20):
        cache = P.DMCCache(P.make_config(1, B, Hkv * G, Hkv, d, dtype, page_size=page,
                                         max_slots_per_seq=cap, split_tile=split,
                                         num_pages=2 * B * Hkv * -(-cap // page)))
        cache.import_(0, K, V, ln, z)
        outs = []
        for q, k, v in steps:
            slot = torch.empty((B, Hkv), dtype=torch.int32, device="cuda")
            outs.append((cache.decode_step(0, q, k, v, slot_index=slot), slot, cache.lengths(0)))
        got.append((outs, cache.export(0), cache.status()))
    atol, rtol = TOL[dtype]
    full = any((slot < 0).any() for _, slot, _ in got[0][0])   # a full unit dropped a token
    for (a, sa, la), (b, sb, lb) in zip(got[0][0], got[1][0]):
        assert (sa == sb).all() and (la == lb).all()
        keep = (sa >= 0).repeat_interleave(G, 1)   # (outputs of a dropped token are undefined)
        torch.testing.assert_close(a.float()[keep], b.float()[keep], rtol=rtol, atol=atol)
    for a, b in zip(got[0][1], got[1][1]):
        assert torch.equal(a, b)
    assert got[0][2] == got[1][2] and (got[0][2] == P.binding.DMC_ERR_CAPACITY) == bool(full)
