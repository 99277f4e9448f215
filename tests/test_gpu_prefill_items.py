"""GPU: the prompt compactor's work items at their edges -- item sizes of one
to several batches, pages shared by the waves of a workgroup (transposed value
pages of highly compressed heads), heads that accumulate the whole prompt, and
importances averaged over a group -- against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import Pair, assert_close, f64, log, torch_dtype
from workloads import decision_logits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,Hq,Hkv,d,page,n,crs,window,omega", [
    # transposed value pages, 16-token items: 8 and 16 slots per wave, and whole pages
    ("bf16", 2, 16, 4, 128, 32, 515, (1, 2, 8, 32), 0, "lead"),
    ("bf16", 3, 16, 2, 64, 32, 129, (4, 1e9), 0, "group_mean"),
    ("bf16", 2, 16, 4, 128, 32, 700, (1, 3, 8, 1e9), 12, "group_mean"),
    # 32-token items (units * n above 6144 * 16)
    ("bf16", 26, 16, 4, 128, 32, 1000, (1, 2, 4, 16), 0, "group_mean"),
    ("bf16", 25, 16, 4, 64, 32, 1000, (2, 5, 16, 64), 5, "lead"),
    # row caches: runs of any slot count
    ("bf16", 1, 4, 4, 128, 8, 257, (1, 2, 7, 1e9), 0, "lead"),
    ("fp32", 2, 8, 4, 64, 16, 333, (1, 3, 32, 1e9), 0, "group_mean"),
    ("bf16", 25, 4, 4, 64, 64, 1000, (1, 2, 16, 1e9), 0, "uniform"),
])
def test_prefill_items(torch_cuda, dtype, B, Hq, Hkv, d, page, n, crs, window, omega):
    import torch
    log(f"case items {dtype} B={B} {Hq}/{Hkv} d={d} page={page} n={n} {crs} w={window} {omega}")
    rng = np.random.default_rng(n + B)
    pair = Pair(1, B, Hq, Hkv, d, dtype, page, n + 4, omega_src=omega, window=window)
    k = rng.standard_normal((B, n, Hkv, d), dtype=np.float32)
    v = rng.standard_normal((B, n, Hkv, d), dtype=np.float32)
    q0 = rng.standard_normal((B, n, Hq), dtype=np.float32)
    k[..., 0] = decision_logits(rng.uniform(size=(B, n, Hkv)), np.asarray(crs)[None, None])
    dt = torch_dtype(dtype)
    kt, vt, qt = (torch.from_numpy(x).to(dt).cuda() for x in (k, v, q0))
    lens = rng.integers(1, n + 1, size=B)
    lens[0] = n
    pair.prefill(0, kt, vt, qt, prompt_lens=lens)
    pair.compare_cache(0)
    # the caches then decode (a token per sequence, through the pages just written)
    q, kk, vv = (torch.from_numpy(rng.standard_normal((B, h, d), dtype=np.float32)).to(dt).cuda()
                 for h in (Hq, Hkv, Hkv))
    pair.decode(0, q, kk, vv)
    pair.ok()


@pytest.mark.parametrize("d,omega,attend", [(64, "group_mean", False), (128, "lead", True)])
def test_full_items_staged(torch_cuda, d, omega, attend):
    """128-token items (units * n above 6144 * 112) on transposed value pages with staged
    importances: every unit's slot indices and lengths against the decisions, sampled
    units' caches (and prompt outputs) against a per-unit oracle."""
    import torch
    import paper_2403_09636_amd as P
    B, Hq, Hkv, n, G = 44, 16, 4, 4096, 4
    log(f"case full items d={d} {omega} attend={attend}")
    gen = torch.Generator(device="cuda").manual_seed(d)

    def rnd(heads):
        return torch.randn((B, n, heads, d), generator=gen, device="cuda", dtype=torch.bfloat16)

    k, v, q = rnd(Hkv), rnd(Hkv), rnd(Hq)
    rng = np.random.default_rng(d)
    k0 = decision_logits(rng.uniform(size=(B, n, Hkv)), np.array([1, 2, 9, 1e9])[None, None])
    k[..., 0] = torch.from_numpy(k0).to(k)
    lens = rng.integers(n // 2, n + 1, size=B)
    lens[0] = n
    cache = P.DMCCache(P.make_config(1, B, Hq, Hkv, d, "bf16", max_slots_per_seq=n, max_prompt_len=n,
                                     omega_src=omega))
    slot = torch.empty((B, Hkv, n), dtype=torch.int32, device="cuda")
    lens_t = torch.as_tensor(lens, dtype=torch.int32, device="cuda")
    if attend:
        out = cache.prefill_attend(0, k, v, q, prompt_lens=lens_t, slot_index=slot)
    else:
        cache.prefill(0, k, v, q, prompt_lens=lens_t, slot_index=slot)
    cache.check()
    alpha = oracle.decision(f64(k[..., 0]), 0.0)
    alpha[:, 0] = 0
    want = (np.cumsum(1 - alpha, axis=1) - 1).transpose(0, 2, 1)
    want = np.where(np.arange(n) < lens[:, None, None], want, -1)
    assert (slot.cpu().numpy() == want).all()
    lengths = cache.lengths(0).cpu().numpy()
    assert (lengths == want.max(axis=2) + 1).all()
    K, V, z = cache.export(0, dense_slots=n)
    for b, g in [(0, 0), (0, 1), (17, 2), (30, 3), (43, 1)]:
        m, hs = int(lens[b]), slice(g * G, (g + 1) * G)
        orc = oracle.DMCOracle(1, 1, G, 1, d, max_slots=n, omega_src=omega)
        kb, vb, qb = f64(k[b:b + 1, :m, g:g + 1]), f64(v[b:b + 1, :m, g:g + 1]), f64(q[b:b + 1, :m, hs])
        if attend:
            o_ref, _ = orc.prefill_attend(0, qb, kb, vb)
            assert_close(f64(out[b, :m, hs]), o_ref[0], "bf16", f"outputs of unit {(b, g)}")
            assert (out[b, m:, hs] == 0).all()
        else:
            orc.prefill(0, kb, vb, qb[..., 0])
        K_ref, V_ref, l_ref, z_ref = orc.export(0)
        l = int(l_ref[0, 0])
        assert_close(f64(K[b, g, :l]), K_ref[0, 0, :l], "bf16", f"keys of unit {(b, g)}")
        assert_close(f64(V[b, g, :l]), V_ref[0, 0, :l], "bf16", f"values of unit {(b, g)}")
        assert np.isclose(float(z[b, g]), z_ref[0, 0], rtol=1e-4)
