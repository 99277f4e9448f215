"""GPU: the prompt compactor's work items at their edges -- item sizes of one
to several batches, pages shared by the waves of a workgroup (transposed value
pages of highly compressed heads), heads that accumulate the whole prompt, and
importances averaged over a group -- against the oracle."""
import numpy as np
import pytest

from tests.gpu_helpers import Pair, log, torch_dtype
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
