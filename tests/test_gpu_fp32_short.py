"""GPU: fp32 prompt and training attention of short sequences -- both sides of the
lines between the vector-ALU and the matrix kernels, ragged and windowed -- against
float64."""
import numpy as np
import pytest

import oracle.dmc_train as T
from tests.gpu_helpers import Pair, f64, log
from tests.test_gpu_train import _close_scaled, _grad_close, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G,B,Hkv,n,window", [
    (64, 1, 2, 3, 4, 0), (64, 1, 2, 3, 5, 0), (64, 2, 30, 8, 6, 0), (64, 8, 40, 8, 9, 5), (64, 8, 20, 8, 9, 0),
    (128, 4, 2, 3, 8, 0), (128, 4, 2, 3, 9, 3), (128, 8, 10, 8, 20, 0), (128, 8, 2, 8, 20, 0),
    (128, 8, 9, 8, 36, 12), (128, 8, 4, 8, 36, 0), (128, 1, 1, 2, 1, 0),
])
def test_short_prompt(torch_cuda, d, G, B, Hkv, n, window):
    import torch
    log(f"case short fp32 prompt d={d} G={G} B={B} Hkv={Hkv} n={n} w={window}")
    rng = np.random.default_rng(n * d + G)
    pair = Pair(1, B, Hkv * G, Hkv, d, "fp32", 16, n + 2, max_prompt_len=n, window=window)
    k, v = (rng.standard_normal((B, n, Hkv, d), dtype=np.float32) for _ in range(2))
    q = rng.standard_normal((B, n, Hkv * G, d), dtype=np.float32)
    lens = rng.integers(0, n + 1, size=B)
    lens[0] = n
    pair.prefill_attend(0, *(torch.from_numpy(x).cuda() for x in (k, v, q)), prompt_lens=lens)
    pair.compare_cache(0)
    pair.ok()


@pytest.mark.parametrize("d,G,B,Hkv,n,window", [
    (64, 4, 2, 3, 4, 3), (64, 8, 2, 3, 4, 3), (64, 1, 64, 8, 12, 5), (64, 1, 64, 8, 13, 5),
    (128, 2, 2, 3, 8, 12), (128, 2, 2, 3, 9, 12), (128, 8, 56, 8, 17, 4), (128, 1, 64, 8, 33, 4),
    (128, 1, 64, 8, 37, 4), (128, 1, 1, 1, 1, 1),
])
def test_short_training(torch_cuda, d, G, B, Hkv, n, window):
    import torch
    import paper_2403_09636_amd as P
    log(f"case short fp32 training d={d} G={G} B={B} Hkv={Hkv} n={n} w={window}")
    rng = np.random.default_rng(n * d + G)
    q, k, v, noise, dout, dalpha = _inputs(rng, B, n, Hkv, G, d, [2.0, 1.0, 4.0, 8.0, 2.0, 1.0, 4.0, 8.0][:Hkv], 5.0)
    trainer = P.DMCTrainer(P.make_train_config(B, n, Hkv * G, Hkv, d, "fp32", window=window), "cuda")
    gq, gk, gv, gn, gdo, gda = (torch.from_numpy(x).cuda() for x in (q, k, v, noise, dout, dalpha))
    out = trainer.forward(gq, gk, gv, gn)
    grads = trainer.backward(gq, gk, gv, gn, out, gdo, dalpha=gda)
    for b in {0, B // 2, B - 1}:   # (sequences are independent)
        one = [torch.from_numpy(x[b:b + 1].astype(np.float64)) for x in (q, k, v, noise, dout, dalpha)]
        want = T.train_forward(*one[:4], window=window)[0]
        _close_scaled(f64(out[b:b + 1]), np.asarray(want), "fp32", f"out of sequence {b}")
        ref = T.train_backward(*one[:5], dalpha=one[5], window=window)
        for name, got, w in zip(("dq", "dk", "dv"), grads, ref):
            _grad_close(f64(got[b:b + 1]), np.asarray(w), "fp32", f"{name} of sequence {b}")
