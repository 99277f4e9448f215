"""The one-pass tensor checks of a decode step (_DecodeCall) accept exactly what
check_decode_args accepts: every single-property break, on CPU tensors."""
import pytest
import torch

import paper_2403_09636_amd as P
from paper_2403_09636_amd import binding as Bd

DEV = torch.device("cpu")
B, HQ, HKV, D = 2, 8, 2, 64


def _args(dtype):
    return dict(q=torch.zeros(B, HQ, D, dtype=dtype), k=torch.zeros(B, HKV, D, dtype=dtype),
                v=torch.zeros(B, HKV, D, dtype=dtype), out=torch.zeros(B, HQ, D, dtype=dtype),
                slot_index=torch.zeros(B, HKV, dtype=torch.int32))


def _breaks(name, t):
    """Versions of one argument with one property changed (and the argument itself)."""
    yield "same", t
    yield "dtype", t.to(torch.int64 if name == "slot_index" else torch.float16)
    yield "rank", t[None]
    yield "size", torch.cat([t, t], -1)
    yield "layout", t.transpose(0, 1).contiguous().transpose(0, 1)
    yield "strided", torch.cat([t, t], -1)[..., :t.shape[-1]]
    base = torch.zeros(t.numel() + 1, dtype=t.dtype)
    yield "offset by one element", base[1:].view(t.shape)
    yield "device", t.to("meta")
    yield "not a tensor", [0]
    yield "parameter", torch.nn.Parameter(t, requires_grad=False)
    if name == "slot_index":
        yield "none", None


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("name", ["q", "k", "v", "out", "slot_index"])
def test_same_verdict_as_full_checks(name, dtype):
    cfg = P.make_config(1, B, HQ, HKV, D, dtype, max_slots_per_seq=128)
    call = Bd._DecodeCall(cfg, DEV)
    for what, bad in _breaks(name, _args(Bd.cache_dtype(cfg))[name]):
        a = dict(_args(Bd.cache_dtype(cfg)), **{name: bad})
        try:
            Bd.check_decode_args(cfg, DEV, **a)
            fine = True
        except P.DMCError:
            fine = False
        got = call.pointers(**a)
        assert (got is not None) == fine, (name, what, fine)
        if fine:
            assert got == tuple(None if t is None else t.data_ptr()
                                for t in (a["q"], a["k"], a["v"], a["out"], a["slot_index"]))


@pytest.mark.parametrize("other", ["q", "k", "v"])
@pytest.mark.parametrize("shift", [0, 8, 16, HQ * D - 8, HQ * D])
def test_overlap_verdict(other, shift):
    cfg = P.make_config(1, B, HQ, HKV, D, "fp32", max_slots_per_seq=128)
    a = _args(torch.float32)
    n, m = a["out"].numel(), a[other].numel()
    pool = torch.zeros(n + m + shift)
    a["out"] = pool[:n].view(B, HQ, D)
    a[other] = pool[shift:shift + m].view(a[other].shape)
    try:
        Bd.check_decode_args(cfg, DEV, **a)
        fine = True
    except P.DMCError:
        fine = False
    assert (Bd._DecodeCall(cfg, DEV).pointers(**a) is not None) == fine
