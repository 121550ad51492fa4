"""The argument check in front of the hot calls (csrc/tng_call.cpp) on device tensors: what it takes as plain reaches the entry
point by address, everything else is left to ctypes, which raises.  The entry points are host stand-ins: nothing is launched."""
import ctypes

import pytest
import torch

from gpu_util import DEV, make_ctx
from paper_1901_08227_amd import binding as B

pytestmark = pytest.mark.gpu

D, M, WORDS = 40, 3, 5
SIZES = {"d": D, "g": M * D, "c": M * WORDS, "s": M}


class Subclass(torch.Tensor):
    pass


@pytest.fixture
def entry():
    B.lib()
    seen = []
    fn = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p)(
        lambda h, it, a, b: seen.append((h, it, a, b)) or 5)
    at = ctypes.cast(fn, ctypes.c_void_p).value
    yield lambda kind, t: B._call(at, 4096, 9, kind + "d", D, M, WORDS, t, None), seen
    del fn


def tensor(kind, n=None, dtype=None):
    return torch.zeros(SIZES[kind] if n is None else n, dtype=dtype or (torch.int32 if kind == "c" else torch.float32), device=DEV)


@pytest.mark.parametrize("kind", "dgcs")
def test_plain_tensors_reach_the_entry_point(entry, kind):
    call, seen = entry
    n = SIZES[kind]
    whole = tensor(kind, n + 7)
    plain = [tensor(kind), whole, whole[3:3 + n], tensor(kind, 2 * n).view(2, n), tensor(kind).view(n, 1)]
    if kind != "c":
        plain.append(torch.nn.Parameter(tensor(kind)))  # (a plain tensor to the check, as it was to ctypes' way)
    for t in plain:
        del seen[:]
        assert call(kind, t) == 5 and seen == [(4096, 9, t.data_ptr(), None)]


@pytest.mark.parametrize("kind", "dgcs")
def test_other_tensors_do_not(entry, kind):
    call, seen = entry
    n = SIZES[kind]
    other = [tensor(kind, n - 1), tensor(kind, 2 * n)[::2], tensor(kind, 2 * n).view(n, 2)[:, 0], tensor(kind, 2 * n).view(n, 2).t(),
             tensor(kind).cpu(), tensor(kind).as_subclass(Subclass), torch.zeros(1, device=DEV).expand(n),
             tensor(kind).to_sparse(), [0.0] * n]
    for dtype in (torch.float64, torch.float16, torch.bfloat16, torch.int64, torch.int16, torch.uint8,
                  torch.float32 if kind == "c" else torch.int32):
        other.append(tensor(kind, dtype=dtype))
    for t in other:
        assert call(kind, t) is None, t
    assert seen == []


def test_the_context_calls_refuse_what_they_refused():
    ctx = make_ctx(D, M, 2, B.NORM_SUB)
    assert ctx.words == -(-D // 16)
    good = dict(w=tensor("d"), gref=tensor("d"), g=tensor("g"), codes=tensor("c", M * ctx.words), scales=tensor("s"), vbar=tensor("d"))
    calls = {"step": "w gref g codes scales vbar", "normalize_encode": "g gref codes scales", "decode_aggregate": "codes scales gref vbar",
             "update_reference": "vbar gref", "local_grad": "w g"}
    for name, names in calls.items():
        for bad in names.split():
            n = good[bad].numel()
            for t, error in ((good[bad].cpu(), TypeError), (good[bad].to(torch.float64), TypeError),
                             (torch.cat([good[bad], good[bad]])[::2], TypeError), (good[bad][:n - 1].clone(), ValueError), ("x", TypeError)):
                args = [t if k == bad else good[k] for k in names.split()]
                with pytest.raises(error):
                    getattr(ctx, name)(*([] if name == "decode_aggregate" else [0]), *args)
            if name != "local_grad":  # (a null pointer is the entry point's to refuse; a problem without data is, before it)
                args = [None if k == bad else good[k] for k in names.split()]
                with pytest.raises(B.TngError) as e:
                    getattr(ctx, name)(*([] if name == "decode_aggregate" else [0]), *args)
                assert e.value.status == B.TNG_ERR_INVALID_ARG
    ctx.close()
