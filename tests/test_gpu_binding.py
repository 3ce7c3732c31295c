"""The Python binding's checks: what it refuses, with which error, through every
entry point that takes a batch; and that calls go to the current stream."""
import numpy as np
import pytest
import torch

import paper_2603_26110_amd as tq
from gpu_cases import Case

pytestmark = pytest.mark.gpu


def _setup():
    case = Case(91, 1, 2, 3, 80, flags=tq.V_ROTATE, slots=3 * 128, slot0=[0, 128, 256])
    cache = tq.Cache(1, 2, 3 * 128)
    case.gpu_quantize(cache)
    lens = torch.full((3,), 70, dtype=torch.int32, device="cuda")
    common = dict(pi=case.t("pi"), lut_k=case.t("lut_k"), lut_v=case.t("lut_v"), qjl_s=case.t("S"))
    decode = dict(q=case.t("q"), seq_slot0=case.t("slot0"), seq_len=lens, max_len=80, **common)
    new = dict(k=case.t("k")[:, :, 79].contiguous(), v=case.t("v")[:, :, 79].contiguous(), pos=lens)
    return case.params(), cache, {
        tq.quantize_pack: dict(k=case.t("k"), v=case.t("v"), pos0=case.t("pos0"), slot0=case.t("slot0"), **common),
        tq.decode_attend: dict(q_pos=lens, **decode),
        tq.decode_attend_noalloc: dict(q_pos=lens, **decode),
        tq.decode_step: dict(**new, **decode),
    }


def test_wrong_tensors_are_refused():
    params, cache, calls = _setup()
    for f, args in calls.items():
        f(params, cache, **args)
        for name, t in args.items():
            if not isinstance(t, torch.Tensor):
                continue
            for bad in (t.cpu(), t.cpu().numpy(), None, t.double()):
                with pytest.raises(TypeError):
                    f(params, cache, **{**args, name: bad})
            strided = torch.stack([t, t], -1)[..., 0]
            with pytest.raises(ValueError):
                f(params, cache, **{**args, name: strided})
        for name in ("q", "k", "v"):
            if name in args:
                with pytest.raises(ValueError):
                    f(params, cache, **{**args, name: args[name][..., :32].contiguous()})
    with pytest.raises(ValueError):
        tq.quantize_pack(params, cache, **{**calls[tq.quantize_pack], "pos0": torch.zeros(2, dtype=torch.int32).cuda()})
    for f in (tq.decode_attend, tq.decode_step):
        with pytest.raises(TypeError):
            f(params, cache, **calls[f], ebar=torch.zeros(1, 2, 2))
        with pytest.raises(TypeError):
            f(params, cache, **calls[f], out=torch.empty_like(calls[f]["q"], dtype=torch.float32))


def test_calls_go_to_the_current_stream():
    params, cache, calls = _setup()
    f, args = tq.decode_attend, calls[tq.decode_attend]
    ref = f(params, cache, **args)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    q = torch.zeros_like(args["q"])
    with torch.cuda.stream(side):
        for _ in range(20):                       # work that the call has to come after
            big = torch.randn(4096, 4096, device="cuda") @ torch.randn(4096, 4096, device="cuda")
        q.copy_(args["q"])
        got = f(params, cache, **{**args, "q": q})
    side.synchronize()
    assert big.shape == (4096, 4096) and torch.equal(got, ref)
    for o in (got, f(params, cache, **args, out=torch.empty_like(ref))):
        assert o.shape == ref.shape and o.stride() == ref.stride() and o.dtype == ref.dtype
    p32 = tq.Params(params.num_layers, params.num_heads, params.rope_cs, flags=tq.V_ROTATE | tq.OUT_FP32)
    assert f(p32, cache, **args).dtype == torch.float32
