"""Decode calls that may read more cache bytes (by max_len) than the Infinity Cache keeps take another instantiation,
which loads its tiles with a hint where the lengths say that they do: the same outputs as with a max_len close to the
lengths, and as among other lengths. 8 waves per block (more tiles than waves), 4 waves with V signs, and few units,
whose blocks and splits depend on max_len."""
import pytest
import torch

import paper_2603_26110_amd as tq
from gpu_cases import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,H,B,T,near,max_len,flags,same", [
    (33, 20, 1, 1100, 1152, 6400, tq.V_ROTATE, True),
    (33, 20, 10, 70, 128, 640, tq.V_ROTATE | tq.V_QJL, True),
    (4, 2, 2, 1217, 1280, 262144, tq.V_ROTATE, False),
])
def test_outputs_do_not_depend_on_the_load_hint(L, H, B, T, near, max_len, flags, same):
    assert 72 * L * H * B * max_len > 300e6 > 72 * L * H * B * near
    case = Case(96, L, H, B, T, flags=flags, slots=B * max_len, slot0=[b * max_len for b in range(B)])
    cache = tq.Cache(L, H, B * max_len)
    case.gpu_quantize(cache)
    n = torch.full((B,), T, dtype=torch.int32).cuda()
    p = case.params(flags | tq.OUT_FP32)
    out = [tq.decode_attend(p, cache, case.t("q"), n - 1, case.t("slot0"), n, m, case.t("pi"), case.t("lut_k"),
                            case.t("lut_v"), case.t("S")) for m in (near, max_len)]
    assert bool(torch.isfinite(out[0]).all())
    if same:
        assert torch.equal(*out)
    else:     # fp32 sums of T weights in another order: 1e-5 of the largest value
        assert float((out[0] - out[1]).abs().max()) <= 1e-5 * float(out[0].abs().max())


@pytest.mark.parametrize("L,H,B,T,others,flags", [
    (1, 40, 16, 8000, 100, tq.V_ROTATE),                 # 8 waves per block
    (2, 40, 70, 1000, 64, tq.V_ROTATE | tq.V_QJL),        # more sequences than lanes; 4 waves
    (33, 20, 1, 7000, None, tq.V_ROTATE),                 # one sequence of 16-wave blocks
])
def test_outputs_do_not_depend_on_the_other_sequences_lengths(L, H, B, T, others, flags):
    # the hint follows the lengths that a call reads: all sequences long, against
    # one of them among short ones (the same blocks and splits, no hint)
    cap = (T + 63) // 64 * 64
    case = Case(97, L, H, B, 1, flags=flags, slots=B * cap, slot0=[b * cap for b in range(B)])
    cache = tq.Cache(L, H, B * cap)
    g = torch.Generator(device="cuda").manual_seed(98)
    for p in (cache.k_codes, cache.v_codes):
        p.copy_(torch.randint(0, 256, p.shape, generator=g, device="cuda", dtype=torch.uint8))
    cache.scalars.copy_(torch.rand(cache.scalars.shape, generator=g, device="cuda").half().view(torch.int16))
    assert 72 * L * H * B * T > 300e6
    run = lambda n: tq.decode_attend(case.params(flags | tq.OUT_FP32), cache, case.t("q"), n * 0, case.t("slot0"), n, T,
                                     case.t("pi"), case.t("lut_k"), case.t("lut_v"), case.t("S"))
    whole = run(torch.full((B,), T, dtype=torch.int32).cuda())
    assert bool(torch.isfinite(whole).all())
    for b in {0, B // 2, B - 1}:
        n = torch.full((B,), others or T, dtype=torch.int32)
        n[b] = T
        assert others is None or 72 * L * H * int(n.sum()) < 300e6
        assert torch.equal(run(n.cuda())[:, b], whole[:, b])
