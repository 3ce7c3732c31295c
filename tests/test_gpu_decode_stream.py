"""Decode calls over more cache bytes (by max_len) than the Infinity Cache keeps load their tiles with another
hint: the same outputs as with a max_len close to the lengths, which does not. 8 waves per block (more tiles than
waves), 4 waves with V signs, and few units, whose blocks and splits depend on max_len."""
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
