"""tq_dequantize writes the same rows whichever number of tiles its blocks take
(one for few tiles, two and three at these sizes, four from 4096 tiles on),
ragged lengths among them; rows past a length stay as they were."""
import pytest
import torch

import paper_2603_26110_amd as tq
from gpu_cases import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,H,lens,flags", [
    (26, 20, [250], tq.V_ROTATE), (33, 20, [65, 300], tq.V_ROTATE | tq.V_QJL), (33, 20, [448, 1], tq.V_ROTATE),
])
def test_rows_do_not_depend_on_the_tiles_per_block(L, H, lens, flags):
    B, T = len(lens), max(lens)
    cap = (T + 63) // 64 * 64
    case = Case(95, L, H, B, T, flags=flags, slots=B * cap, slot0=[b * cap for b in range(B)])
    cache = tq.Cache(L, H, B * cap)
    case.gpu_quantize(cache)
    n = torch.tensor(lens, dtype=torch.int32).cuda()
    args = (case.t("slot0"), n, T, case.t("lut_k"), case.t("lut_v"), case.t("S"))
    out = lambda nl: [torch.full((nl, B, H, T, 64), 7.0, dtype=torch.float16, device="cuda") for _ in range(2)]
    whole = out(L)
    tq.dequantize(case.params(), cache, *args, k_out=whole[0], v_out=whole[1])
    for l in range(0, L, 5):
        one = out(1)
        tq.dequantize(case.params(), cache, *args, layer0=l, nlayers=1, k_out=one[0], v_out=one[1])
        assert torch.equal(whole[0][l:l + 1], one[0]) and torch.equal(whole[1][l:l + 1], one[1])
    for b in range(B):
        assert bool((whole[0][:, b, :, lens[b]:] == 7.0).all()) and bool((whole[1][:, b, :, lens[b]:] == 7.0).all())
