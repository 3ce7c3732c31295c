"""The prefill kernel at the edges of its groups of 32 tokens, of its words and
16-byte runs of slots, of its shares of (layer, head)s, of its windows of 64
sequences, and at the scales where it stops leaving a vector's scale in.

Against the oracle by the rule of assert_agree_up_to_threshold_rounding, and
byte for byte against calls that reach the same tokens another way."""
import numpy as np
import pytest
import torch

import paper_2603_26110_amd as tq
from gpu_cases import Case, assert_agree_up_to_threshold_rounding, device_bytes
from oracle import oracle
from paper_2603_26110_amd import synth

pytestmark = pytest.mark.gpu


def _planes(cache):
    return cache.k_codes.clone(), cache.v_codes.clone(), cache.scalars.clone()


@pytest.mark.parametrize("io", ["f16", "f32"])
@pytest.mark.parametrize("T,first,flags", [
    (64, 0, tq.V_ROTATE), (65, 5, tq.V_ROTATE), (95, 8, 0), (96, 32, tq.V_ROTATE | tq.ROPE_HALF),
    (97, 37, tq.V_ROTATE | tq.V_QJL), (127, 24, tq.V_QJL), (161, 63, tq.V_ROTATE | tq.QJL_PAPER),
    (72, 31, tq.V_ROTATE | tq.QJL_PAPER | tq.V_QJL),
])
def test_prefill_at_group_and_slot_edges(T, first, flags, io):
    B, H = 2, 2
    cap = (T + first + 127) // 64 * 64
    case = Case(70 + T, 1, H, B, T, io=io, flags=flags, slots=B * cap, slot0=[first, cap + first], pos0=[0, 11])
    cache = tq.Cache(1, H, B * cap)
    for t in (cache.k_codes, cache.v_codes):
        t.copy_(torch.randint(0, 256, t.shape, dtype=torch.uint8, device="cuda"))
    before = device_bytes(cache)
    oc = oracle.Cache(1, H, B * cap)
    oc.k[:], oc.v[:] = before.k, before.v                    # (neighbouring slots keep their bits)
    case.gpu_quantize(cache)
    torch.cuda.synchronize()
    case.oracle_quantize(oc)
    got = device_bytes(cache)
    assert_agree_up_to_threshold_rounding(case, got, oc, B, T, H, tokens=sorted({0, 1, 7, 31, 32, T - 2, T - 1}))
    # all bytes of slots that were not written are as they were
    written = np.zeros(B * cap, bool)
    for b in range(B):
        written[b * cap + first:b * cap + first + T] = True
    tiles = lambda p: p.reshape(H, B * cap // 64, 2, 64, 16)
    nib = lambda p: np.stack([tiles(p) & 15, tiles(p) >> 4], -1).reshape(H, B * cap // 64, 2, 64, 32)
    v_got = nib(got.v).transpose(0, 1, 2, 4, 3).reshape(H, B * cap, 64)
    v_old = nib(before.v).transpose(0, 1, 2, 4, 3).reshape(H, B * cap, 64)
    np.testing.assert_array_equal(v_got[:, ~written], v_old[:, ~written])
    k_of = lambda p: tiles(p).transpose(0, 1, 3, 2, 4).reshape(H, B * cap, 32)
    np.testing.assert_array_equal(k_of(got.k)[:, ~written], k_of(before.k)[:, ~written])


def test_ragged_windows_of_many_sequences():
    # 150 sequences (three windows of 64), some empty, against each alone
    g = synth.rng(77)
    B, T, H = 150, 100, 2
    lens = g.integers(0, T + 1, B)
    lens[[0, 3, 63, 64, 127, 149]] = [0, T, 0, 33, 32, T]
    cap = 128
    case = Case(78, 1, H, B, T, slots=B * cap, slot0=[b * cap + b % 9 for b in range(B)], pos0=[b % 7 for b in range(B)])
    args = (case.t("pi"), case.t("lut_k"), case.t("lut_v"), case.t("S"))
    ragged, each = tq.Cache(1, H, B * cap), tq.Cache(1, H, B * cap)
    tokens = torch.tensor(lens, dtype=torch.int32).cuda()
    tq.quantize_pack(case.params(), ragged, case.t("k"), case.t("v"), case.t("pos0"), case.t("slot0"), *args,
                     seq_tokens=tokens)
    for b in range(B):
        tq.quantize_pack(case.params(), each, case.t("k")[:, b:b + 1].contiguous(), case.t("v")[:, b:b + 1].contiguous(),
                         case.t("pos0")[b:b + 1].clone(), case.t("slot0")[b:b + 1].clone(), *args,
                         seq_tokens=tokens[b:b + 1].clone())
    for x, y in zip(_planes(ragged), _planes(each)):
        assert torch.equal(x, y)


def test_shares_over_many_heads():
    # 36 x 40 (layer, head)s of two groups: a block's share takes more than the
    # four that it stages at once; one (layer, head) has a bad table
    L, H, T = 36, 40, 64
    case = Case(79, L, H, 1, T, slots=128)
    case.lut_v[20, 7, 3] = case.lut_v[20, 7, 4]
    args = lambda: (case.t("pi"), case.t("lut_k"), case.t("lut_v"), case.t("S"))
    whole, each = tq.Cache(L, H, 128), tq.Cache(L, H, 128)
    tq.quantize_pack(case.params(), whole, case.t("k"), case.t("v"), case.t("pos0"), case.t("slot0"), *args())
    for l in range(L):
        tq.quantize_pack(case.params(), each, case.t("k")[l:l + 1].contiguous(), case.t("v")[l:l + 1].contiguous(),
                         case.t("pos0"), case.t("slot0"), *args(), layer0=l)
    for x, y in zip(_planes(whole), _planes(each)):
        assert torch.equal(x, y)
    k = whole.k_codes.view(L, H, 128 * 32)
    assert not k[20, 7].any() and all(bool(k[l, h].any()) for l, h in ((20, 6), (20, 8), (0, 0), (35, 39)))


@pytest.mark.parametrize("e", [-60, -39, -20, 30, 41, 50])
def test_codes_do_not_depend_on_a_power_of_two(e):
    # RoPE, the rotation, norms and levels scale exactly while nothing leaves
    # fp32's range: the same codes, signs and residual norms
    case = Case(80, 1, 2, 1, 80, io="f32", flags=tq.V_ROTATE | tq.V_QJL, slots=128)
    one, scaled = tq.Cache(1, 2, 128), tq.Cache(1, 2, 128)
    case.gpu_quantize(one)
    case.gpu_quantize(scaled, k=case.t("k") * 2.0 ** e, v=case.t("v") * 2.0 ** e)
    assert torch.equal(one.k_codes, scaled.k_codes) and torch.equal(one.v_codes, scaled.v_codes)
    assert torch.equal(one.scalars.view(-1, 4)[:, 1::2], scaled.scalars.view(-1, 4)[:, 1::2])


def test_subnormal_fp16_values():
    # fp16 values enter the products as they are; the fp32 path scales them first.
    # Both are within rounding of x^, so codes differ only at thresholds (3e-6 of
    # the coordinates against 64 bits elsewhere) and norms by an fp16 ulp.
    case = Case(81, 1, 4, 1, 256, io="f16", flags=tq.V_ROTATE, slots=256)
    g = synth.rng(82)
    case.v = (g.integers(-255, 256, case.v.shape) * 2.0 ** -24).astype(np.float16)
    half, full = tq.Cache(1, 4, 256), tq.Cache(1, 4, 256)
    case.gpu_quantize(half)
    p = case.params(io="f32")
    tq.quantize_pack(p, full, case.t("k").float(), case.t("v").float(), case.t("pos0"), case.t("slot0"), case.t("pi"),
                     case.t("lut_k"), case.t("lut_v"), case.t("S"))
    assert float((half.v_codes != full.v_codes).float().mean()) <= 1e-4
    n = [c.scalars.view(torch.float16).view(-1, 4)[:, 2].float() for c in (half, full)]
    assert float((n[0] - n[1]).abs().max()) <= 2.0 ** -24 and float(n[0].min()) > 0


@pytest.mark.parametrize("io", ["f16", "f32"])
@pytest.mark.parametrize("T,lens,flags", [
    (1, None, tq.V_ROTATE), (7, None, tq.V_ROTATE), (13, None, tq.V_QJL), (63, None, tq.V_ROTATE | tq.V_QJL),
    (30, [30, 0, 1, 17, 29, 4, 8, 30], tq.V_ROTATE | tq.ROPE_HALF), (20, None, tq.V_ROTATE | tq.QJL_PAPER),
])
def test_short_sequences_in_a_batch_equal_each_alone(T, lens, flags, io):
    # a batch large enough for the kernel that shares a block's Pi and S, against
    # calls that the kernel of one vector per wave takes: the same bytes, and the
    # neighbouring slots untouched (first slots at every remainder of 8)
    H, B = 40, 64 if T == 1 else 8
    cap = 128
    slot0 = [b * cap + (3 * b) % 64 for b in range(B)]
    slot0[B - 1] = B * cap - 1                               # its later tokens have no slot
    case = Case(83 + T, 1, H, B, T, io=io, flags=flags, slots=B * cap, slot0=slot0, pos0=[5 * b for b in range(B)],
                positions=5 * B - 2)                          # and the last position is past the table
    args = (case.t("pi"), case.t("lut_k"), case.t("lut_v"), case.t("S"))
    tokens = None if lens is None else torch.tensor(lens, dtype=torch.int32).cuda()
    batch, each = tq.Cache(1, H, B * cap), tq.Cache(1, H, B * cap)
    for x, y in zip((batch.k_codes, batch.v_codes), (each.k_codes, each.v_codes)):
        x.copy_(torch.randint(0, 256, x.shape, dtype=torch.uint8, device="cuda"))
        y.copy_(x)
    tq.quantize_pack(case.params(), batch, case.t("k"), case.t("v"), case.t("pos0"), case.t("slot0"), *args,
                     seq_tokens=tokens)
    for b in range(B):
        for j in range(0, T, 32):                            # (few enough token-heads at a time for that kernel)
            k, v = (case.t(n)[:, b:b + 1, j:j + 32].contiguous() for n in "kv")
            tq.quantize_pack(case.params(), each, k, v, case.t("pos0")[b:b + 1] + j, case.t("slot0")[b:b + 1] + j, *args,
                             seq_tokens=None if lens is None else tokens[b:b + 1] - j)
    for x, y in zip(_planes(batch), _planes(each)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("flags", [tq.QJL_PAPER, tq.QJL_PAPER | tq.V_QJL])
def test_element_signs_of_vectors_with_nan(flags):
    # sign_i = !(r_i < 0): a NaN residual, of either sign bit, and a zero one have
    # sign 1. Against calls of 16 tokens, which another kernel takes.
    T, H = 96, 2
    flags |= tq.INPUT_ROTATED
    case = Case(84, 1, H, 1, T, io="f32", flags=flags, slots=128)
    case.lut_k[0, 1, 3] = case.lut_v[0, 1, 4] = 0.0          # r = -0 - 0 for a coordinate of -0
    for x in (case.k, case.v):
        x[0, 0, ::2, :, 20:24] = -0.0
        x[0, 0, 3::16, :, 5] = np.inf                        # u = inf * 0 there
        x[0, 0, 5::16, :, 7] = np.nan
        x.view(np.uint32)[0, 0, 7::16, :, 9] = 0xFFC00000     # NaN with the sign bit set
    whole, parts = tq.Cache(1, H, 128), tq.Cache(1, H, 128)
    case.gpu_quantize(whole)
    for j in range(0, T, 16):
        case.gpu_quantize(parts, k=case.t("k")[:, :, j:j + 16].contiguous(), v=case.t("v")[:, :, j:j + 16].contiguous(),
                          pos0=[j], slot0=[j])
    assert all(torch.equal(x, y) for x, y in zip(_planes(whole), _planes(parts)))


@pytest.mark.parametrize("flags", [tq.V_ROTATE, tq.V_ROTATE | tq.V_QJL])
def test_subnormal_fp32_vectors(flags):
    # largest entries of 2^-121 to 2^-149 and exact zeros: every square underflows,
    # so n = 0 and the codes are those of a zero vector, as in calls of 16 tokens
    T, H = 96, 2
    case = Case(85, 1, H, 1, T, io="f32", flags=flags, slots=128)
    g = synth.rng(86)
    for x in (case.k, case.v):
        e = -121.0 - (np.arange(T) % 29)
        x[:] = (g.uniform(-1, 1, x.shape) * 2.0 ** e[:, None, None]).astype(np.float32)
        x[..., ::3] = 0.0
    whole, parts = tq.Cache(1, H, 128), tq.Cache(1, H, 128)
    case.gpu_quantize(whole)
    for j in range(0, T, 16):
        case.gpu_quantize(parts, k=case.t("k")[:, :, j:j + 16].contiguous(), v=case.t("v")[:, :, j:j + 16].contiguous(),
                          pos0=[j], slot0=[j])
    assert not whole.scalars.view(-1, 4)[:T, [0, 2]].any()
    assert all(torch.equal(x, y) for x, y in zip(_planes(whole), _planes(parts)))


@pytest.mark.parametrize("flags", [0, tq.V_QJL])
def test_projected_signs_around_the_guard_band(flags):
    # Rows of S with S_i . r / (||S_i|| ||r||) spread over 2^-20 .. 2^-12, of both
    # signs, for the one residual direction that all tokens of a call share (a
    # vector times powers of two), half of them with partial sums that grow to
    # half of ||S_i|| ||r|| before they cancel: every sign is the chain's.
    g = synth.rng(87)
    T = 64
    for turn in range(12):
        case = Case(88, 1, 1, 1, T, io="f32", flags=flags | tq.INPUT_ROTATED, slots=64)
        x = g.standard_normal(64).astype(np.float32)
        idx, r = _residual(x, case.lut_k[0, 0])
        rd = r.astype(np.float64)
        unit = rd / np.linalg.norm(rd)
        S = g.standard_normal((64, 64))
        S[32:] = np.abs(S[32:]) * np.sign(rd) * np.where(np.arange(64) < 32, 1.0, -1.0)
        S[32:, 32:] *= (S[32:, :32] @ rd[:32] / -(S[32:, 32:] @ rd[32:]))[:, None]
        S -= (S @ unit)[:, None] * unit
        share = 2.0 ** np.linspace(-20, -12, 32) * np.where(np.arange(32) % 2 == turn % 2, 1.0, -1.0)
        S += np.concatenate([share, share])[:, None] * np.linalg.norm(S, axis=1)[:, None] * unit
        case.S = S.astype(np.float32)
        case.k[0, 0, :, 0] = x * 2.0 ** (np.arange(T) % 9 - 4)[:, None]
        case.v = case.k.copy()
        case.lut_v = case.lut_k.copy()
        cache = tq.Cache(1, 1, 64)
        case.gpu_quantize(cache)
        oc = oracle.Cache(1, 1, 64)
        case.oracle_quantize(oc)
        got = device_bytes(cache)
        np.testing.assert_array_equal(got.k, oc.k)
        np.testing.assert_array_equal(got.v, oc.v)


def _residual(x, lut):
    """Levels and binary32 residual of a vector, by the quantizer's steps."""
    s = np.float32(0)
    for v in x:
        s = np.float32(np.float64(v) * np.float64(v) + np.float64(s))
    u = x * np.float32(np.float32(8) / np.sqrt(s))
    idx = (u[:, None] > np.float32(0.5) * (lut[1:] + lut[:-1])).sum(1)
    return idx, u - lut[idx]


@pytest.mark.parametrize("B,every", [(130, 1), (4097, 7), (9000, 40)])
def test_ragged_batches_of_thousands_of_sequences(B, every):
    # more windows of 64 sequences than waves or lanes, most sequences empty,
    # against calls of 60 sequences
    T, H = 64, 1
    g = synth.rng(89)
    lens = np.where(np.arange(B) % every == every // 2, g.integers(1, T + 1, B), 0)
    lens[[0, B - 1]] = [5, T]
    gen = torch.Generator(device="cuda").manual_seed(90)
    k, v = (torch.randn((1, B, T, H, 64), generator=gen, device="cuda").half() for _ in range(2))
    case = Case(91, 1, H, 1, T)
    args = (case.t("pi"), case.t("lut_k"), case.t("lut_v"), case.t("S"))
    pos, first = torch.zeros(B, dtype=torch.int32).cuda(), torch.arange(B).cuda() * 64
    tokens = torch.tensor(lens, dtype=torch.int32).cuda()
    whole, parts = tq.Cache(1, H, B * 64), tq.Cache(1, H, B * 64)
    tq.quantize_pack(case.params(), whole, k, v, pos, first, *args, seq_tokens=tokens)
    for b in range(0, B, 60):
        s = slice(b, b + 60)
        tq.quantize_pack(case.params(), parts, k[:, s].contiguous(), v[:, s].contiguous(), pos[s].clone(),
                         first[s].clone(), *args, seq_tokens=tokens[s].clone())
    assert all(torch.equal(x, y) for x, y in zip(_planes(whole), _planes(parts)))
