"""GPU parity of the prefill's causal attention and its per-row log-sum-exp
(the forward pass whose log-sum-exp Appendix A.7 hands to the score), and of
the single-pass score (Algorithm 2) fed with that log-sum-exp.

Tolerances, from the arithmetic: logits are exact bf16 products summed in
fp32, and the row sums and the log-sum-exp stay in fp32, so the log-sum-exp
is held to 1e-4 absolute.  The output rounds each probability to bf16
(relative error at most 2^-9) before the value product and the finished row
to bf16 once more, so |O - O_ref| <= 2^-9 max|V| + 2^-9 |O_ref| <= 2^-8 max|V|;
the test allows 4.5e-3 max|V|."""

import sys

import numpy as np
import pytest
import torch

from oracle import causal_attention, proxy_scores_grouped
from synth import custom, make_grouped_layer, make_layer
from tests._parity import check_scores

pytestmark = pytest.mark.gpu

nacl = pytest.importorskip("paper_2408_03675_amd.nacl")

LSE_ATOL = 1e-4
O_TOL = 4.5e-3  # times max|V|


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nacl.load_library()


def _f64(t):
    return t.detach().cpu().double().numpy()


def _check(out, lse, q, k, v, s, g, label, rows=None):
    Or, lr = causal_attention(_f64(q), _f64(k), _f64(v), s, q_group=g, rows=rows)
    o = _f64(out) if rows is None else _f64(out[:, :, rows])
    l = _f64(lse) if rows is None else _f64(lse[:, :, rows])
    assert np.isfinite(o).all() and np.isfinite(l).all(), label
    vmax = float(_f64(v).__abs__().max())
    err_o = np.abs(o - Or).max()
    err_l = np.abs(l - lr).max()
    assert err_o <= O_TOL * vmax, f"{label}: output off by {err_o} (max|V| {vmax})"
    assert err_l <= LSE_ATOL, f"{label}: log-sum-exp off by {err_l}"
    return err_o / vmax, err_l


CASES = [
    # name, B, H (K/V heads), q_group, L, D, injected sinks and heavy hitters
    ("d128_ragged300", 1, 2, 1, 300, 128, False),
    ("d64_ragged257", 2, 2, 1, 257, 64, False),
    ("gqa4_d128_640", 1, 2, 4, 640, 128, False),
    ("one_row", 1, 1, 1, 1, 128, False),
    ("one_tile64", 1, 3, 1, 64, 128, False),
    ("tiles_129", 1, 1, 2, 129, 64, False),
    ("sinks_1000", 1, 2, 1, 1000, 128, True),
    ("sinks_d64_777", 2, 1, 1, 777, 64, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_attention_matches_oracle(case):
    name, B, H, g, L, D, inject = case
    print("attention case", name, file=sys.stderr, flush=True)
    P = max(1, L // 50)
    w = custom(name, B, H, L, D, P, dtype="bf16", inject=inject, data_seed=len(name) * 11)
    q, k, v = make_grouped_layer(w, g, device="cuda") if g > 1 else make_layer(w, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    _check(out, lse, q, k, v, prob.c.sm_scale, g, name)


def test_attention_strided_layout():
    """Q, K, V as [B, L, H, D] buffers viewed as [B, H, L, D] (row stride H * D)."""
    B, H, g, L, D = 2, 2, 2, 333, 128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    qb = torch.randn((B, L, H * g, D), generator=gen, device="cuda").to(torch.bfloat16)
    kb = torch.randn((B, L, H, D), generator=gen, device="cuda").to(torch.bfloat16)
    vb = torch.randn((B, L, H, D), generator=gen, device="cuda").to(torch.bfloat16)
    q, k, v = qb.transpose(1, 2), kb.transpose(1, 2), vb.transpose(1, 2)
    pos = list(range(7, L, 41))
    prob = nacl.Problem.from_tensors(q, k, v, pos)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    _check(out, lse, q, k, v, prob.c.sm_scale, g, "strided")


@pytest.mark.parametrize("g", [1, 4])
def test_single_pass_score_from_attention_lse(g):
    """Appendix A.7's pipeline: the attention's log-sum-exp at the proxy rows
    feeds the score's column reduction (Algorithm 2), which must give the
    oracle's F; the gathered rows must equal the full log-sum-exp's."""
    B, H, L, D, P = 2, 2, 2500, 128, 40
    w = custom(f"a7_{g}", B, H, L, D, P, dtype="bf16", inject=(g == 1), data_seed=77 + g)
    q, k, v = make_grouped_layer(w, g, device="cuda") if g > 1 else make_layer(w, device="cuda")
    pos_dev = torch.tensor(w.proxy_pos, dtype=torch.int32, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos, proxy_pos_dev=pos_dev)
    out, lse, lp = nacl.attention(prob, q, k, v, lse_proxy=True)
    F = nacl.score(prob, q, k, nacl.workspace(prob), lse=lp)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(lp.cpu().numpy(), lse[:, :, w.proxy_pos].cpu().numpy())
    Fr, lr = proxy_scores_grouped(_f64(q), _f64(k), w.proxy_pos, prob.c.sm_scale, g)
    assert np.abs(_f64(lp) - lr).max() <= LSE_ATOL
    check_scores(F.cpu().numpy(), Fr, f"a7_g{g}")


def test_attention_prefill_32k_sampled_rows():
    """The 32k prefill layer at full size (B = 4, H = 32, L = 32768, D = 128,
    bf16, injected sinks and heavy hitters): every row's log-sum-exp is
    finite, and sampled rows of sampled heads match the oracle."""
    B, H, L, D, P = 4, 32, 32768, 128, 128
    w = custom("prefill_32k_attention", B, H, L, D, P, dtype="bf16", inject=True, data_seed=3)
    q, k, v = make_layer(w, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    assert torch.isfinite(lse).all()
    rows = np.array([0, 1, 127, 128, 4095, 16384, 32766, 32767])
    for b, h in ((0, 0), (1, 17), (3, 31)):
        sl = slice(h, h + 1)
        _check(out[b:b + 1, sl], lse[b:b + 1, sl], q[b:b + 1, sl], k[b:b + 1, sl], v[b:b + 1, sl],
               prob.c.sm_scale, 1, f"32k b{b} h{h}", rows=rows)


def test_attention_d64_grouped_4k_sampled_rows():
    """Head dim 64 with two query heads per K/V head over 4097 tokens (33
    query tiles of 128 rows per head, the last holding one row): sampled rows
    of every head, and every log-sum-exp finite."""
    B, H, g, L, D, P = 2, 4, 2, 4097, 64, 64
    w = custom("gqa_d64_4k", B, H, L, D, P, dtype="bf16", data_seed=41)
    q, k, v = make_grouped_layer(w, g, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    assert torch.isfinite(lse).all()
    rows = np.array([0, 63, 64, 127, 128, 255, 256, 2048, 4095, 4096])
    _check(out, lse, q, k, v, prob.c.sm_scale, g, "gqa_d64_4k", rows=rows)


@pytest.mark.parametrize("L,g,scale", [(128, 1, 0.05), (256, 8, None), (2, 1, 2.0)])
def test_attention_tile_multiples_and_scales(L, g, scale):
    """Exact multiples of the 128-row and 64-key tiles, eight query heads per
    K/V head, two rows, and logit scales other than 1/sqrt(D)."""
    B, H, D = 1, 2, 128
    w = custom(f"edge_{L}_{g}", B, H, L, D, 1, dtype="bf16", data_seed=L + g)
    q, k, v = make_grouped_layer(w, g, device="cuda") if g > 1 else make_layer(w, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos, sm_scale=scale)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    _check(out, lse, q, k, v, prob.c.sm_scale, g, f"edge L{L} g{g}")


def test_attention_rejects_unsupported():
    q = torch.zeros((1, 1, 16, 64), dtype=torch.float32, device="cuda")
    prob = nacl.Problem.from_tensors(q, q, q, [3])
    with pytest.raises(nacl.NaclError) as e:
        nacl.attention(prob, q, q, q, out=torch.empty_like(q))
    assert e.value.status == 2
    qb = torch.zeros((1, 1, 16, 64), dtype=torch.bfloat16, device="cuda")
    prob = nacl.Problem.from_tensors(qb, qb, qb, [3])
    with pytest.raises(nacl.NaclError):
        nacl.attention(prob, qb, qb, qb, lse_proxy=True)  # no proxy_pos_dev


# Edges of the work-groups of 128 rows, tiles of 64 keys, heads that 8 XCDs do
# not divide, and groups of heads sharing K and V.
TILE_CASES = [
    # B, H, q_group, L, D
    (1, 1, 1, 63, 128), (1, 1, 1, 65, 64), (1, 3, 1, 127, 128), (2, 5, 1, 193, 64),
    (1, 9, 1, 320, 128), (1, 4, 2, 255, 64),
    (1, 67, 1, 65, 128), (2, 9, 4, 192, 64), (1, 64, 1, 256, 128), (4, 17, 1, 129, 64),
    (1, 33, 1, 321, 128), (1, 9, 8, 257, 64), (1, 16, 1, 1025, 128),
]


@pytest.mark.parametrize("B,H,g,L,D", TILE_CASES)
def test_attention_tile_edges(B, H, g, L, D):
    print("attention tiles", B, H, g, L, D, file=sys.stderr, flush=True)
    w = custom("edges", B, H, L, D, 1, dtype="bf16", data_seed=B + 3 * H + L)
    q, k, v = make_grouped_layer(w, g, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    _check(out, lse, q, k, v, prob.c.sm_scale, g, f"{B}x{H}x{g} L{L} D{D}")


@pytest.mark.parametrize("D", (64, 128))
@pytest.mark.parametrize("H", (2, 64))
def test_attention_rising_logits(D, H):
    """Keys whose logits pass every earlier one by far (the reference of the
    exponentials has to move, tile after tile and by more than one step), and
    rows whose first tile holds the largest by far.  Logits reach a few
    hundred, so the log-sum-exp is held to 1e-4 plus 2^-22 of its size (two
    roundings of a product and a sum in fp32)."""
    L = 700
    w = custom("rise", 1, H, L, D, 1, dtype="bf16", data_seed=D + H)
    q, k, v = make_grouped_layer(w, 1, device="cuda")
    q = q.abs()
    up = torch.ones(L, device="cuda")
    for j, x in ((70, 3.0), (200, 9.0), (201, 10.0), (400, 30.0), (640, 60.0)):
        up[j] = x
    k = (k.abs() * up[None, None, :, None]).to(torch.bfloat16)
    k[:, 1::2] = k[:, 1::2].flip(2)
    prob = nacl.Problem.from_tensors(q, k, v, w.proxy_pos)
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    Or, lr = causal_attention(_f64(q), _f64(k), _f64(v), prob.c.sm_scale)
    assert np.isfinite(_f64(out)).all()
    assert np.abs(_f64(out) - Or).max() <= O_TOL * np.abs(_f64(v)).max()
    assert (np.abs(_f64(lse) - lr) <= LSE_ATOL + 2.0 ** -22 * np.abs(lr)).all()


# Long rows of 128 with at least 256 work-groups of 256 rows: waves of 64 rows.
# Whole tiles, one row in the last wave, waves without rows, grouped heads.
LONG_CASES = [
    # B, H, q_group, L, [B, L, H, D] layout
    (1, 11, 1, 6144, False), (2, 3, 2, 6145, True), (1, 11, 1, 6335, False), (1, 2, 8, 6207, True),
]


@pytest.mark.parametrize("B,H,g,L,blhd", LONG_CASES)
def test_attention_long_rows(B, H, g, L, blhd):
    """64 consecutive rows (each of a wave's rows is rescaled by its own
    factors), the first, middle and last rows."""
    print("attention long", B, H, g, L, file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L + H)
    shape = [(B, L, H * g, 128), (B, L, H, 128), (B, L, H, 128)] if blhd else [(B, H * g, L, 128), (B, H, L, 128), (B, H, L, 128)]
    q, k, v = (torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16) for s in shape)
    if blhd:
        q, k, v = (x.transpose(1, 2) for x in (q, k, v))
    prob = nacl.Problem.from_tensors(q, k, v, [L - 1])
    out, lse, _ = nacl.attention(prob, q, k, v)
    torch.cuda.synchronize()
    assert torch.isfinite(lse).all()
    again, lse2, _ = nacl.attention(prob, q, k, v)
    assert torch.equal(out, again) and torch.equal(lse, lse2)
    rows = np.unique(np.concatenate([np.arange(0, 300, 37), np.arange(2944, 3008), [L - 66, L - 65, L - 64, L - 2, L - 1]]))
    heads = sorted({0, H // 2, H - 1})
    for h in heads:
        qs = slice(h * g, h * g + g)
        _check(out[:, qs], lse[:, qs], q[:, qs], k[:, h:h + 1], v[:, h:h + 1], prob.c.sm_scale, g, f"long h{h}", rows=rows)


@pytest.mark.parametrize("H,L,D", [(2, 700, 64), (2, 700, 128), (11, 6144, 128)])
def test_attention_largest_probability_is_exact(H, L, D):
    """A key whose logit lies less than 2^8 above the first tile's carries all of
    the output (the other value rows are zeros).  Against the row's own maximum
    its probability is 1, exact in bf16, so the output is w V with one rounding
    to bf16: within 2^-8 of its size, and 2^-14 for the fp32 logit and sum.  A
    probability of up to 2^8 would be rounded as well, by up to 2^-8 more."""
    at = 70
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + H)
    q = torch.zeros((1, H, L, D), device="cuda")
    k, v = torch.zeros_like(q), torch.zeros_like(q)
    q[..., 0] = 1.0 + 4.5 * torch.rand((1, H, L), generator=gen, device="cuda")  # logits of 1.4 .. 7.9 in base 2
    k[:, :, at, 0] = 1.0
    v[:, :, at] = torch.randn((1, H, D), generator=gen, device="cuda") + 2.0
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    prob = nacl.Problem.from_tensors(q, k, v, [L - 1], sm_scale=1.0)
    out, lse, _ = nacl.attention(prob, q, k, v)
    rows = torch.arange(at, L, device="cuda", dtype=torch.float64)
    e = q[0, :, at:, 0].double().exp()
    l = e + rows  # row r sees r other keys, whose logits are 0
    ref = (e / l)[..., None] * v[0, :, at].double()[:, None]
    err = ((out[0, :, at:].double() - ref).abs() / ref.abs().clamp_min(1e-30)).max().item()
    assert err <= 2.0 ** -8 + 2.0 ** -14, err / 2.0 ** -8
    assert (lse[0, :, at:].double() - l.log()).abs().max().item() <= LSE_ATOL


@pytest.mark.parametrize("H,L", [(2, 700), (11, 6144)])
def test_attention_nan_key_stays_in_its_rows(H, L):
    """A key of NaNs makes the rows that see it NaN and no others."""
    at = 333
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H)
    q, k, v = (torch.randn((1, H, L, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    k[:, 1, at] = float("nan")
    prob = nacl.Problem.from_tensors(q, k, v, [L - 1])
    out, lse, _ = nacl.attention(prob, q, k, v)
    assert torch.isfinite(out[:, 0]).all() and torch.isfinite(out[:, 2:]).all()
    assert torch.isfinite(out[:, 1, :at]).all() and torch.isfinite(lse[:, 1, :at]).all()
    assert torch.isnan(out[:, 1, at:]).all() and torch.isnan(lse[:, 1, at:]).all()
