"""GPU parity of the score kernels that larger bf16 launches and row counts
choose, at the edges of their ranges: keys held in registers with both passes
in one work-group (up to one 512-key chunk per CU, two for 65 to 128 rows), keys in
registers with the passes queued (D = 64 over 128 rows, 257 to 512 rows), the
split kernel (65 to 128 rows), the block kernel (129 to 256 rows), and the split
kernels with shortened items.

The scores are compared with the float64 oracle within 1e-3 relative, the bound
of every score test: logits are float32 sums of at most 128 exact bf16
products, |logit| < 2^5 here, so their error of 2^-24 * 128 * 2^5 stays below
2.5e-4, and an exponential's relative error is that of its argument."""

import sys
import zlib

import numpy as np
import pytest
import torch

from oracle import SAMPLE_SOFTMAX, proxy_scores, proxy_scores_grouped
from synth import custom, make_layer
from tests._parity import check_scores

pytestmark = pytest.mark.gpu

nacl = pytest.importorskip("paper_2408_03675_amd.nacl")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nacl.load_library()


def _np(t):
    return t.detach().float().cpu().numpy()


KERNELS = {"held": "score_keys_kernel, both passes", "queued": "score_keys_kernel", "split": "score_split_kernel",
           "block": "score_block_kernel", "wide": "score_split_wide_kernel", "tiles": "score_kernel",
           "few": "score_rows_logits_kernel"}


def check_kernel(name, prob):
    """The case runs the kernel that its name says."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert nacl.score_kernel(prob, cus=cus) == KERNELS[name.split("_")[0]], name


def suffix(L, P):
    return list(range(L - P, L))


def spread(L, P):
    return sorted({int(x) for x in np.linspace(0, L - 1, P)})


CASES = [
    # name, B, H, L, D, positions
    # both passes in one work-group: rows about a multiple of 32 and of the row buffers
    ("held_17_rows", 1, 17, 1025, 128, suffix(1025, 17)),
    ("tiles_32_rows_few_chunks", 1, 3, 513, 128, suffix(513, 32)),
    ("held_32_rows_d64", 2, 2, 511, 64, spread(511, 32)),
    ("held_32_rows", 1, 33, 511, 128, spread(511, 32)),
    ("held_33_rows", 1, 2, 512, 128, spread(512, 33)),
    ("held_127_rows_d64", 1, 2, 1025, 64, suffix(1025, 127)),
    ("held_129_rows", 1, 2, 1537, 128, spread(1537, 129)),
    ("held_256_rows_early_d64", 1, 2, 2100, 64, list(range(256))),
    ("held_257_rows", 2, 1, 1500, 128, suffix(1500, 257)),
    ("held_512_rows", 1, 2, 2047, 128, spread(2047, 512)),
    ("held_512_rows_d64", 1, 1, 1100, 64, suffix(1100, 512)),
    # two chunks per work-group: the first one's keys and rows are read again
    ("held_twice_65_rows", 2, 50, 1300, 128, suffix(1300, 65)),
    ("held_twice_128_rows_d64", 1, 170, 1030, 64, spread(1030, 128)),
    # beyond those: tiles, split with short items, block, keys with queued passes, wide
    ("tiles_64_rows", 2, 86, 1100, 128, suffix(1100, 64)),
    ("tiles_24_rows_few_chunks", 1, 4, 2048, 128, spread(2048, 24)),
    ("tiles_16_rows_d64_few_chunks", 1, 3, 513, 64, suffix(513, 16)),
    ("tiles_24_rows", 2, 45, 1100, 128, spread(1100, 24)),
    ("tiles_28_rows_d64", 2, 45, 1100, 64, suffix(1100, 28)),
    ("tiles_60_rows_d64", 1, 90, 1045, 64, list(range(30, 90))),
    ("tiles_128_rows_d64", 1, 175, 1100, 64, spread(1100, 128)),
    ("tiles_513_rows_d64", 1, 2, 1100, 64, suffix(1100, 513)),
    # long items, later ones past the last proxy
    ("split_128_items_past_the_proxies", 1, 100, 5000, 128, list(range(200, 328))),
    ("split_128_short_items", 2, 90, 1100, 128, spread(1100, 128)),
    ("split_65_rows", 2, 130, 1100, 128, suffix(1100, 65)),
    ("split_97_rows", 3, 61, 1500, 128, spread(1500, 97)),
    ("split_127_rows_early", 2, 90, 1300, 128, list(range(300, 427))),
    ("block_129_rows", 1, 90, 1100, 128, suffix(1100, 129)),
    ("block_200_rows_early", 2, 45, 1300, 128, list(range(100, 300))),
    ("block_256_rows", 1, 60, 2300, 128, spread(2300, 256)),
    ("queued_129_rows_d64", 1, 90, 1100, 64, suffix(1100, 129)),
    ("queued_300_rows", 2, 45, 1100, 128, spread(1100, 300)),
    ("queued_511_rows_d64", 1, 90, 1045, 64, list(range(30, 541))),
    ("queued_long_items", 1, 130, 8200, 64, suffix(8200, 150)),
    # 257 to 512 rows of D = 128 on both sides of the line between keys and wide:
    # 385 and more rows past one item per CU, padded to 512 in the wide kernel
    ("queued_384_rows", 4, 130, 700, 128, suffix(700, 384)),
    ("wide_385_rows", 4, 130, 700, 128, spread(700, 385)),
    ("wide_450_rows_early", 3, 130, 800, 128, list(range(100, 550))),
    ("wide_512_rows", 2, 140, 1100, 128, suffix(1100, 512)),
    ("queued_512_rows", 1, 90, 1100, 128, suffix(1100, 512)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_score_paths_match_oracle(case):
    """The scores, with the library's and the caller's log-sum-exp; the scores
    a second time (bit-reproducible, on a used workspace); a whole eviction's
    keep set against the selection on those scores."""
    name, B, H, L, D, pos = case
    print("score path", name, file=sys.stderr, flush=True)
    w = custom(name, B, H, L, D, len(pos), dtype="bf16", data_seed=zlib.crc32(name.encode()) % 1000)
    q, k, v = make_layer(w, 0, device="cuda")
    prob = nacl.Problem.from_tensors(q, k, v, pos)
    check_kernel(name, prob)
    ws = nacl.workspace(prob)
    F = nacl.score(prob, q, k, ws).clone()
    again = nacl.score(prob, q, k, ws)
    assert torch.equal(F, again)
    heads = range(0, H, 1 if L < 4000 else 33)  # the oracle over the long case's heads takes minutes
    qn, kn = _np(q[:, heads]), _np(k[:, heads])
    Fr, lse = proxy_scores(qn, kn, pos, prob.c.sm_scale)
    check_scores(_np(F[:, heads]), Fr, name)
    total = _np(F).astype(np.float64).sum(-1)
    np.testing.assert_allclose(total, len(pos), rtol=1e-5)
    if len(heads) == H:
        given = nacl.score(prob, q, k, ws, lse=torch.from_numpy(lse.astype(np.float32)).cuda())
        check_scores(_np(given), Fr, name + " caller lse")
    C = len(pos) + 40
    Fe, keep, _, _ = nacl.evict(prob, q, k, v, C, 30, SAMPLE_SOFTMAX, 11, 2, ws=ws)
    assert torch.equal(Fe, F)
    assert torch.equal(keep, nacl.select(prob, F, C, 30, SAMPLE_SOFTMAX, 11, 2, ws=ws))


@pytest.mark.parametrize("H,P,D", [(90, 129, 128), (90, 300, 128), (180, 128, 128), (180, 70, 128), (90, 200, 64)])
def test_score_paths_large_logits(H, P, D):
    """One key far above the others of its chunk (about 180 above in the
    exponent): references taken from other keys overflow, and every path has
    to end with that key's mass."""
    L = 1100
    g = torch.Generator(device="cuda").manual_seed(11)
    q = torch.randn((1, H, L, D), generator=g, device="cuda")
    k = torch.randn((1, H, L, D), generator=g, device="cuda")
    pos = suffix(L, P)
    q[:, :, L - P:] += 2.0 * (128 / D) ** 0.5
    k[:, ::2, 400] = 8.0
    k[:, 1::2, 700] = 8.0
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    prob = nacl.Problem.from_tensors(q, k, k, pos)
    F = nacl.score(prob, q, k, nacl.workspace(prob))
    heads = [0, 1, H // 2, H - 1]
    Fr, _ = proxy_scores(_np(q[:, heads]), _np(k[:, heads]), pos, prob.c.sm_scale)
    check_scores(_np(F[:, heads]), Fr, "large logits")
    np.testing.assert_allclose(_np(F).astype(np.float64).sum(-1), P, rtol=1e-5)


@pytest.mark.parametrize("H,P,D,dt", [(90, 24, 128, "bf16"), (90, 64, 128, "bf16"), (90, 20, 64, "bf16"), (90, 60, 64, "bf16"),
                                      (180, 100, 64, "bf16"), (3, 600, 64, "bf16"), (3, 40, 128, "f32"), (3, 30, 64, "f32"),
                                      (3, 60, 64, "f32")])
def test_tile_kernel_large_logits(H, P, D, dt):
    """The same for each form of the per-wave-tile kernel (two, four and eight
    blocks of rows, both types), which recomputes such a range's sums against
    its exact maximum."""
    L = 1100
    g = torch.Generator(device="cuda").manual_seed(12)
    q, k = (torch.randn((1, H, L, D), generator=g, device="cuda") for _ in range(2))
    pos = suffix(L, P)
    q[:, :, L - P:] += 2.0 * (128 / D) ** 0.5
    k[:, ::2, 400] = 8.0
    k[:, 1::2, 700 if P < 400 else 480] = 8.0
    q, k = (x.to(torch.bfloat16 if dt == "bf16" else torch.float32) for x in (q, k))
    prob = nacl.Problem.from_tensors(q, k, k, pos)
    check_kernel("tiles", prob)
    F = nacl.score(prob, q, k, nacl.workspace(prob))
    heads = [0, 1, H - 1]
    Fr, _ = proxy_scores(_np(q[:, heads]), _np(k[:, heads]), pos, prob.c.sm_scale)
    check_scores(_np(F[:, heads]), Fr, "large logits")
    np.testing.assert_allclose(_np(F).astype(np.float64).sum(-1), P, rtol=1e-5)


GROUPED_CASES = [
    # name, B, H (K/V heads), q_group, L, D, P: [B, L, H, D] layout, rows = q_group * P
    ("held_192", 2, 4, 4, 3000, 128, 48), ("held_90_d64", 2, 3, 3, 1037, 64, 30),
    ("split_100", 2, 90, 2, 1100, 128, 50), ("block_200", 2, 45, 4, 1100, 128, 50), ("queued_320", 1, 90, 8, 1100, 128, 40),
    ("queued_200_d64", 1, 90, 4, 1100, 64, 50), ("wide_560", 1, 4, 8, 1100, 128, 70), ("wide_416", 1, 400, 8, 600, 128, 52),
    ("tiles_48", 2, 45, 2, 1100, 128, 24), ("tiles_28_d64", 1, 90, 2, 1100, 64, 14), ("tiles_100_d64", 1, 180, 4, 1100, 64, 25),
    ("tiles_560_d64", 1, 2, 8, 1100, 64, 70),
]


@pytest.mark.parametrize("case", GROUPED_CASES, ids=[c[0] for c in GROUPED_CASES])
def test_score_paths_grouped_and_strided(case):
    """Grouped query heads with rows of Q and K that lie between other heads'
    rows, with the library's and the caller's log-sum-exp."""
    name, B, H, g, L, D, P = case
    print("grouped path", name, file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(P + H)
    q = torch.randn((B, L, H * g, D), generator=gen, device="cuda").to(torch.bfloat16).permute(0, 2, 1, 3)
    k = torch.randn((B, L, H, D), generator=gen, device="cuda").to(torch.bfloat16).permute(0, 2, 1, 3)
    pos = spread(L - 3, P)
    prob = nacl.Problem.from_tensors(q, k, k, pos)
    check_kernel(name, prob)
    ws = nacl.workspace(prob)
    F = nacl.score(prob, q, k, ws)
    heads = sorted({0, H // 2, H - 1})
    Fr, lse = proxy_scores_grouped(_np(q.unflatten(1, (H, g))[:, heads].flatten(1, 2)), _np(k[:, heads]), pos, prob.c.sm_scale, g)
    check_scores(_np(F[:, heads]), Fr, name)
    np.testing.assert_allclose(_np(F).astype(np.float64).sum(-1), len(pos) * g, rtol=1e-5)
    given = torch.zeros((B, H, g, len(pos)), device="cuda")
    given[:, heads] = torch.from_numpy(lse.astype(np.float32)).cuda().reshape(B, len(heads), g, len(pos))
    F = nacl.score(prob, q, k, ws, lse=given.flatten(1, 2).contiguous())
    check_scores(_np(F[:, heads]), Fr, name + " caller lse")


ODD_CASES = [
    # name, H, L, D, P, dtype: one case per kernel
    ("held_200", 2, 1100, 128, 200, "bf16"), ("held_40_d64", 2, 1100, 64, 40, "bf16"), ("queued_300", 90, 1100, 128, 300, "bf16"),
    ("queued_200_d64", 90, 1100, 64, 200, "bf16"), ("split_128", 180, 1100, 128, 128, "bf16"),
    ("block_200", 90, 1100, 128, 200, "bf16"), ("wide_600", 90, 1100, 128, 600, "bf16"), ("wide_400", 520, 700, 128, 400, "bf16"),
    ("split_100", 180, 1100, 128, 100, "bf16"), ("tiles_50", 180, 1100, 128, 50, "bf16"), ("tiles_100_d64", 180, 1100, 64, 100, "bf16"), ("tiles_f32", 3, 700, 64, 40, "f32"), ("few_rows", 3, 700, 128, 12, "bf16"),
]


@pytest.mark.parametrize("case", ODD_CASES, ids=[c[0] for c in ODD_CASES])
def test_score_odd_row_stays_below_its_position(case):
    """A query row of NaNs, and caller log-sum-exps of -inf, NaN and +inf: the
    scores of keys past the row's position are those of the other rows."""
    name, H, L, D, P, dt = case
    g = torch.Generator(device="cuda").manual_seed(5)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    q, k = (torch.randn((1, H, L, D), generator=g, device="cuda").to(dtype) for _ in range(2))
    pos = spread(L - 90, P)
    P = len(pos)
    prob = nacl.Problem.from_tensors(q, k, k, pos)
    check_kernel(name, prob)
    ws = nacl.workspace(prob)
    heads = [0, H - 1]
    Fr, lse = proxy_scores(_np(q[:, heads]), _np(k[:, heads]), pos, prob.c.sm_scale)
    qn, kn = _np(q[0, heads]).astype(np.float64), _np(k[0, heads]).astype(np.float64)

    def others(r):
        """The scores without row r."""
        a = np.einsum("hd,hld->hl", qn[:, pos[r]], kn) * prob.c.sm_scale
        return Fr[0] - np.where(np.arange(L)[None] <= pos[r], np.exp(a - lse[0, :, r, None]), 0.0)

    r = P // 2
    odd = q.clone()
    odd[:, :, pos[r]] = float("nan")
    F = _np(nacl.score(prob, odd, k, ws))[0, heads]
    check_scores(F[:, pos[r] + 1:], others(r)[:, pos[r] + 1:], name + " NaN row")
    assert np.isnan(F[:, :pos[r] + 1]).all()

    full = torch.zeros((1, H, P), device="cuda")
    full[:, heads] = torch.from_numpy(lse.astype(np.float32)).cuda()
    for r, x in ((P // 3, -np.inf), (P // 2, np.nan), (2 * P // 3, np.inf)):
        given = full.clone()
        given[:, :, r] = float(x)
        F = _np(nacl.score(prob, q, k, ws, lse=given))[0, heads]
        want = others(r)
        check_scores(F[:, pos[r] + 1:], want[:, pos[r] + 1:], f"{name} log-sum-exp {x}")
        if x == np.inf:
            assert (np.abs(F - want) <= 1e-3 * Fr[0]).all()  # the row adds nothing
        else:
            assert (np.isposinf if x == -np.inf else np.isnan)(F[:, :pos[r] + 1]).all()
