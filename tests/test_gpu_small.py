"""GPU parity, element by element, at sizes the oracle finishes in seconds: several tiles
and ragged tails, MHA and GQA, both head sizes, both modes, and the degenerate cases."""
import numpy as np
import pytest
import torch

import ems_inputs
from oracle import ems_ref
from paper_2412_08521_amd import binding as B
from gpu_util import (RTOL, RTOL_MERGE, assert_dest_valid, assert_rel, check_band, dev_tensor, is_sorted_unique,
                      ref_params, score_forms, score_products)

pytestmark = pytest.mark.gpu

MODES = [B.EMS_BF16, B.EMS_F32]

# (batch, q_heads, kv_heads, head_dim, seq_len, window)
SCORE_SHAPES = [
    (1, 2, 2, 64, 1, 1),
    (1, 2, 1, 128, 31, 7),
    (2, 4, 2, 64, 777, 33),        # ragged tail, GQA
    (1, 2, 2, 128, 1000, 32),      # several key tiles + tail
    (1, 4, 1, 128, 300, 300),      # window == length
    (1, 8, 2, 128, 2500, 64),      # several row chunks in pass 2
    (1, 2, 2, 64, 4099, 70),       # window straddles a chunk boundary
    (1, 6, 3, 128, 6000, 64),      # heads that do not divide over the XCDs
]


def _log(*a):
    print(*a, flush=True)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", SCORE_SHAPES)
def test_score_matches_oracle(shape, mode):
    b, hq, hkv, d, n, w = shape
    _log("score", shape, "mode", mode)
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=n + d)
    p = B.EmsParams(b, hq, hkv, d, n, w, dtype=mode)
    q, k = dev_tensor(inp.q, mode), dev_tensor(inp.k, mode)
    s_glo, s_loc, lse = B.ems_global_local_score(p, q, k, want_lse=True)
    torch.cuda.synchronize()
    o_glo, o_loc, o_lse = ems_ref.score(ref_params(p), inp.f32("q"), inp.f32("k"), want_lse=True)
    rtol = RTOL[mode]
    assert_rel(s_glo.cpu().numpy(), o_glo, rtol, "s_glo")
    assert_rel(s_loc.cpu().numpy(), o_loc, rtol, "s_loc")
    np.testing.assert_allclose(lse.cpu().numpy(), o_lse, rtol=0, atol=2e-5 if mode == B.EMS_F32 else 2e-2)
    # invariants that hold at any size: weights of every row sum to one
    G = hq // hkv
    np.testing.assert_allclose(s_glo.sum(-1).cpu().numpy(), G * n, rtol=1e-4)
    np.testing.assert_allclose(s_loc.sum(-1).cpu().numpy(), G * w, rtol=1e-4)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("group", [1, 2, 3, 4])
def test_score_every_remainder_of_interior_stages(group, mode):
    """The pipelined loops of both passes take whole trips of 4 stages (2 in f32 mode); what does not fill
    a trip goes through the masked loop.  Lengths 32 apart walk through every remainder, for every group size
    (the trip counts stages of all q-heads of a group), plus one ragged length."""
    lengths = [1312 + 32 * i for i in range(6 if mode == B.EMS_F32 else 4)] + [1333]
    for d in ([64, 128] if group in (1, 3) else [64]):
        for n in lengths:
            _log("score remainders: group", group, "d", d, "n", n, "mode", mode)
            inp = ems_inputs.small(1, group, 1, d, n, seed=n + group)
            p = B.EmsParams(1, group, 1, d, n, 32, dtype=mode)
            s_glo, s_loc, lse = B.ems_global_local_score(p, dev_tensor(inp.q, mode), dev_tensor(inp.k, mode), want_lse=True)
            torch.cuda.synchronize()
            o_glo, o_loc, o_lse = ems_ref.score(ref_params(p), inp.f32("q"), inp.f32("k"), want_lse=True)
            assert_rel(s_glo.cpu().numpy(), o_glo, RTOL[mode], f"s_glo n={n} d={d}")
            assert_rel(s_loc.cpu().numpy(), o_loc, RTOL[mode], f"s_loc n={n} d={d}")
            np.testing.assert_allclose(lse.cpu().numpy(), o_lse, rtol=0, atol=2e-5 if mode == B.EMS_F32 else 2e-2)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [
    (1, 1030, 1030, 64, 70, 5),      # more heads than resident waves: one stretch per head
    (1, 40, 40, 64, 1111, 100),      # stretches that end inside the diagonal stages and inside the window
    (2, 16, 2, 128, 1537, 600),      # eight q-heads per kv-head; the window spans several stretches and key tiles
    (5, 5, 5, 64, 257, 64),          # second unit of one row; most stretches shorter than their lead
    (1, 96, 32, 64, 3000, 33),       # three q-heads per kv-head, several units per stretch
])
def test_score_even_deal(shape, mode):
    """Launches that are cut by stages: every part of every unit is counted once, whatever a stretch's
    ends fall on.  Tolerance: the stated bars."""
    b, hq, hkv, d, n, w = shape
    _log("even deal", shape, "mode", mode)
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=n + w)
    p = B.EmsParams(b, hq, hkv, d, n, w, dtype=mode)
    s_glo, s_loc, lse = B.ems_global_local_score(p, dev_tensor(inp.q, mode), dev_tensor(inp.k, mode), want_lse=True)
    o_glo, o_loc, o_lse = ems_ref.score(ref_params(p), inp.f32("q"), inp.f32("k"), want_lse=True)
    assert_rel(s_glo.cpu().numpy(), o_glo, RTOL[mode], "s_glo")
    assert_rel(s_loc.cpu().numpy(), o_loc, RTOL[mode], "s_loc")
    np.testing.assert_allclose(lse.cpu().numpy(), o_lse, rtol=0, atol=2e-5 if mode == B.EMS_F32 else 2e-2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [600, 1300, 1400, 1470, 1500, 1660, 1750, 1850])
def test_score_short_float32_stretches(n, d):
    """Stretches of four to eight stages (8 heads over 2): either number of the ring's two slots, the first looks at the sums."""
    test_score_even_deal((1, 8, 2, d, n, 40), B.EMS_F32)


@pytest.mark.parametrize("what", ["wide", "tiny", "huge", "infinite"])
@pytest.mark.parametrize("d", [64, 128])
def test_score_float32_values_that_do_not_split(what, d):
    """The float32 passes multiply bf16 pieces of their operands; values without three such pieces are redone by float32
    products.  "wide": elements over 40 binary orders, which do split.  "tiny" and "huge": some of one side's elements times
    2^-112 or 2^70, the other side's the other way.  "infinite": keys of -inf where every query is positive (logits of -inf: no weight),
    and rows next to float32's largest value.  Tolerance: the stated bars."""
    b, hq, hkv, n, w = 1, 4, 2, 700, 40
    gen = np.random.default_rng(len(what) + d)
    q, k = (gen.standard_normal((b, h, n, d)).astype(np.float32) for h in (hq, hkv))
    if what == "wide":
        q *= 2.0 ** gen.integers(-40, 1, q.shape).astype(np.float32)
    elif what == "tiny":
        q[..., :8] *= np.float32(2.0 ** 112); k[..., :8] *= np.float32(2.0 ** -112)
    elif what == "huge":
        q[..., 5] *= np.float32(2.0 ** -70); k[..., 5] *= np.float32(2.0 ** 70)
    else:
        q[..., 3] = np.abs(q[..., 3]) + np.float32(0.1)
        k[:, 0, 100:400:7, 3] = -np.inf
        q[..., 9] *= np.float32(2.0 ** -124)
        k[:, 1, ::5, 9] = np.float32(-3.4e38)
    p = B.EmsParams(b, hq, hkv, d, n, w, dtype=B.EMS_F32)
    s_glo, s_loc, lse = B.ems_global_local_score(p, torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), want_lse=True)
    o_glo, o_loc, o_lse = ems_ref.score(ref_params(p), q, k, want_lse=True)
    live = ~np.isneginf(k).any(-1)
    assert (s_glo.cpu().numpy()[~live] == 0).all() and (s_loc.cpu().numpy()[~live] == 0).all()
    assert_rel(s_glo.cpu().numpy()[live], o_glo[live], RTOL[B.EMS_F32], "s_glo")
    assert_rel(s_loc.cpu().numpy()[live], o_loc[live], RTOL[B.EMS_F32], "s_loc")
    np.testing.assert_allclose(lse.cpu().numpy(), o_lse, rtol=0, atol=2e-5)


@pytest.mark.parametrize("d", [64, 128])
def test_score_float32_is_as_close_as_float32_products(d):
    """Row log-sum-exp of heavy-tailed logits against 64 bits, rms over all rows of four seeds.  Bound: what float32 products
    left is 6.9e-7 (64) and 7.7e-7 (128), of which the two roundings of the result are 3.9e-7 (base 2, then natural, at 8 to 16:
    2^-20 / sqrt(12) each, the first times ln 2; half of the rows' lie in 16 to 32 in base 2); the six products of pieces in the
    order of the columns 6.1e-7 and 6.7e-7, those with a lower piece first 4.6e-7 for both."""
    n = 3000
    p = B.EmsParams(1, 8, 2, d, n, 32, dtype=B.EMS_F32)
    causal = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
    square = 0.0
    for seed in range(4):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        randn = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
        u = randn(2, 1, d)
        u /= u.norm(dim=-1, keepdim=True)
        heavy = torch.empty((2, n, 1), device="cuda").exponential_(1.0, generator=gen)
        k = (randn(2, n, d) + 0.25 * d ** 0.5 * heavy * u)[None]
        q = (randn(2, 4, n, d) + 4.0 * u[:, None]).reshape(1, 8, n, d)
        lse = B.ems_attention_lse(p, q, k)
        for h in range(8):
            logits = (q[0, h].double() @ k[0, h // 4].double().T * d ** -0.5).masked_fill(~causal, -torch.inf)
            square += float((lse[0, h].double() - torch.logsumexp(logits, -1)).square().mean()) / 32
    assert square ** 0.5 < 5.3e-7


def _check_reached(glo, loc, lse, o_glo, o_loc, o_lse, nan_row, nan_is_key, no_weight):
    """One kv-head's scores and row log-sum-exp against the oracle's on finite values, apart from what a NaN reaches: of query row
    `nan_row` (second q-head, which is before the window) its own log-sum-exp and the columns up to it, of key `nan_row` every later
    row and through them every column.  Columns `no_weight` are keys of -inf."""
    rows, cols, local = np.ones(lse.shape, bool), np.ones(len(glo), bool), np.ones(len(glo), bool)
    if nan_row is not None and nan_is_key:
        rows[:, nan_row:] = cols[:] = local[:] = False
    elif nan_row is not None:
        rows[1, nan_row] = cols[:nan_row + 1] = False
    # (a row of nothing but NaN logits has no maximum: where its parts are combined, its log-sum-exp is that of no parts)
    assert not np.isfinite(lse[~rows]).any() and np.isnan(glo[~cols]).all() and np.isnan(loc[~local]).all()
    np.testing.assert_allclose(lse[rows], o_lse[rows], rtol=0, atol=2e-5)
    if no_weight is not None:
        assert (glo[no_weight] == 0).all() and (loc[no_weight] == 0).all()
        cols[no_weight] = local[no_weight] = False
    for got, ref, at, what in ((glo, o_glo, cols, "s_glo"), (loc, o_loc, local, "s_loc")):
        if at.any():
            assert_rel(got[at], ref[at], RTOL[B.EMS_F32], what)


@pytest.mark.parametrize("d", [64, 128])
def test_score_float32_values_that_do_not_split_in_queues(d):
    """The same where the passes take whole items from queues.  One (batch, kv-head) pair each: keys of 2^70, keys of -inf, a query
    row of NaN (of which only the rows' own weights are lost), a key of NaN.  Against the oracle, for NaN on finite values in their
    place, what they reach apart; tolerance: the stated bars."""
    hkv, g, n, w, row = 400, 2, 2503, 70, 1777
    p = B.EmsParams(1, g * hkv, hkv, d, n, w, dtype=B.EMS_F32)
    assert score_forms(p) == ("queue", "queue")
    _log("values that do not split, in queues", d)
    gen = torch.Generator(device="cuda").manual_seed(d)
    k = torch.randn((1, hkv, n, d), device="cuda", generator=gen)
    q = torch.randn((1, g * hkv, n, d), device="cuda", generator=gen)
    huge, inf, nan_q, nan_k = 3, 8, 201, 399
    k[0, huge, :, 5] *= 2.0 ** 70; q[0, g * huge:g * huge + g, :, 5] *= 2.0 ** -70
    q[0, g * inf:g * inf + g, :, 3] = q[0, g * inf:g * inf + g, :, 3].abs() + 0.1
    k[0, inf, 100:2000:97, 3] = -torch.inf
    kept = {h: (q[:, g * h:g * h + g].cpu().numpy(), k[:, h:h + 1].cpu().numpy()) for h in (huge, inf, nan_q, nan_k, 0)}
    q[0, g * nan_q + 1, row, 7] = torch.nan
    k[0, nan_k, row, 7] = torch.nan
    s_glo, s_loc, lse = (x.cpu().numpy() for x in B.ems_global_local_score(p, q, k, want_lse=True))
    for h, (qh, kh) in kept.items():
        o_glo, o_loc, o_lse = ems_ref.score(ems_ref.RefParams(1, g, 1, d, n, w), qh, kh, want_lse=True)
        _check_reached(s_glo[0, h], s_loc[0, h], lse[0, g * h:g * h + g], o_glo[0, 0], o_loc[0, 0], o_lse[0],
                       row if h in (nan_q, nan_k) else None, h == nan_k, slice(100, 2000, 97) if h == inf else None)


def test_score_float32_values_that_do_not_split_cost_float32_products():
    """Items with such values go by float32 products from there on, at 1.8 times the time of the pieces: one key of -inf, which
    every later row of its head streams, takes a score call to no more than that (1.80 measured; 2.9 when items began anew without a pipeline)."""
    p = B.EmsParams(1, 32, 8, 128, 6000, 64, 256, dtype=B.EMS_F32)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k = (torch.randn((1, h, 6000, 128), device="cuda", generator=gen) for h in (32, 8))
    q[..., 3] = q[..., 3].abs() + 0.1
    odd = k.clone()
    odd[0, 0, 100, 3] = -torch.inf
    ws = torch.empty(B.ems_workspace_bytes(p)[0], dtype=torch.uint8, device="cuda")
    out = tuple(torch.empty((1, 8, 6000), device="cuda") for _ in range(2))

    def us(keys):
        times = []
        for _ in range(12):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            B.ems_global_local_score(p, q, keys, ws=ws, out=out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    us(k)
    assert us(odd) < 2.3 * us(k)


@pytest.mark.parametrize("mode,shape,forms", [
    (B.EMS_BF16, (1, 32, 16, 128, 8177, 90), ("deal", "deal")),      # 132 stages a stretch: every set-aside of both passes
    (B.EMS_BF16, (1, 256, 8, 64, 2040, 100), ("block", "deal")),     # two row tiles per wave, one pair per XCD
    (B.EMS_BF16, (1, 64, 2, 128, 8177, 90), ("block", "deal")),      # the q-heads of a row tile together
    (B.EMS_BF16, (1, 64, 8, 128, 8177, 90), ("block", "deal")),
    (B.EMS_BF16, (1, 80, 8, 128, 8177, 33), ("queue", "deal")),
    (B.EMS_BF16, (1, 320, 8, 128, 2040, 100), ("queue", "deal")),
    (B.EMS_BF16, (1, 500, 5, 64, 1270, 33), ("queue", "deal")),
    (B.EMS_BF16, (1, 804, 804, 64, 5003, 1500), ("queue", "block")),  # pairs that do not divide over the XCDs
    (B.EMS_BF16, (1, 804, 804, 128, 5003, 40), ("queue", "block")),
    (B.EMS_BF16, (2, 800, 400, 64, 5003, 1500), ("queue", "queue")),  # the window crosses a row chunk's end
    (B.EMS_BF16, (1, 800, 800, 128, 5003, 907), ("queue", "queue")),
    (B.EMS_F32, (1, 804, 804, 64, 2503, 600), ("queue", "block")),
    (B.EMS_F32, (1, 804, 402, 128, 2503, 600), ("queue", "block")),
    (B.EMS_F32, (1, 800, 800, 64, 2503, 600), ("queue", "queue")),
    (B.EMS_F32, (1, 800, 400, 128, 2503, 70), ("queue", "queue")),
])
def test_score_whole_items(mode, shape, forms):
    """Launches whose passes take whole items, by block index or from queues, at ragged lengths: first, middle and last
    (batch, kv-head) pair against the oracle (heads are independent).  Tolerance: the stated bars."""
    b, hq, hkv, d, n, w = shape
    g = hq // hkv
    _log("whole items", mode, shape)
    p = B.EmsParams(b, hq, hkv, d, n, w, dtype=mode)
    assert score_forms(p) == forms
    if mode == B.EMS_BF16:
        assert score_products(p) == (16 if n == 8177 and hkv >= 8 else 32)       # (of the listed ones)
    gen = torch.Generator(device="cuda").manual_seed(n + hq)
    k = torch.randn((b, hkv, n, d), device="cuda", generator=gen).to(torch.bfloat16).to(p.torch_dtype)
    q = torch.empty((b, hq, n, d), dtype=p.torch_dtype, device="cuda")
    for h in range(hkv):
        q[:, h * g:(h + 1) * g] = torch.randn((b, g, n, d), device="cuda", generator=gen).to(torch.bfloat16).to(p.torch_dtype)
    s_glo, s_loc, lse = B.ems_global_local_score(p, q, k, want_lse=True)
    np.testing.assert_allclose(s_glo.sum(-1).cpu().numpy(), g * n, rtol=1e-4)
    np.testing.assert_allclose(s_loc.sum(-1).cpu().numpy(), g * w, rtol=1e-4)
    for i, h in ((0, 0), (b - 1, hkv // 2), (b - 1, hkv - 1)):
        ref = ems_ref.RefParams(1, g, 1, d, n, w)
        o = ems_ref.score(ref, q[i:i + 1, h * g:(h + 1) * g].float().cpu().numpy(), k[i:i + 1, h:h + 1].float().cpu().numpy(), want_lse=True)
        assert_rel(s_glo[i, h].cpu().numpy(), o[0][0, 0], RTOL[mode], "s_glo")
        assert_rel(s_loc[i, h].cpu().numpy(), o[1][0, 0], RTOL[mode], "s_loc")
        np.testing.assert_allclose(lse[i, h * g:(h + 1) * g].cpu().numpy(), o[2][0], rtol=0, atol=2e-5 if mode == B.EMS_F32 else 2e-2)


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("group,n", [(3, 3232), (3, 3264), (3, 3296), (3, 3328), (3, 3233), (1, 3360), (4, 3231), (4, 3200)])
def test_score_by_the_smaller_products(group, n, far):
    """Launches of 70 to 1024 stages of 32 x 256 per resident wave, 3200 rows and more, at head size 128, which run by 16x16x32
    products: every remainder of the trips, ragged ends.  far: later logits exceed the first stage's by more than the float range, so that parts are
    redone with a running maximum (bounds as in the test below).  First and last kv-head against the oracle."""
    b, hkv, d, w = 4, 36 // group, 128, 40
    _log("smaller products", group, n, far)
    p = B.EmsParams(b, 36, hkv, d, n, w)
    assert score_products(p) == 16
    gen = torch.Generator(device="cuda").manual_seed(n)
    k = torch.randn((b, hkv, n, d), device="cuda", generator=gen).to(torch.bfloat16)
    q = torch.randn((b, 36, n, d), device="cuda", generator=gen).to(torch.bfloat16)
    if far:
        k[:, :, 700:] *= 64.0                                # exact in bf16
    s_glo, s_loc, lse = B.ems_global_local_score(p, q, k, want_lse=True)
    rtol = 4e-4 if far else 1e-5                             # (without far: the float32 mode's bar, the products of bf16 inputs are exact)
    for i, h in ((0, 0), (b - 1, hkv - 1)):
        ref = ems_ref.RefParams(1, group, 1, d, n, w)
        o = ems_ref.score(ref, q[i:i + 1, h * group:(h + 1) * group].float().cpu().numpy(), k[i:i + 1, h:h + 1].float().cpu().numpy(), want_lse=True)
        assert_rel(s_glo[i, h].cpu().numpy(), o[0][0, 0], rtol, "s_glo")
        assert_rel(s_loc[i, h].cpu().numpy(), o[1][0, 0], rtol, "s_loc")
        np.testing.assert_allclose(lse[i, h * group:(h + 1) * group].cpu().numpy(), o[2][0], rtol=2e-6, atol=1e-4 if far else 2e-5)


@pytest.mark.parametrize("b,d,n,products", [(4, 128, 3233, 16), (1, 128, 3100, 32), (1, 64, 3233, 32)])
def test_score_infinite_and_nan_values(b, d, n, products):
    """16-bit calls, one (batch, kv-head) pair each: keys of -inf where every query is positive (logits of -inf: no weight), a query
    row of NaN (only its own weights are lost), a key of NaN (every later row's).  Against the oracle, for NaN on finite values in
    their place, what they reach apart.  Tolerance: the float32 mode's bar, the products of bf16 inputs are exact."""
    hkv, g, w, row = 12, 3, 40, 1777
    p = B.EmsParams(b, g * hkv, hkv, d, n, w)
    assert score_products(p) == products
    _log("infinite and NaN", b, d, n)
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    k = torch.randn((b, hkv, n, d), device="cuda", generator=gen).to(torch.bfloat16)
    q = torch.randn((b, g * hkv, n, d), device="cuda", generator=gen).to(torch.bfloat16)
    plain, inf, nan_q, nan_k = 0, 4, 7, 11
    q[0, g * inf:g * inf + g, :, 3] = q[0, g * inf:g * inf + g, :, 3].abs() + 0.125
    k[0, inf, 100:2000:97, 3] = -torch.inf
    kept = {h: (q[:1, g * h:g * h + g].float().cpu().numpy(), k[:1, h:h + 1].float().cpu().numpy()) for h in (plain, inf, nan_q, nan_k)}
    q[0, g * nan_q + 1, row, 7] = torch.nan
    k[0, nan_k, row, 7] = torch.nan
    s_glo, s_loc, lse = (x.cpu().numpy() for x in B.ems_global_local_score(p, q, k, want_lse=True))
    for h, (qh, kh) in kept.items():
        o_glo, o_loc, o_lse = ems_ref.score(ems_ref.RefParams(1, g, 1, d, n, w), qh, kh, want_lse=True)
        _check_reached(s_glo[0, h], s_loc[0, h], lse[0, g * h:g * h + g], o_glo[0, 0], o_loc[0, 0], o_lse[0],
                       row if h in (nan_q, nan_k) else None, h == nan_k, slice(100, 2000, 97) if h == inf else None)


@pytest.mark.parametrize("mode", MODES)
def test_score_first_stage_far_below_the_others(mode):
    """The first stage of a part gives the reference exponent; here later logits exceed it by far more than
    the float range, so the sums overflow and the parts are redone with a running maximum.  A weight is
    2^x with |x| up to 4 * 64 * 1.44 = 370 formed in float32: relative error a few times 370 * 2^-23 * ln 2 = 3e-5."""
    b, hq, hkv, d, n, w = 1, 4, 2, 64, 1500, 40
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=21)
    kf = inp.f32("k").copy()
    kf[:, :, 700:] *= 64.0                                   # exact in bf16
    q, k = dev_tensor(inp.q, mode), torch.from_numpy(kf).cuda().to(torch.float32 if mode == B.EMS_F32 else torch.bfloat16)
    p = B.EmsParams(b, hq, hkv, d, n, w, dtype=mode)
    s_glo, s_loc, lse = B.ems_global_local_score(p, q, k, want_lse=True)
    o_glo, o_loc, o_lse = ems_ref.score(ref_params(p), inp.f32("q"), kf, want_lse=True)
    assert_rel(s_glo.cpu().numpy(), o_glo, max(RTOL[mode], 4e-4), "s_glo")
    assert_rel(s_loc.cpu().numpy(), o_loc, max(RTOL[mode], 4e-4), "s_loc")
    np.testing.assert_allclose(lse.cpu().numpy(), o_lse, rtol=2e-6, atol=1e-4)


@pytest.mark.parametrize("mode", MODES)
def test_score_reference_follows_the_stages(mode):
    """The first 32 keys lie 100 powers of two below the others: no redo, but an exponent formed against them is
    rounded at 2^-18 (2.6e-6 of its weight).  Logits are exact in float32 and at most 12 in base 2; what is left
    is the rounding of small exponents, of 2^x and of the log-sum-exp itself: 1.2e-6 together."""
    b, h, d, n = 1, 16, 64, 256
    rng = np.random.default_rng(3)
    qf, kf = np.zeros((b, h, n, d), np.float32), np.zeros((b, h, n, d), np.float32)
    qf[..., 0], qf[..., 1] = 1.0, 2.0 ** -11
    kf[..., 0] = rng.integers(-8, 9, (b, h, n)) / 4.0
    kf[:, :, :32, 0] = -100.0
    kf[..., 1] = rng.integers(128, 256, (b, h, n)) / 256.0          # exact in bf16
    p = B.EmsParams(b, h, h, d, n, 16, dtype=mode, softmax_scale=float(np.float32(np.log(2.0))))
    q, k = (dev_tensor(ems_inputs.f32_to_bf16_bits(x), mode) for x in (qf, kf))
    lse = B.ems_attention_lse(p, q, k)
    _, _, o_lse = ems_ref.score(ref_params(p), qf, kf, want_lse=True)
    np.testing.assert_allclose(lse.cpu().numpy()[:, :, 32:], o_lse[:, :, 32:], rtol=0, atol=1.2e-6)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [(1, 4, 2, 64, 4100), (1, 2, 1, 128, 3000)])
def test_score_sums_do_not_drift(shape, mode):
    """Column sums against 64 bits, as a 2-norm (one heavy key takes most of it).  A chain of 512 additions in
    float32 is off by 512^0.5 * 2^-24 / 3 = 4.5e-7 of its sum; sixteen such chains make a column's: 1.1e-7,
    and three times that is allowed.  A stretch summed in one go is outside it."""
    b, hq, hkv, d, n = shape
    rng = np.random.default_rng(n)
    u = rng.standard_normal((b, hkv, 1, d))
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    kf = rng.standard_normal((b, hkv, n, d)) + 0.75 * d ** 0.5 * rng.exponential(1.0, (b, hkv, n, 1)) * u
    qf = rng.standard_normal((b, hq, n, d)) + 4.0 * np.repeat(u, hq // hkv, axis=1)
    kb, qb = (ems_inputs.f32_to_bf16_bits(x.astype(np.float32)) for x in (kf, qf))
    p = B.EmsParams(b, hq, hkv, d, n, 32, dtype=mode)
    s_glo, _ = B.ems_global_local_score(p, dev_tensor(qb, mode), dev_tensor(kb, mode))
    o_glo, _ = ems_ref.score(ref_params(p), ems_inputs.bf16_bits_to_f32(qb), ems_inputs.bf16_bits_to_f32(kb))[:2]
    err = np.linalg.norm(s_glo.cpu().numpy() - o_glo) / np.linalg.norm(o_glo)
    assert err <= 3.4e-7, err


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("heads", [8, 1600])                  # cut by stages; work queues
def test_score_two_halves_leave_the_float_range_together(heads, mode):
    """Two keys of one interior stage, one in each half of the wave, lie 127.5 powers of two above the reference:
    each half's sum is inside the float range, their total is not.  log2 of the row sum is 64.5 (two weights of
    2^63.5) or, before the keys, -64 + log2(i + 1): float32 rounding of a number below 128, twice."""
    d, n = 64, 1111
    qf, kf = np.zeros((1, 1, n, d), np.float32), np.zeros((1, 1, n, d), np.float32)
    qf[..., 0], kf[..., 0] = 1.0, -64.0
    kf[:, :, [64, 68], 0] = 63.5
    p = B.EmsParams(1, heads, heads, d, n, 16, dtype=mode, softmax_scale=float(np.float32(np.log(2.0))))
    q, k = (dev_tensor(ems_inputs.f32_to_bf16_bits(x), mode).expand(1, heads, n, d).contiguous() for x in (qf, kf))
    s_glo, _, lse = B.ems_global_local_score(p, q, k, want_lse=True)
    want = -64.0 + np.log2(np.arange(1.0, n + 1))
    want[64:68], want[68:] = 63.5, 64.5
    np.testing.assert_allclose(lse.cpu().numpy() / np.log(2.0), np.broadcast_to(want, lse.shape), rtol=0, atol=2.0 ** -16)
    np.testing.assert_allclose(s_glo.sum(-1).cpu().numpy(), n, rtol=1e-4)


def test_score_custom_scale_and_large_logits():
    """Logits of magnitude ~40: the running maximum of pass 1 has to do its job."""
    b, hq, hkv, d, n, w = 1, 2, 2, 128, 600, 16
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=77, scale=2.0)
    for mode in MODES:
        p = B.EmsParams(b, hq, hkv, d, n, w, softmax_scale=0.3, dtype=mode)
        s_glo, s_loc = B.ems_global_local_score(p, dev_tensor(inp.q, mode), dev_tensor(inp.k, mode))
        o_glo, o_loc = ems_ref.score(ref_params(p), inp.f32("q"), inp.f32("k"))
        assert_rel(s_glo.cpu().numpy(), o_glo, max(RTOL[mode], 1e-4), "s_glo")
        assert_rel(s_loc.cpu().numpy(), o_loc, max(RTOL[mode], 1e-4), "s_loc")


def test_score_zero_queries_is_harmonic():
    """Closed form (uniform rows): s_glo[j] = G * sum_{i>=j} 1/(i+1), on the GPU itself."""
    b, hq, hkv, d, n, w = 1, 4, 2, 128, 1500, 40
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=5)
    p = B.EmsParams(b, hq, hkv, d, n, w)
    q = torch.zeros((b, hq, n, d), dtype=torch.bfloat16, device="cuda")
    s_glo, s_loc = B.ems_global_local_score(p, q, dev_tensor(inp.k, B.EMS_BF16))
    inv = 1.0 / np.arange(1, n + 1)
    tail = np.cumsum(inv[::-1])[::-1]
    np.testing.assert_allclose(s_glo[0, 0].cpu().numpy(), 2 * tail, rtol=1e-5)
    np.testing.assert_allclose(s_loc[0, 1].cpu().numpy(),
                               2 * np.array([tail[max(j, n - w)] for j in range(n)]), rtol=1e-5)


def test_score_runs_are_bit_identical_and_heads_independent():
    b, hq, hkv, d, n, w = 2, 8, 2, 128, 1300, 32
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=9)
    p = B.EmsParams(b, hq, hkv, d, n, w)
    q, k = dev_tensor(inp.q, B.EMS_BF16), dev_tensor(inp.k, B.EMS_BF16)
    a = B.ems_global_local_score(p, q, k)
    c = B.ems_global_local_score(p, q, k)
    assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
    p1 = B.EmsParams(1, 4, 1, d, n, w)
    one = B.ems_global_local_score(p1, q[1:, 4:].contiguous(), k[1:, 1:].contiguous())
    assert torch.equal(one[0][0, 0], a[0][1, 1]) and torch.equal(one[1][0, 0], a[1][1, 1])


# ---------------------------------------------------------------------------- select
SELECT_SHAPES = [
    # (bh, n, w, budget, r, pool)
    (3, 1024, 32, 64, 0.5, 7),
    (2, 4099, 32, 256, 0.5, 7),
    (2, 3000, 64, 128, 3.0, 1),
    (1, 200, 10, 190, 5.0, 3),       # N_tbm clamped, everything kept or merged
    (1, 70000, 64, 2048, 0.5, 7),    # long sequences: chunks of 2048 positions over many blocks per head
    (2, 33, 1, 2, 0.0, 1),
    (3, 8192, 32, 100, 0.5, 7),      # the longest sequence the one-block kernel takes
    (3, 8193, 32, 100, 0.5, 7),      # the shortest the chunked kernels take: a second chunk of one position
    (2, 20000, 2047, 4000, 1.0, 5),  # window ends inside a chunk; a large budget (many candidates)
    (1, 12288, 4096, 8000, 0.5, 63), # whole chunks inside the window; widest pooling kernel
    (2, 10000, 8, 9000, 0.5, 1),     # nearly everything kept: the candidate list is almost the whole head
    (1, 1000003, 64, 3000, 0.5, 7),  # 489 chunks: more than one chunk per thread when the factor is formed
    (1, 1 << 22, 64, 5000, 1.0, 7),  # the longest sequence the interface takes: 2048 chunks
]


# sizes where the select's and the merge's ways of working change: candidate lists of up to and over 4096 and
# 16384 tokens, whole lists in ties; one and several rows per merge wave, a TBM list of more than one piece,
# a zero class shared by several blocks, larger token tiles of the destination search
# (bh, n, w, budget, r, d)
MERGE_EDGES = [
    (2, 9000, 16, 2066, 1.0, 64),        # 2050 centres in 9 slices, 2066 tokens: the zero class in four blocks
    (8, 20000, 64, 4100, 1.0, 128),      # more than 4096 candidates; rows of a wave by lane group
    (1, 40000, 32, 9000, 0.6, 64),       # 14400 candidates; 5400 tokens: two pieces, one row per wave
    (1, 70000, 32, 12000, 0.5, 64),      # over 16384 candidates
    (33, 1500, 100, 700, 1.1, 128),      # heads that do not divide over the XCDs
    (8, 33000, 64, 2500, 2.0, 128),      # 5000 tokens, token tiles of 64
]


@pytest.mark.parametrize("tau", [-2.0, 0.3, 2.0])
@pytest.mark.parametrize("shape", MERGE_EDGES)
def test_select_and_merge_where_the_ways_change(shape, tau):
    """Index sets against the oracle's partition of the GPU's keys, destinations and rows against the
    oracle's: the stated bars."""
    bh, n, w, budget, r, d = shape
    _log("select and merge", shape, tau)
    p = B.EmsParams(1, bh, bh, d, n, w, budget, merge_ratio=r, tau=tau)
    glo, loc = _rand_scores(bh, n, w, seed=budget)
    imp, tbm, pooled = B.ems_select(p, torch.from_numpy(glo).cuda(), torch.from_numpy(loc).cuda(), want_pooled=True)
    x_imp, x_tbm = ems_ref.partition(ref_params(p), pooled.cpu().numpy().astype(np.float64))
    assert (imp.cpu().numpy() == x_imp).all() and (tbm.cpu().numpy() == x_tbm).all()
    if bh > 8:
        rows = [0, 1, bh // 2, bh - 1]
    else:
        rows = [0, bh - 1]
    gen = torch.Generator().manual_seed(n)
    k, v = (torch.randn((1, bh, n, d), generator=gen).to(torch.bfloat16) for _ in range(2))
    hot = x_imp[0, 0, 3]                                 # one centre of the first head that many tokens join
    k[0, 0, torch.from_numpy(x_tbm[0, 0, ::3].astype(np.int64))] = k[0, 0, int(hot)].clone()
    out = {name: t.cpu() for name, t in B.ems_evict_merge(p, k.cuda(), v.cuda(), imp, tbm).items()}
    sub = ems_ref.RefParams(1, len(rows), len(rows), d, n, w, budget=budget, merge_ratio=r, tau=tau)
    kf, vf = k[:, rows].float().numpy(), v[:, rows].float().numpy()
    s_imp, s_tbm = x_imp[:, rows], x_tbm[:, rows]
    dest = out["tbm_dest"].numpy()[:, rows]
    if tau == 0.3:
        o_dest, _ = ems_ref.dest(sub, kf, s_imp, s_tbm)[:2]
        assert assert_dest_valid(dest, o_dest, kf, s_imp, s_tbm, tau, budget) <= dest.size // 100
    else:
        assert (dest == budget).all() if tau > 1 else (dest < s_imp.shape[-1]).all()
    k_ref, v_ref, kept, cnt = ems_ref.merge(sub, kf, vf, s_imp, s_tbm, dest)
    assert (out["slot_count"].numpy()[:, rows] == cnt).all() and (out["kept_pos"].numpy()[:, rows] == kept).all()
    for got, ref in ((out["k_out"], k_ref), (out["v_out"], v_ref)):
        got = got.float().numpy()[:, rows]
        rms = np.sqrt((ref.astype(np.float64) ** 2).mean(-1, keepdims=True))
        assert (np.abs(got - ref) <= 2e-2 * np.maximum(np.abs(ref), rms) + 1e-6).all()


def _rand_scores(bh, n, w, seed):
    rng = np.random.default_rng(seed)
    glo = (rng.random((1, bh, n)) ** 4 * 5 + 1e-3).astype(np.float32)
    loc = (rng.random((1, bh, n)) ** 6 * w / n * 20).astype(np.float32)
    return glo, loc


@pytest.mark.parametrize("shape", SELECT_SHAPES)
def test_select_matches_oracle(shape):
    bh, n, w, nb, r, pk = shape
    _log("select", shape)
    glo, loc = _rand_scores(bh, n, w, n)
    p = B.EmsParams(1, bh, bh, 128, n, w, nb, merge_ratio=r, pool_kernel=pk)
    imp, tbm, pooled = B.ems_select(p, torch.from_numpy(glo).cuda(), torch.from_numpy(loc).cuda(),
                                    want_pooled=True)
    imp, tbm, pooled = imp.cpu().numpy(), tbm.cpu().numpy(), pooled.cpu().numpy()
    rp = ref_params(p)
    o_pooled, o_imp, o_tbm = ems_ref.select(rp, glo, loc)
    assert_rel(pooled, o_pooled, 1e-5, "pooled score")
    # integer work is bit-exact given the keys: oracle partition of the GPU's own keys
    x_imp, x_tbm = ems_ref.partition(rp, pooled.astype(np.float64))
    np.testing.assert_array_equal(imp, x_imp)
    np.testing.assert_array_equal(tbm, x_tbm)
    # and against the full fp64 oracle with a band at the cuts
    for h in range(bh):
        check_band(imp[0, h], tbm[0, h], o_pooled[0, h], n - w, 1e-5)
        assert is_sorted_unique(imp[0, h]) and (tbm.shape[-1] == 0 or is_sorted_unique(tbm[0, h]))


@pytest.mark.parametrize("n", [1023, 1025, 2048, 2049, 3071, 3073, 4096, 4097, 5120, 5121, 6144, 6145, 7168, 7169, 8191])
def test_select_every_item_count(n):
    """One to eight positions per thread of the one-block kernel, its last ones in use and not."""
    test_select_matches_oracle((2, n, 32, 300, 0.75, 7))
    test_select_exact_ties_rank_by_position(n, 4)


@pytest.mark.parametrize("levels", [4, 1])
@pytest.mark.parametrize("n", [5000, 20000])
def test_select_exact_ties_rank_by_position(n, levels):
    """Scores quantised to a few levels (or all equal): almost everything ties, on the chunked path the
    candidate list is then most of the head; pooling off so the keys are exactly the inputs and the
    index sets must equal the oracle's exactly."""
    bh, w, nb = 2, 16, 300
    _log("select ties", n, levels)
    rng = np.random.default_rng(1)
    loc = rng.integers(1, levels + 1, (1, bh, n)).astype(np.float32)
    glo = np.full((1, bh, n), 1e-6, np.float32)      # aligned s_glo never wins the max
    p = B.EmsParams(1, bh, bh, 64, n, w, nb, merge_ratio=2.0, pool_kernel=1)
    imp, tbm = B.ems_select(p, torch.from_numpy(glo).cuda(), torch.from_numpy(loc).cuda())
    _, o_imp, o_tbm = ems_ref.select(ref_params(p), glo, loc)
    np.testing.assert_array_equal(imp.cpu().numpy(), o_imp)
    np.testing.assert_array_equal(tbm.cpu().numpy(), o_tbm)


# ---------------------------------------------------------------------------- evict-merge
MERGE_SHAPES = [
    # (b, hkv, d, n, w, budget, r)
    (1, 2, 64, 700, 16, 48, 1.5),
    (2, 2, 128, 1500, 32, 256, 0.5),
    (1, 3, 128, 4096, 64, 128, 3.0),
    (1, 1, 128, 3000, 32, 512, 2.0),       # centre list searched in slices
    (1, 2, 128, 12000, 32, 1100, 5.0),     # 5500 to-be-merged tokens: two LDS pieces in the merge
    (1, 1, 64, 9000, 16, 2300, 0.6),       # several stages of centres per slice
]


def _random_partition(p, seed):
    n_imp, n_tbm = B.ems_partition_sizes(p)
    rng = np.random.default_rng(seed)
    imp = np.empty((p.batch, p.kv_heads, n_imp), np.int32)
    tbm = np.empty((p.batch, p.kv_heads, n_tbm), np.int32)
    for b in range(p.batch):
        for h in range(p.kv_heads):
            perm = rng.permutation(p.seq_len - p.window)
            imp[b, h] = np.sort(perm[:n_imp])
            tbm[b, h] = np.sort(perm[n_imp:n_imp + n_tbm])
    return imp, tbm


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("tau", [0.6, 0.22, -2.0, 2.0])
@pytest.mark.parametrize("shape", MERGE_SHAPES)
def test_evict_merge_matches_oracle(shape, tau, mode):
    b, hkv, d, n, w, nb, r = shape
    _log("evict_merge", shape, "tau", tau, "mode", mode)
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=nb)
    # plant near-duplicates so that tau = 0.6 merges something
    kf = inp.f32("k").copy()
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=r, tau=tau, dtype=mode)
    imp, tbm = _random_partition(p, seed=nb + 1)
    rng = np.random.default_rng(3)
    for bb in range(b):
        for h in range(hkv):
            for t in tbm[bb, h, ::5]:
                c = imp[bb, h, rng.integers(0, imp.shape[-1])]
                kf[bb, h, t] = 0.8 * kf[bb, h, c] + 0.45 * kf[bb, h, t]
    inp.k = ems_inputs.f32_to_bf16_bits(kf)
    kf, vf = inp.f32("k"), inp.f32("v")

    out = B.ems_evict_merge(p, dev_tensor(inp.k, mode), dev_tensor(inp.v, mode),
                            torch.from_numpy(imp).cuda(), torch.from_numpy(tbm).cuda())
    out = {k_: v_.float().cpu().numpy() if v_.is_floating_point() else v_.cpu().numpy()
           for k_, v_ in out.items()}
    rp = ref_params(p)
    ref = ems_ref.evict_merge(rp, kf, vf, imp, tbm)
    n_imp, n_tbm = B.ems_partition_sizes(p)

    # destinations: equal except where the decision is inside float32 noise
    np.testing.assert_allclose(out["tbm_sim"], ref["tbm_sim"], rtol=0, atol=5e-6)
    np.testing.assert_allclose(out["k_norm"], ref["k_norm"], rtol=1e-6)
    n_diff = assert_dest_valid(out["tbm_dest"], ref["tbm_dest"], kf, imp, tbm, tau, nb)
    assert n_diff < 0.01 * ref["tbm_dest"].size
    # stage isolation: the oracle's average for the GPU's own destinations
    k_ref, v_ref, kept_ref, cnt_ref = ems_ref.merge(rp, kf, vf, imp, tbm, out["tbm_dest"])
    np.testing.assert_array_equal(out["kept_pos"], kept_ref)
    np.testing.assert_array_equal(out["slot_count"], cnt_ref)
    rtol = RTOL_MERGE[mode]
    for name, got, want in (("k_out", out["k_out"], k_ref), ("v_out", out["v_out"], v_ref)):
        # per-row floor: 1e-2 of the row's RMS
        rms = np.sqrt((want ** 2).mean(-1, keepdims=True))
        err = np.abs(got - want) / np.maximum(np.abs(want), 1e-2 * np.maximum(rms, 1e-30))
        assert err.max() <= rtol, f"{name}: {err.max():.3e}"
    # rows nobody merged into, and the local rows, are bit-exact copies
    alone = cnt_ref[..., :n_imp] == 1
    src_k, src_v = (kf, vf)
    for bb in range(b):
        for h in range(hkv):
            rows = np.nonzero(alone[bb, h])[0]
            np.testing.assert_array_equal(out["k_out"][bb, h, rows], src_k[bb, h, imp[bb, h, rows]])
            np.testing.assert_array_equal(out["v_out"][bb, h, rows], src_v[bb, h, imp[bb, h, rows]])
            np.testing.assert_array_equal(out["k_out"][bb, h, n_imp:nb], src_k[bb, h, n - w:])
            np.testing.assert_array_equal(out["v_out"][bb, h, n_imp:nb], src_v[bb, h, n - w:])
    if tau >= 1:
        assert (out["tbm_dest"] == nb).all() and (out["slot_count"][..., -1] == n_tbm).all()
    if tau <= -1:
        assert (out["tbm_dest"] < n_imp).all() and (out["slot_count"][..., -1] == 0).all()
    if tau == 0.6:
        assert (out["tbm_dest"] < n_imp).any() and (out["tbm_dest"] == nb).any()


def test_evict_merge_many_centres():
    """12000 class centres (the destination search cuts them into 16 slices of three rounds each) and 6016
    to-be-merged tokens (two LDS pieces in the merge), checked like the small shapes."""
    test_evict_merge_matches_oracle((1, 1, 128, 40000, 32, 12032, 0.5), 0.22, B.EMS_BF16)


def test_merge_ratio_zero_is_bit_exact_gather():
    b, hkv, d, n, w, nb = 1, 2, 128, 900, 32, 100
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=4)
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=0.0)
    imp, tbm = _random_partition(p, seed=2)
    assert tbm.shape[-1] == 0
    k, v = dev_tensor(inp.k, B.EMS_BF16), dev_tensor(inp.v, B.EMS_BF16)
    out = B.ems_evict_merge(p, k, v, torch.from_numpy(imp).cuda(), torch.from_numpy(tbm).cuda())
    for h in range(hkv):
        kept = np.concatenate([imp[0, h], np.arange(n - w, n)])
        np.testing.assert_array_equal(out["kept_pos"][0, h].cpu().numpy(), kept)
        assert torch.equal(out["k_out"][0, h, :nb], k[0, h, torch.from_numpy(kept).cuda()])
        assert torch.equal(out["v_out"][0, h, :nb], v[0, h, torch.from_numpy(kept).cuda()])
        assert (out["k_out"][0, h, nb] == 0).all() and (out["v_out"][0, h, nb] == 0).all()
    assert (out["slot_count"][..., :-1] == 1).all() and (out["slot_count"][..., -1] == 0).all()


# ---------------------------------------------------------------------------- end to end
@pytest.mark.parametrize("mode", MODES)
def test_tiny_config_end_to_end(mode):
    """BASELINE config 1 (4 heads, D 64, N 1024, W 32, budget 64, r 0.5), full chain with
    every stage also checked in isolation on the GPU's own upstream output."""
    w = ems_inputs.WORKLOADS["tiny"]
    inp = ems_inputs.generate(w)
    for tau in (0.6, 0.3):
        p = B.EmsParams(w.batch, w.q_heads, w.kv_heads, w.head_dim, w.seq_len, w.window, w.budget,
                        merge_ratio=w.merge_ratio, tau=tau, pool_kernel=w.pool_kernel, dtype=mode)
        q, k, v = (dev_tensor(getattr(inp, x), mode) for x in "qkv")
        s_glo, s_loc = B.ems_global_local_score(p, q, k)
        imp, tbm, pooled = B.ems_select(p, s_glo, s_loc, want_pooled=True)
        out = B.ems_evict_merge(p, k, v, imp, tbm)
        out2 = B.ems_evict_merge(p, k, v, imp, tbm)
        for name in out:
            assert torch.equal(out[name], out2[name]), name        # reproducible bit for bit
        rp = ref_params(p)
        qf, kf, vf = inp.f32("q"), inp.f32("k"), inp.f32("v")
        o_glo, o_loc = ems_ref.score(rp, qf, kf)
        rtol = RTOL[mode]
        assert_rel(s_glo.cpu().numpy(), o_glo, rtol, "s_glo")
        assert_rel(s_loc.cpu().numpy(), o_loc, rtol, "s_loc")
        o_pooled, o_imp, o_tbm = ems_ref.select(rp, o_glo, o_loc)
        assert_rel(pooled.cpu().numpy(), o_pooled, rtol, "pooled")
        imp_n, tbm_n = imp.cpu().numpy(), tbm.cpu().numpy()
        for h in range(w.kv_heads):
            check_band(imp_n[0, h], tbm_n[0, h], o_pooled[0, h], w.seq_len - w.window, rtol)
        x_imp, x_tbm = ems_ref.partition(rp, pooled.cpu().numpy().astype(np.float64))
        np.testing.assert_array_equal(imp_n, x_imp)
        np.testing.assert_array_equal(tbm_n, x_tbm)
        ref = ems_ref.evict_merge(rp, kf, vf, imp_n, tbm_n)
        n_diff = assert_dest_valid(out["tbm_dest"].cpu().numpy(), ref["tbm_dest"], kf, imp_n, tbm_n, tau, w.budget)
        assert n_diff <= max(1, ref["tbm_dest"].size // 100)
        k_ref, v_ref, kept_ref, cnt_ref = ems_ref.merge(rp, kf, vf, imp_n, tbm_n,
                                                        out["tbm_dest"].cpu().numpy())
        np.testing.assert_array_equal(out["slot_count"].cpu().numpy(), cnt_ref)
        np.testing.assert_array_equal(out["kept_pos"].cpu().numpy(), kept_ref)
        for name, want in (("k_out", k_ref), ("v_out", v_ref)):
            got = out[name].float().cpu().numpy()
            rms = np.sqrt((want ** 2).mean(-1, keepdims=True))
            err = np.abs(got - want) / np.maximum(np.abs(want), 1e-2 * np.maximum(rms, 1e-30))
            assert err.max() <= RTOL_MERGE[mode], f"{name}: {err.max():.3e}"
        assert out["k_out"].shape == (1, 4, w.budget + 1, w.head_dim)


@pytest.mark.parametrize("mode", MODES)
def test_score_split_calls_match_fused_call(mode):
    """Row log-sum-exp alone, then the column sums from it: same scores as the one call."""
    b, hq, hkv, d, n, w = 1, 4, 2, 128, 1111, 32
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=21)
    p = B.EmsParams(b, hq, hkv, d, n, w, dtype=mode)
    q, k = dev_tensor(inp.q, mode), dev_tensor(inp.k, mode)
    s_glo, s_loc, lse = B.ems_global_local_score(p, q, k, want_lse=True)
    lse2 = B.ems_attention_lse(p, q, k)
    assert torch.equal(lse, lse2)
    g2, l2 = B.ems_global_local_score_from_lse(p, q, k, lse2)
    assert_rel(g2.cpu().numpy(), s_glo.cpu().numpy(), 1e-5, "s_glo from lse")
    assert_rel(l2.cpu().numpy(), s_loc.cpu().numpy(), 1e-5, "s_loc from lse")
    # an lse computed by the oracle (as an attention kernel would hand over) works as well
    _, _, o_lse = ems_ref.score(ref_params(p), inp.f32("q"), inp.f32("k"), want_lse=True)
    o_glo, o_loc = ems_ref.score(ref_params(p), inp.f32("q"), inp.f32("k"))
    g3, l3 = B.ems_global_local_score_from_lse(p, q, k, torch.from_numpy(o_lse.astype(np.float32)).cuda())
    assert_rel(g3.cpu().numpy(), o_glo, max(RTOL[mode], 2e-5), "s_glo from oracle lse")
    assert_rel(l3.cpu().numpy(), o_loc, max(RTOL[mode], 2e-5), "s_loc from oracle lse")


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("similarity", [B.EMS_SIM_KEY, B.EMS_SIM_VALUE])
@pytest.mark.parametrize("shape", [(1, 400, 48), (1, 4000, 1300), (8, 9000, 2066)])   # one slice of centres, several, two token tiles per wave
def test_destinations_of_rows_without_a_norm(shape, similarity, mode):
    """Tokens whose reciprocal norm is zero.  An infinity or a NaN in the row: every product is infinite or no
    number, hence no similarity (-inf) and the zero class, whatever tau.  Rows of zeros, and rows whose squares
    leave the float range on either side: similarity 0 to every centre, so the lowest one.  The other tokens
    of the same wave: float32 rounding of the similarity only."""
    bh, n, nb = shape
    d, w = 64, 16
    p = B.EmsParams(1, bh, bh, d, n, w, nb, merge_ratio=1.0, tau=-2.0, dtype=mode)
    n_imp, n_tbm = B.ems_partition_sizes(p)
    gen = torch.Generator().manual_seed(n)
    rows = torch.randn((1, bh, n, d), generator=gen).to(p.torch_dtype)
    other = torch.randn((1, bh, n, d), generator=gen).to(p.torch_dtype).cuda()
    imp, tbm = (torch.arange(a, b, dtype=torch.int32).repeat(1, bh, 1).cuda() for a, b in ((0, n_imp), (n_imp, n_imp + n_tbm)))

    def dest(x):
        k, v = (x, other) if similarity == B.EMS_SIM_KEY else (other, x)
        out = B.ems_evict_merge_variant(p, similarity, k, v, None, imp, tbm)
        return out["tbm_sim"].cpu().numpy()[0], out["tbm_dest"].cpu().numpy()[0]

    plain_sim, plain_dest = dest(rows.cuda())
    t = n_imp
    rows[0, -1, t + 2, 3] = float("inf")
    rows[0, -1, t + 3, 40] = -float("inf")
    rows[0, -1, t + 5, 1:3] = torch.tensor([float("inf"), -float("inf")])
    rows[0, -1, t + 6, 9] = float("nan")
    rows[0, -1, t + 8] = 0.0
    rows[0, -1, t + 9] *= 2.0 ** 66
    rows[0, -1, t + 11] *= 2.0 ** -100
    sim, where = dest(rows.cuda())
    none, zero = [2, 3, 5, 6], [8, 9, 11]
    assert (sim[-1, none] == -np.inf).all() and (where[-1, none] == nb).all(), (sim[-1, none], where[-1, none])
    assert (sim[-1, zero] == 0).all() and (where[-1, zero] == 0).all(), (sim[-1, zero], where[-1, zero])
    rest = np.setdiff1d(np.arange(n_tbm), none + zero)
    np.testing.assert_allclose(sim[-1, rest], plain_sim[-1, rest], rtol=2.0 ** -22)     # two roundings, in another order
    assert (where[-1, rest] != plain_dest[-1, rest]).sum() <= max(1, n_tbm // 1000)     # ties within that rounding
    np.testing.assert_array_equal(sim[:-1], plain_sim[:-1])


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("similarity", [B.EMS_SIM_KEY, B.EMS_SIM_KEY_VALUE])
@pytest.mark.parametrize("heads,n_imp,n_tbm", [(1, 1, 33), (2, 65, 129), (1, 256, 40), (1, 257, 40), (3, 513, 385), (2, 1030, 1000),
                                               (16, 1090, 2100), (1, 4097, 130)])
def test_destinations_of_equal_centres(heads, n_imp, n_tbm, similarity, mode):
    """One-hot rows: products of 1 and 0, so a token's centres tie bit for bit and the lowest of them is its
    destination, whatever the slices, stages and pairs that the search cuts the centres into (their last ones in part)."""
    d, w = 64, 8
    n = n_imp + n_tbm + w
    p = B.EmsParams(1, heads, heads, d, n, w, n_imp + w, merge_ratio=(n_tbm + 0.5) / (n_imp + w), tau=-2.0, dtype=mode)
    assert B.ems_partition_sizes(p) == (n_imp, n_tbm)
    rng = np.random.default_rng(n)
    hot = rng.integers(0, d, (heads, n))
    hot[:, :n_imp // 2] %= d // 2                        # the higher half first occurs far down the list
    order = np.stack([rng.permutation(n - w) for _ in range(heads)])
    imp, tbm = np.sort(order[:, :n_imp]), np.sort(order[:, n_imp:])
    k = torch.nn.functional.one_hot(torch.from_numpy(hot), d)[None].to(p.torch_dtype).cuda()
    out = B.ems_evict_merge_variant(p, similarity, k, k, None, *(torch.from_numpy(x.astype(np.int32))[None].cuda() for x in (imp, tbm)))
    rows = np.arange(heads)[:, None]
    same = hot[rows, tbm][:, :, None] == hot[rows, imp][:, None, :]
    np.testing.assert_array_equal(out["tbm_dest"].cpu().numpy()[0], same.argmax(-1))      # (none alike: 0 with all, the first)
    np.testing.assert_array_equal(out["tbm_sim"].cpu().numpy()[0], same.any(-1).astype(np.float32))


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("exponent", [-60, -66, -70])
def test_key_norms_of_tiny_rows(exponent, mode):
    """Rows whose squares are subnormal sums: they are kept, to the spacing of subnormal numbers.  64 squares of 2^(2e),
    each addition off by at most 2^-150: half of 64 * 2^-150 / 2^(6 + 2e) relative on the norm, and the ordinary
    float32 rounding of 64 additions (half of 64 * 2^-24)."""
    d, n, w, nb = 64, 400, 16, 48
    gen = torch.Generator().manual_seed(1)
    k = torch.randn((1, 2, n, d), generator=gen).sign() * (1 + torch.randint(0, 128, (1, 2, n, d), generator=gen) / 128)
    k = (k * 2.0 ** exponent).to(torch.float32 if mode == B.EMS_F32 else torch.bfloat16)     # exact
    p = B.EmsParams(1, 2, 2, d, n, w, nb, merge_ratio=1.0, tau=0.3, dtype=mode)
    n_imp, n_tbm = B.ems_partition_sizes(p)
    imp, tbm = (torch.arange(a, b, dtype=torch.int32).repeat(1, 2, 1).cuda() for a, b in ((0, n_imp), (n_imp, n_imp + n_tbm)))
    for sim in (B.EMS_SIM_KEY, B.EMS_SIM_VALUE, B.EMS_SIM_KEY_VALUE):
        out = B.ems_evict_merge_variant(p, sim, k.cuda(), k.cuda(), None, imp, tbm)
        norm = out["k_norm"].cpu().double()
        want = k[:, :, :n_imp + n_tbm].double().norm(dim=-1)
        assert float((norm / want - 1).abs().max()) <= 2.0 ** -19 + 2.0 ** (-151 - 2 * exponent)


# ---------------------------------------------------------------------------- expansion
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("tau", [0.6, -2.0, 2.0])
@pytest.mark.parametrize("shape", MERGE_SHAPES[:3])
def test_expand_matches_oracle(shape, tau, mode):
    """Shared-entry expansion of the GPU's own compact cache against the oracle's expansion
    of the same cache (App. A): positions exact, keys/values to the rounding of one product."""
    b, hkv, d, n, w, nb, r = shape
    _log("expand", shape, "tau", tau, "mode", mode)
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=nb + 7)
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=r, tau=tau, dtype=mode)
    imp, tbm = _random_partition(p, seed=nb + 2)
    kf = inp.f32("k").copy()
    rng = np.random.default_rng(5)
    for bb in range(b):
        for h in range(hkv):
            for t in tbm[bb, h, ::4]:
                c = imp[bb, h, rng.integers(0, imp.shape[-1])]
                kf[bb, h, t] = 0.9 * kf[bb, h, c] + 0.4 * kf[bb, h, t]
    inp.k = ems_inputs.f32_to_bf16_bits(kf)
    tbm_d = torch.from_numpy(tbm).cuda()
    merged = B.ems_evict_merge(p, dev_tensor(inp.k, mode), dev_tensor(inp.v, mode),
                               torch.from_numpy(imp).cuda(), tbm_d)
    k_exp, v_exp, pos = B.ems_expand(p, merged, tbm_d)
    host = {k_: (v_.float().cpu().numpy() if v_.is_floating_point() else v_.cpu().numpy())
            for k_, v_ in merged.items()}
    ko, vo, po = ems_ref.expand(ref_params(p), host["k_out"], host["v_out"], host["kept_pos"], tbm,
                                host["tbm_dest"], host["k_norm"])
    np.testing.assert_array_equal(pos.cpu().numpy(), po)
    np.testing.assert_array_equal(v_exp.float().cpu().numpy(), vo)            # values are copies
    got = k_exp.float().cpu().numpy()
    rtol = 2.0 ** -8 if mode == B.EMS_BF16 else 1e-6                          # one rounding of n/n_c * k
    rms = np.sqrt((ko ** 2).mean(-1, keepdims=True))
    err = np.abs(got - ko) / np.maximum(np.abs(ko), 1e-2 * np.maximum(rms, 1e-30))
    assert err.max() <= rtol, err.max()
    n_imp, n_tbm = B.ems_partition_sizes(p)
    assert k_exp.shape == (b, hkv, n_imp + n_tbm + w, d)
    if tau >= 1:
        assert (pos[..., n_imp:n_imp + n_tbm] == -1).all()
    if tau == 0.6:
        sel = pos[..., n_imp:n_imp + n_tbm]
        assert (sel == -1).any() and (sel >= 0).any()


# ---------------------------------------------------------------------------- merge variants
def _unit64(x):
    x = x.astype(np.float64)
    return x / np.linalg.norm(x, axis=-1, keepdims=True)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("sim", [B.EMS_SIM_KEY, B.EMS_SIM_VALUE, B.EMS_SIM_KEY_VALUE])
@pytest.mark.parametrize("shape", MERGE_SHAPES[:3])
def test_evict_merge_variant_matches_oracle(shape, sim, weighted, mode):
    """Redundancy as key / value / key x value cosine (Sec. 4.1) and the score-weighted merge
    (Sec. 4.2) against the oracle's versions of both."""
    b, hkv, d, n, w, nb, r = shape
    tau = 0.5
    _log("variant", shape, "sim", sim, "weighted", weighted, "mode", mode)
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=nb + 11)
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=r, tau=tau, dtype=mode)
    imp, tbm = _random_partition(p, seed=nb + 5)
    kf, vf = inp.f32("k").copy(), inp.f32("v").copy()
    rng = np.random.default_rng(9)
    for bb in range(b):
        for h in range(hkv):
            for t in tbm[bb, h, ::3]:                      # near-duplicates in keys AND values
                c = imp[bb, h, rng.integers(0, imp.shape[-1])]
                kf[bb, h, t] = 0.9 * kf[bb, h, c] + 0.3 * kf[bb, h, t]
                vf[bb, h, t] = 0.8 * vf[bb, h, c] + 0.35 * vf[bb, h, t]
    inp.k, inp.v = ems_inputs.f32_to_bf16_bits(kf), ems_inputs.f32_to_bf16_bits(vf)
    kf, vf = inp.f32("k"), inp.f32("v")
    wt = None
    if weighted:
        wt = rng.uniform(0.0, 2.0, (b, hkv, n)).astype(np.float32)
        wt[..., ::7] = 0.0
        wt[..., 3::11] = -0.5                               # counts as 0

    out = B.ems_evict_merge_variant(p, sim, dev_tensor(inp.k, mode), dev_tensor(inp.v, mode),
                                    None if wt is None else torch.from_numpy(wt).cuda(),
                                    torch.from_numpy(imp).cuda(), torch.from_numpy(tbm).cuda())
    out = {k_: v_.float().cpu().numpy() if v_.is_floating_point() else v_.cpu().numpy()
           for k_, v_ in out.items()}
    rp = ref_params(p)
    d_ref, s_ref, n_ref = ems_ref.dest_sim(rp, sim, kf, vf, imp, tbm)
    n_imp, n_tbm = B.ems_partition_sizes(p)
    np.testing.assert_allclose(out["tbm_sim"], s_ref, rtol=0, atol=1e-5)
    np.testing.assert_allclose(out["k_norm"], n_ref, rtol=1e-6)
    differ = out["tbm_dest"] != d_ref
    for bb, h, i in zip(*np.nonzero(differ)):
        ck = _unit64(kf[bb, h, imp[bb, h]]) @ _unit64(kf[bb, h, tbm[bb, h, i]])
        cv = _unit64(vf[bb, h, imp[bb, h]]) @ _unit64(vf[bb, h, tbm[bb, h, i]])
        top2 = np.sort([ck, cv, ck * cv][sim])[-2:]
        assert top2[1] - top2[0] < 4e-5 or abs(top2[1] - tau) < 4e-5, (bb, h, i, top2)
    assert differ.mean() < 0.01
    assert (out["tbm_dest"] < n_imp).any() and (out["tbm_dest"] == nb).any()

    if weighted:
        k_ref, v_ref, kept_ref, cnt_ref = ems_ref.merge_weighted(rp, kf, vf, wt, imp, tbm, out["tbm_dest"])
    else:
        k_ref, v_ref, kept_ref, cnt_ref = ems_ref.merge(rp, kf, vf, imp, tbm, out["tbm_dest"])
    np.testing.assert_array_equal(out["kept_pos"], kept_ref)
    np.testing.assert_array_equal(out["slot_count"], cnt_ref)
    for name, got, want in (("k_out", out["k_out"], k_ref), ("v_out", out["v_out"], v_ref)):
        rms = np.sqrt((want ** 2).mean(-1, keepdims=True))
        err = np.abs(got - want) / np.maximum(np.abs(want), 1e-2 * np.maximum(rms, 1e-30))
        assert err.max() <= RTOL_MERGE[mode], f"{name}: {err.max():.3e}"


def test_variant_with_key_cosine_and_no_weights_is_evict_merge():
    b, hkv, d, n, w, nb, r = MERGE_SHAPES[1]
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=77)
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=r, tau=0.2)
    imp, tbm = _random_partition(p, seed=78)
    k, v = dev_tensor(inp.k, B.EMS_BF16), dev_tensor(inp.v, B.EMS_BF16)
    i_d, t_d = torch.from_numpy(imp).cuda(), torch.from_numpy(tbm).cuda()
    a = B.ems_evict_merge(p, k, v, i_d, t_d)
    c = B.ems_evict_merge_variant(p, B.EMS_SIM_KEY, k, v, None, i_d, t_d)
    for name in a:
        assert torch.equal(a[name].view(torch.uint8), c[name].view(torch.uint8)), name
    # constant weights: same destinations, same averages up to the rounding of the weights' products
    ones = torch.full((b, hkv, n), 0.5, device="cuda")
    e = B.ems_evict_merge_variant(p, B.EMS_SIM_KEY, k, v, ones, i_d, t_d)
    assert torch.equal(a["tbm_dest"], e["tbm_dest"]) and torch.equal(a["slot_count"], e["slot_count"])
    torch.testing.assert_close(e["v_out"].float(), a["v_out"].float(), rtol=2e-2, atol=1e-3)


def test_all_zero_weights_keep_the_centres_on_gpu():
    b, hkv, d, n, w, nb, r = MERGE_SHAPES[0]
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=79)
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=r, tau=-2.0)
    imp, tbm = _random_partition(p, seed=80)
    k, v = dev_tensor(inp.k, B.EMS_BF16), dev_tensor(inp.v, B.EMS_BF16)
    i_d, t_d = torch.from_numpy(imp).cuda(), torch.from_numpy(tbm).cuda()
    o = B.ems_evict_merge_variant(p, B.EMS_SIM_KEY_VALUE, k, v, torch.zeros((b, hkv, n), device="cuda"), i_d, t_d)
    n_imp, _ = B.ems_partition_sizes(p)
    for h in range(hkv):
        assert torch.equal(o["k_out"][0, h, :n_imp], k[0, h, i_d[0, h].long()])
        assert torch.equal(o["v_out"][0, h, :n_imp], v[0, h, i_d[0, h].long()])
    assert (o["slot_count"][..., :n_imp].sum(-1) == n_imp + (o["tbm_dest"] < n_imp).sum(-1)).all()


# ---------------------------------------------------------------------------- degenerate inputs
@pytest.mark.parametrize("mode", MODES)
def test_zero_keys_identical_keys_and_full_budget(mode):
    """Keys of norm 0 have similarity 0 and unit key 0; identical keys tie and go to the lowest
    slot; budget = N leaves nothing to merge or evict."""
    b, hkv, d, n, w, nb, r = 1, 2, 64, 400, 8, 40, 2.0
    inp = ems_inputs.small(b, hkv, hkv, d, n, seed=31)
    kf = inp.f32("k").copy()
    p = B.EmsParams(b, hkv, hkv, d, n, w, nb, merge_ratio=r, tau=-0.5, dtype=mode)
    imp, tbm = _random_partition(p, seed=32)
    kf[0, 0, tbm[0, 0, 3]] = 0.0                         # a to-be-merged key of norm 0
    kf[0, 0, imp[0, 0, 5]] = 0.0                         # a centre of norm 0
    kf[0, 1, :] = kf[0, 1, 0]                            # head 1: every key the same
    inp.k = ems_inputs.f32_to_bf16_bits(kf)
    kf, vf = inp.f32("k"), inp.f32("v")
    out = B.ems_evict_merge(p, dev_tensor(inp.k, mode), dev_tensor(inp.v, mode),
                            torch.from_numpy(imp).cuda(), torch.from_numpy(tbm).cuda())
    out = {k_: v_.float().cpu().numpy() if v_.is_floating_point() else v_.cpu().numpy() for k_, v_ in out.items()}
    rp = ref_params(p)
    ref = ems_ref.evict_merge(rp, kf, vf, imp, tbm)
    assert out["tbm_sim"][0, 0, 3] == 0.0 and out["k_norm"][0, 0, p.budget - w + 3] == 0.0
    np.testing.assert_allclose(out["tbm_sim"][0, 0], ref["tbm_sim"][0, 0], atol=5e-6)
    # head 1: all cosines are 1 up to rounding, so any slot is within noise; the merged rows must
    # still be the oracle's average for the kernel's own destinations
    np.testing.assert_allclose(out["tbm_sim"][0, 1], 1.0, atol=5e-6)
    k_ref, v_ref, kept_ref, cnt_ref = ems_ref.merge(rp, kf, vf, imp, tbm, out["tbm_dest"])
    np.testing.assert_array_equal(out["slot_count"], cnt_ref)
    for name, want in (("k_out", k_ref), ("v_out", v_ref)):
        rms = np.sqrt((want ** 2).mean(-1, keepdims=True))
        err = np.abs(out[name] - want) / np.maximum(np.abs(want), 1e-2 * np.maximum(rms, 1e-30))
        assert err.max() <= RTOL_MERGE[mode], f"{name}: {err.max():.3e}"
    assert np.isfinite(out["k_out"]).all() and np.isfinite(out["v_out"]).all()

    # budget = N: every position before the window is a centre, nothing is merged or evicted
    p2 = B.EmsParams(b, hkv, hkv, d, n, w, n, merge_ratio=3.0, tau=0.6, dtype=mode)
    assert B.ems_partition_sizes(p2) == (n - w, 0)
    s = torch.rand((b, hkv, n), device="cuda")
    imp2, tbm2 = B.ems_select(p2, s, s.clone())
    assert torch.equal(imp2, torch.arange(n - w, device="cuda", dtype=torch.int32).expand(b, hkv, -1))
    kd, vd = dev_tensor(inp.k, mode), dev_tensor(inp.v, mode)
    o2 = B.ems_evict_merge(p2, kd, vd, imp2, tbm2)
    assert torch.equal(o2["k_out"][:, :, :n], kd) and torch.equal(o2["v_out"][:, :, :n], vd)
    assert (o2["slot_count"][..., :-1] == 1).all() and (o2["slot_count"][..., -1] == 0).all()


def test_probe_kernels_run():
    """The benchmark's measurement kernels: the copy copies, the MFMA loop leaves finite values."""
    from paper_2412_08521_amd import bench_probe
    src = torch.randn(1 << 20, device="cuda")
    dst = torch.zeros_like(src)
    assert bench_probe.probe_copy(src, dst) == 2 * src.numel() * 4
    sink = torch.empty(8 * 256, dtype=torch.float32, device="cuda")
    assert bench_probe.probe_mfma(8, 10, sink) == 8 * 4 * 10 * 32 * 32768
    torch.cuda.synchronize()
    assert torch.equal(src, dst) and torch.isfinite(sink).all()
    ops = torch.randn(bench_probe.OPERAND_BYTES // 2, device="cuda").to(torch.bfloat16)
    bench_probe.probe_mfma(8, 100, sink, operands=ops)
    torch.cuda.synchronize()
    assert torch.isfinite(sink).all()


def test_probe_of_the_smaller_tile_runs():
    from paper_2412_08521_amd import bench_probe
    sink = torch.full((8 * 256,), float("nan"), device="cuda")
    ops = torch.randn(bench_probe.OPERAND_BYTES // 2, device="cuda").to(torch.bfloat16)
    for operands in (None, ops):
        assert bench_probe.probe_mfma(8, 100, sink, operands=operands, tile=16) == 8 * 4 * 100 * 32 * 32768
        torch.cuda.synchronize()
        assert torch.isfinite(sink).all()
