"""GPU parity of the decode-time path (ems_decode_init, ems_decode_step) against the numpy
oracle.  Every step is checked in isolation: the oracle starts from the GPU's own state before
the step, so that one flipped near-tie cannot hide or fake later differences."""
import sys

import numpy as np
import pytest
import torch

import ems_inputs
from gpu_util import decode_launches, dev_tensor, ref_params
from oracle import ems_decode_ref as dec
from oracle import ems_ref
from paper_2412_08521_amd import binding as B

pytestmark = pytest.mark.gpu

MODES = [B.EMS_BF16, B.EMS_F32]
SHAPES = [
    # (b, hq, hkv, d, n, w, budget, r)
    (1, 4, 2, 64, 600, 16, 48, 1.5),
    (2, 8, 2, 128, 1500, 32, 160, 2.0),
    (1, 2, 2, 128, 900, 8, 200, 3.0),
    (1, 8, 1, 64, 700, 8, 40, 1.0),
]


def _log(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def _np(t):
    return t.float().cpu().numpy() if t.is_floating_point() else t.cpu().numpy()


def _prefill(shape, mode, tau, seed):
    """Prompt compressed by the library; returns params, device tensors and the state."""
    b, hq, hkv, d, n, w, nb, r = shape
    inp = ems_inputs.small(b, hq, hkv, d, n, seed=seed)
    p = B.EmsParams(b, hq, hkv, d, n, w, nb, merge_ratio=r, tau=tau, pool_kernel=3, dtype=mode)
    q, k, v = (dev_tensor(getattr(inp, x), mode) for x in "qkv")
    s_glo, s_loc = B.ems_global_local_score(p, q, k)
    imp, tbm = B.ems_select(p, s_glo, s_loc)
    pre = B.EmsParams(b, hq, hkv, d, n, w, nb, merge_ratio=r, tau=0.25, pool_kernel=3, dtype=mode)
    merged = B.ems_evict_merge(pre, k, v, imp, tbm)
    st = B.ems_decode_init(p, merged, tbm, s_glo, s_loc)
    return p, merged, tbm, s_glo, s_loc, st


def _host_state(st, b, h):
    out = {}
    for name in B.STATE_FIELDS:
        if name == "step_count":
            continue
        a = _np(getattr(st, name)[b, h])
        out[name] = a.astype(np.int64) if a.dtype.kind == "i" else a.astype(np.float64)
    return out


def _new_token(p, rng, mode):
    def mk(heads):
        x = ems_inputs.f32_to_bf16_bits(rng.standard_normal((p.batch, heads, p.head_dim)).astype(np.float32))
        return x
    return mk(p.q_heads), mk(p.kv_heads), mk(p.kv_heads)


def run_and_check_step(p, st, t, qb, kb, vb, tau, units, mode):
    """One ems_decode_step on the GPU, checked in isolation for the given (batch, kv-head) units:
    the oracle takes the same step from the GPU's own state before it.  qb, kb, vb are bf16 bit
    patterns [B, heads, D].  Returns (decisions flipped inside float32 noise, merges, evictions)."""
    G, W = p.q_heads // p.kv_heads, p.window
    # merged rows: one bf16 rounding of the stored row; in f32 mode about ten float32 roundings with
    # cancellation between the two entries (the f32 bar of the prefill merge is the same 1e-5)
    cache_rtol = 2.0 ** -7 if mode == B.EMS_BF16 else 1e-5
    before = {u: _host_state(st, *u) for u in units}
    out = B.ems_decode_step(p, st, t, dev_tensor(qb, mode), dev_tensor(kb, mode), dev_tensor(vb, mode),
                            want_attn=True)
    attn, decision, sim = _np(out["attn"]), _np(out["decision"]), _np(out["sim"])
    qf, kf, vf = (ems_inputs.bf16_bits_to_f32(x).astype(np.float64) for x in (qb, kb, vb))
    n_flip = n_merge = n_evict = 0
    for (b, h) in units:
        ref = before[(b, h)]
        info = dec.decode_step(ref, t, W, p.budget, tau, 0.0, qf[b, h * G:(h + 1) * G], kf[b, h], vf[b, h],
                               p.seq_len + t)
        got = _host_state(st, b, h)
        np.testing.assert_allclose(attn[b, h * G:(h + 1) * G], info["attn"], rtol=2e-5, atol=1e-9)
        if tuple(decision[b, h]) != (info["tbm_entry"], info["dest"]):
            # a different decision is legitimate only inside float32 noise of a tie or of tau
            sc, sims = info["centre_score"], info["centre_sims"]
            gs, gd = int(decision[b, h, 0]), int(decision[b, h, 1])
            if gs != info["tbm_entry"]:
                assert abs(sc[gs] - sc[info["tbm_entry"]]) <= 1e-5 * np.abs(sc).max(), (t, b, h)
            elif gd >= 0 and info["dest"] >= 0:
                assert abs(sims[gd] - sims[info["dest"]]) < 2e-5, (t, b, h)
            else:
                assert abs(info["sim"] - tau) < 2e-5, (t, b, h)
            n_flip += 1
            continue
        n_merge += info["dest"] >= 0
        n_evict += info["dest"] < 0
        if np.isfinite(info["sim"]):
            assert abs(sim[b, h] - info["sim"]) < 1e-5
        for name in ("entry_count", "entry_tok", "tok_pos", "tok_row"):
            np.testing.assert_array_equal(got[name], ref[name], err_msg=f"{name} step {t}")
        for name in ("tok_norm", "tok_glo", "tok_past", "tok_cur", "row_norm"):
            np.testing.assert_allclose(got[name], ref[name], rtol=2e-5, atol=1e-9, err_msg=f"{name} step {t}")
        for name in ("k_cache", "v_cache"):
            want, have = ref[name][:p.budget], got[name][:p.budget]
            rms = np.sqrt((want ** 2).mean(-1, keepdims=True))
            err = np.abs(have - want) / np.maximum(np.abs(want), 1e-2 * np.maximum(rms, 1e-30))
            assert err.max() <= cache_rtol, f"{name} step {t}: {err.max():.3e}"
    return n_flip, n_merge, n_evict


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", SHAPES[:3])
def test_decode_init_matches_oracle(shape, mode):
    _log("decode_init", shape, mode)
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, mode, 0.3, seed=5)
    m = {k_: _np(v_) for k_, v_ in merged.items()}
    for b in range(p.batch):
        for h in range(p.kv_heads):
            ref = dec.decode_init(p.seq_len, p.window, p.budget, p.merge_ratio, m["k_out"][b, h], m["v_out"][b, h],
                                  m["kept_pos"][b, h], _np(tbm)[b, h], m["tbm_dest"][b, h], m["k_norm"][b, h],
                                  m["slot_count"][b, h], _np(s_glo)[b, h], _np(s_loc)[b, h])
            got = _host_state(st, b, h)
            for name in ("entry_count", "entry_tok", "tok_pos", "tok_row"):
                np.testing.assert_array_equal(got[name], ref[name], err_msg=name)
            for name in ("tok_glo", "tok_past", "tok_cur"):
                np.testing.assert_array_equal(got[name], ref[name], err_msg=name)   # gathers: exact
            np.testing.assert_allclose(got["tok_norm"], ref["tok_norm"], rtol=1e-6)
            np.testing.assert_allclose(got["row_norm"], ref["row_norm"], rtol=1e-6)
    assert (st.tok_row < 0).any() and (st.tok_row >= 0).any()


# large caches: with so few heads the bf16 step runs as three or four launches, all but the last over slices, with the
# logits in the workspace; in float32 it is one launch, whose row dots BIG stages in the workspace (they do not fit
# in LDS) and BIG_LDS in LDS
BIG = (1, 8, 1, 64, 4000, 8, 1800, 0.5)
BIG_LDS = (1, 8, 2, 128, 5000, 16, 1100, 0.5)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("tau", [0.3, -2.0, 2.0])
@pytest.mark.parametrize("shape", SHAPES + [BIG, BIG_LDS])
def test_decode_steps_match_oracle(shape, tau, mode):
    _log("decode_step", shape, "tau", tau, "mode", mode)
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, mode, tau, seed=shape[6])
    n_imp, n_tbm = B.ems_partition_sizes(p)
    G, W, D = p.q_heads // p.kv_heads, p.window, p.head_dim
    assert (shape == BIG) == (4 * (G + 1) * p.budget > 60 * 1024)
    rng = np.random.default_rng(17)
    n_merge = n_evict = n_flip = 0
    for t in range(W + 6):
        qb, kb, vb = _new_token(p, rng, mode)
        if t % 3 == 1:                                    # make some new keys similar to an entry
            src = ems_inputs.f32_to_bf16_bits(_np(st.k_cache[:, :, (3 * t) % n_imp]).astype(np.float32))
            kb = src
        units = [(b, h) for b in range(p.batch) for h in range(p.kv_heads)]
        c = run_and_check_step(p, st, t, qb, kb, vb, tau, units, mode)
        n_flip += c[0]; n_merge += c[1]; n_evict += c[2]
    total = (W + 6) * p.batch * p.kv_heads
    assert n_flip <= max(1, total // 20), (n_flip, total)
    if tau >= 1:
        assert n_merge == 0
    elif tau <= -1:
        assert n_evict == 0
    elif shape not in (BIG, BIG_LDS):                     # with a thousand random centres something is always similar
        assert n_merge > 0 and n_evict > 0, (n_merge, n_evict)


def test_decode_invariants_over_many_steps():
    shape = SHAPES[1]
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, B.EMS_BF16, 0.3, seed=3)
    n_imp, n_tbm = B.ems_partition_sizes(p)
    E, W, N = n_imp + n_tbm, p.window, p.seq_len
    g = torch.Generator(device="cpu").manual_seed(1)
    steps = 40 * W + 5                                  # long enough for every entry to be replaced several times
    qs = torch.randn((steps, p.batch, p.q_heads, p.head_dim), generator=g).to(torch.bfloat16).cuda()
    ks = torch.randn((steps, p.batch, p.kv_heads, p.head_dim), generator=g).to(torch.bfloat16).cuda()
    vs = torch.randn((steps, p.batch, p.kv_heads, p.head_dim), generator=g).to(torch.bfloat16).cuda()
    ws = torch.empty(max(B.ems_decode_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")
    out = None
    for t in range(steps):
        out = B.ems_decode_step(p, st, t, qs[t], ks[t], vs[t], ws=ws, out=out)
    torch.cuda.synchronize()
    rows, pos = _np(st.tok_row), _np(st.tok_pos)
    for b in range(p.batch):
        for h in range(p.kv_heads):
            np.testing.assert_array_equal(np.sort(pos[b, h, E:]), np.arange(N + steps - W, N + steps))
            live = rows[b, h] >= 0
            assert (rows[b, h, :E][live[:E]] < n_imp).all()
            assert len(np.unique(pos[b, h][live])) == live.sum()
            np.testing.assert_array_equal(rows[b, h][_np(st.entry_tok)[b, h]], np.arange(n_imp))
            assert (_np(st.entry_count)[b, h] >= 1).all()
            assert np.isfinite(_np(st.k_cache)[b, h]).all() and np.isfinite(_np(st.tok_glo)[b, h]).all()


# tables and centre lists so long that their slices hold several tiles (bf16; more than 32 slices of 128)
@pytest.mark.parametrize("tau", [0.3, 2.0])
@pytest.mark.parametrize("shape", [
    (1, 4, 1, 64, 6000, 8, 2083, 1.0),       # 4166 table elements: slices of two tiles, the last one ragged
    (1, 8, 1, 128, 9000, 8, 4200, 1.0),      # 8400: slices of four tiles, over two rounds of weights; 4192 centres: slices of 256
])
def test_decode_steps_of_long_tables_match_oracle(shape, tau):
    _log("decode_step", shape, "tau", tau)
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, B.EMS_BF16, tau, seed=shape[6])
    n_imp, n_tbm = B.ems_partition_sizes(p)
    assert n_imp + n_tbm + p.window > 32 * 128
    rng = np.random.default_rng(19)
    n_merge = n_evict = n_flip = 0
    for t in range(p.window + 2):
        qb, kb, vb = _new_token(p, rng, B.EMS_BF16)
        if t % 3 == 1:                                    # make some new keys similar to an entry
            kb = ems_inputs.f32_to_bf16_bits(_np(st.k_cache[:, :, n_imp - 1 - t]).astype(np.float32))
        c = run_and_check_step(p, st, t, qb, kb, vb, tau, [(0, 0)], B.EMS_BF16)
        n_flip += c[0]; n_merge += c[1]; n_evict += c[2]
    assert n_flip <= 1                                    # (at 128 elements the best of 4192 random cosines is itself about 0.3)
    assert n_merge > 0 if tau < 1 else n_merge == 0 and n_evict > 0


# head counts and centre lists on both sides of the sizes where the least important centre is chosen in a launch of its own
# (four launches: blocks x centres x (q-heads + 1) over 3 million), last slices of a few rows; units: a first, a middle and the last head.
# Bounds as in the tests above; all steps of a unit count for the flips.
@pytest.mark.parametrize("shape,launches", [
    ((2, 32, 4, 64, 3000, 8, 1290, 0.5), 3),      # 8 heads of 8, 1282 centres: 16 slices of the table, the last of 15: 1.5 million
    ((4, 64, 8, 64, 3000, 8, 1033, 0.5), 4),      # 32 heads of 8, 1025 centres, one of them in the last slice: 3.8 million
    ((1, 16, 16, 128, 9000, 8, 4200, 1.0), 3),    # 16 heads of 1, 17 slices of the table (512) and of 4192 centres (256): 2.3 million
    ((1, 64, 16, 128, 9000, 8, 4200, 1.0), 4),    # the same of 4: 5.7 million
    ((1, 32, 32, 64, 9000, 8, 4200, 1.0), 4),     # 32 heads of 1: 4.6 million
    ((2, 32, 16, 128, 3000, 8, 1410, 1.0), 4),    # 32 heads of 2, 1402 centres: 3.1 million
])
def test_decode_steps_choose_in_one_launch_or_two(shape, launches):
    _log("decode_step", shape)
    tau = 0.3
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, B.EMS_BF16, tau, seed=shape[6])
    assert decode_launches(p) == launches
    n_imp, n_tbm = B.ems_partition_sizes(p)
    rng = np.random.default_rng(29)
    n_merge = n_flip = 0
    units = [(0, 0), (p.batch // 2, p.kv_heads // 2), (p.batch - 1, p.kv_heads - 1)]
    for t in range(p.window + 2):
        qb, kb, vb = _new_token(p, rng, B.EMS_BF16)
        if t % 3 == 1:                                    # make some new keys similar to an entry
            kb = ems_inputs.f32_to_bf16_bits(_np(st.k_cache[:, :, n_imp - 1 - t]).astype(np.float32))
        c = run_and_check_step(p, st, t, qb, kb, vb, tau, units, B.EMS_BF16)
        n_flip += c[0]; n_merge += c[1]
    assert n_flip <= 1 and n_merge > 0


# more heads than the table's slices are for: the step goes over slices of the cache rows instead
@pytest.mark.parametrize("tau", [0.3, 2.0])
@pytest.mark.parametrize("shape", [
    (5, 8, 8, 64, 2000, 8, 560, 0.5),        # 40 heads; rows and new key in five slices, the last of 49 rows
    (3, 32, 16, 128, 2500, 8, 639, 1.0),     # two q-heads per kv-head; rows and new key fill five slices
    (5, 64, 8, 64, 4000, 8, 1800, 0.5),      # eight; the staged dots do not fit in LDS
])
def test_decode_steps_of_many_heads_match_oracle(shape, tau):
    _log("decode_step", shape, "tau", tau)
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, B.EMS_BF16, tau, seed=shape[6])
    n_imp, n_tbm = B.ems_partition_sizes(p)
    G, heads = p.q_heads // p.kv_heads, p.batch * p.kv_heads
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    assert B.ems_decode_workspace_bytes(p) == up(4 * heads * (G + 1) * p.budget) + up(4 * heads * 1024)    # dots and norms staged, records
    rng = np.random.default_rng(23)
    n_flip = 0
    units = [(0, 0), (1, p.kv_heads // 2), (p.batch - 1, p.kv_heads - 1)]
    for t in range(p.window + 2):
        qb, kb, vb = _new_token(p, rng, B.EMS_BF16)
        if t % 3 == 1:                                    # make some new keys similar to an entry
            kb = ems_inputs.f32_to_bf16_bits(_np(st.k_cache[:, :, n_imp - 1 - t]).astype(np.float32))
        n_flip += run_and_check_step(p, st, t, qb, kb, vb, tau, units, B.EMS_BF16)[0]
    assert n_flip <= 1
    ws = torch.empty(B.ems_decode_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    q, k, v = (dev_tensor(x, B.EMS_BF16) for x in _new_token(p, rng, B.EMS_BF16))
    B.ems_decode_step(p, st, B.EMS_STEP_FROM_STATE, q, k, v, ws=ws)
    assert int(st.step_count) == p.window + 3


# the one-launch step keeps its first rows (128 in 16 bits and 64 in float32 at head size 128, twice as many at 64) for the
# search: a chosen centre among them and behind them, tables over one batch of 1024, centre tokens that do not fit LDS
@pytest.mark.parametrize("shape,mode", [
    ((1, 4, 1, 128, 1500, 8, 136, 0.5), B.EMS_BF16),      # 128 centres: the last is the last kept row
    ((1, 2, 1, 128, 1500, 8, 137, 1.0), B.EMS_BF16),      # one more
    ((1, 8, 1, 64, 4000, 16, 500, 2.0), B.EMS_BF16),      # a table of 1500, 484 centres
    ((1, 2, 2, 128, 900, 8, 73, 0.5), B.EMS_F32),
    ((1, 1, 1, 64, 7000, 8, 5400, 0.25), B.EMS_F32),      # staged rows fit LDS, the centres' tokens behind them do not
])
def test_decode_steps_around_the_kept_rows(shape, mode):
    _log("decode_step", shape, mode)
    p, merged, tbm, s_glo, s_loc, st = _prefill(shape, mode, 0.3, seed=shape[6])
    n_imp, n_tbm = B.ems_partition_sizes(p)
    rng = np.random.default_rng(29)
    n_flip = 0
    for t in range(p.window + 2):
        if t % 2 == 0:                                    # the least important centre: by turns the last one and the first
            want = n_imp - 1 if t % 4 == 0 else 0
            at = int(st.entry_tok[0, 0, want])
            for x in (st.tok_glo, st.tok_past, st.tok_cur):
                x[:, :, at] = 0.0
        qb, kb, vb = _new_token(p, rng, mode)
        n_flip += run_and_check_step(p, st, t, qb, kb, vb, 0.3, [(0, 0)], mode)[0]
    assert n_flip <= 1
