"""GPU parity of short calls in one launch: sizes around the tiles, the key tiles of a wave, the row tiles and the limits of the rule, every type,
masks, strides, budgets of their own, handed-over normalisers, keys that weigh nothing, the flag that keeps such calls on the passes, the profiled call."""
import numpy as np
import pytest
import torch

import paper_2503_17922_amd as W
import wkv_synth as S
from tests import parity as P
from tests.test_gpu_parity import batched_intermediates, run_and_check

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(name="short", seed=733, dtype="bf16", n_groups=1, gamma=2, n_q_heads=4, n_kv_heads=2, head_dim=128, w_obs=8,
                seq_len=[500], win=[8], top_p=[8], k_windows=[6])
    base.update(kw)
    return S.Workload(**base)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("L", [9, 24, 127, 128, 129, 511, 512, 513, 1023, 1024, 1025])
def test_lengths(dtype, d, L, device):
    # 16 rows: four key tiles a wave up to 512 keys, eight up to 1024 (512-byte rows: none), then in several launches
    nw = -(-(L - 8) // 8)
    run_and_check(_w(dtype=dtype, head_dim=d, seq_len=[L], k_windows=[min(nw, 9)]), device)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f16", 128), ("f16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("L", [450, 900])
@pytest.mark.parametrize("q_heads,w_obs", [(2, 1), (2, 16), (2, 17), (6, 11), (8, 16), (10, 13), (14, 16), (8, 32), (10, 26)])
def test_row_counts(dtype, d, L, q_heads, w_obs, device):
    # 1 to 130 rows a KV head, four and eight key tiles a wave: every kernel that the rule can choose, and both sides of its lines
    run_and_check(_w(dtype=dtype, head_dim=d, n_q_heads=q_heads, w_obs=w_obs, seq_len=[L, w_obs], win=[24, 8], top_p=[12, 8], k_windows=[5, 0]), device)


@pytest.mark.parametrize("kw", [
    dict(n_groups=8, gamma=1, seq_len=[300, 40], win=[8] * 2, top_p=[8] * 2, k_windows=[3, 1]),       # as many groups as one launch takes
    dict(n_groups=2, gamma=4, n_kv_heads=2, seq_len=[290 - 30 * b for b in range(8)], win=[16, 8] * 4, top_p=[5, 8] * 4, k_windows=[4] * 8),     # 256 pairs
    dict(n_groups=1, gamma=3, n_q_heads=86, n_kv_heads=43, seq_len=[200]),                             # 258: in several launches
    dict(seq_len=[900, 700], win=[128, 1], top_p=[100, 1], k_windows=[3, 300], w_obs=16),              # the largest and the smallest windows
    dict(seq_len=[528, 900], win=[128, 1], top_p=[100, 1], k_windows=[3, 300], w_obs=16),              # a token a thread ranked: in one launch
    dict(seq_len=[529, 900], win=[65, 64], top_p=[40, 64], k_windows=[3, 3], w_obs=16),
])
def test_calls(kw, device):
    run_and_check(_w(**kw), device)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_selection_and_gather_of_longer_calls(dtype, device):
    # one launch for these two, behind the score passes: budgets of their own, padding kept or filled
    w = _w(dtype=dtype, n_groups=4, gamma=2, w_obs=16, seq_len=[1700, 333], win=[8, 32], top_p=[4, 32], k_windows=[20, 5])
    _budgets(w, device)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_budgets_and_kept_padding(dtype, device):
    _budgets(_w(dtype=dtype, n_groups=4, gamma=2, seq_len=[490, 333], win=[8, 32], top_p=[4, 32], k_windows=[20, 5]), device)


def _budgets(w, device):
    budgets = [[20, 0], [3, 5], [0, 0], [11, 2]]
    ref = P.DeviceState(w, device); ref.compress(k_groups=budgets)
    st = P.DeviceState(w, device, flags=W.WKV_KEEP_PADDING); st.compress(k_groups=budgets)
    full = P.DeviceState(w, device); full.compress()
    assert torch.equal(ref.tok_idx, st.tok_idx) and torch.equal(ref.win_idx, st.win_idx) and torch.equal(ref.n_keep, st.n_keep)
    for g, (l, b, h) in ((l // 2, (l, b, h)) for l in range(8) for b in range(2) for h in range(2)):
        n, kept = int(ref.n_keep[g, b, h]), ref.win_idx[g, b, h]
        assert int((kept >= 0).sum()) == budgets[g][b] and bool(np.isin(kept[kept >= 0].cpu(), full.win_idx[g, b, h].cpu()).all())
        rows = ref.tok_idx[g, b, h, :n].to(torch.int64)
        assert torch.equal(ref.k_out[l][b, h, :n], ref.k[l][b, h].index_select(0, rows))
        assert torch.equal(st.v_out[l][b, h, :n], st.v[l][b, h].index_select(0, rows))
        assert not ref.v_out[l][b, h, n:].any() and bool((st.k_out[l][b, h, n:] == 7.0).all())


@pytest.mark.parametrize("dtype,d,L", [("bf16", 128, 500), ("f16", 64, 1000), ("f32", 64, 700), ("f32", 64, 400)])
@pytest.mark.parametrize("w_obs", [8, 32])
def test_normalisers_handed_over(dtype, d, L, w_obs, device):
    w = _w(dtype=dtype, head_dim=d, n_groups=2, w_obs=w_obs, seq_len=[L], win=[16], top_p=[8])
    st = P.DeviceState(w, device); st.compress(lse=[st.oracle_lse(g) for g in range(2)])
    _, s_given = batched_intermediates(st)
    own = P.DeviceState(w, device); own.compress()
    _, s_own = batched_intermediates(own)
    np.testing.assert_allclose(s_given, s_own, rtol=2e-5, atol=1e-12)
    assert torch.equal(st.tok_idx, own.tok_idx) and torch.equal(st.v_out[3], own.v_out[3])


@pytest.mark.parametrize("dtype,d,L", [("bf16", 128, 500), ("f16", 64, 1000), ("f32", 64, 700)])
def test_the_two_passes_where_they_are_asked_for(dtype, d, L, device):
    w = _w(dtype=dtype, head_dim=d, seq_len=[L, 300], win=[16, 8], top_p=[8, 8], k_windows=[6, 6])
    st = P.DeviceState(w, device); st.compress()
    asked = P.DeviceState(w, device, flags=W.WKV_SCORE_TWO_PASS); asked.compress()
    (_, s_short), (_, s_asked) = batched_intermediates(st), batched_intermediates(asked)
    _, s, *_ = asked.stages(0)                                # the stage calls run the same passes: the same bits
    for b, n in enumerate(w.seq_len):
        nw = -(-(n - w.w_obs) // w.win[b])
        assert np.array_equal(s_asked[0, b, :, :nw], s[b, :, :nw].cpu().numpy())
        np.testing.assert_allclose(s_short[0, b, :, :nw], s_asked[0, b, :, :nw], rtol=2e-5, atol=1e-12)
    assert torch.equal(st.tok_idx, asked.tok_idx) and torch.equal(st.k_out[1], asked.k_out[1])


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("handed_over", [False, True])
def test_profiled_call_gives_the_same_results(dtype, d, handed_over, device):
    w = _w(dtype=dtype, head_dim=d, n_groups=2, seq_len=[500, 300], win=[16, 8], top_p=[8, 8], k_windows=[6, 6])
    ref, st = P.DeviceState(w, device), P.DeviceState(w, device)
    lse = [st.oracle_lse(g) for g in range(2)] if handed_over else None
    ref.compress(lse=lse)
    ms = W.CompressCall(st.problem, w.n_groups, w.gamma, st.q, lse, st.k, st.v, st.k_out, st.v_out, st.win_idx, st.tok_idx, st.n_keep,
                        st.workspace).profiled()
    assert 0.0 < ms[1] < 50.0 and ms[0] == ms[2] == ms[3] == 0.0, ms
    (_, want), (_, got) = batched_intermediates(ref), batched_intermediates(st)
    for b, n in enumerate(w.seq_len):
        nw = -(-(n - w.w_obs) // w.win[b])
        assert np.array_equal(got[:, b, :, :nw], want[:, b, :, :nw])          # the same launch: the same bits
    for a, b in zip((st.win_idx, st.tok_idx, st.n_keep, *st.k_out, *st.v_out), (ref.win_idx, ref.tok_idx, ref.n_keep, *ref.k_out, *ref.v_out)):
        assert torch.equal(a, b)


def test_outputs_in_the_memory_of_the_queries(device):
    # the last layer's compact values take the place of the queries
    w = _w(n_q_heads=16, w_obs=16, seq_len=[500], win=[16], top_p=[8])
    ref = P.DeviceState(w, device); ref.compress()
    st = P.DeviceState(w, device)
    room = torch.empty(max(st.q[0].numel(), st.v_out[1].numel()), dtype=torch.bfloat16, device=device)
    q, out = room[:st.q[0].numel()].view_as(st.q[0]), room[:st.v_out[1].numel()].view_as(st.v_out[1])
    for _ in range(20):
        q.copy_(st.q[0])
        st.q[0], st.v_out[1], given = q, out, st.q[0]
        st.compress()
        st.q[0] = given
        assert torch.equal(st.tok_idx, ref.tok_idx) and torch.equal(out, ref.v_out[1]) and torch.equal(st.k_out[0], ref.k_out[0])


def test_strides(device):
    # caches and queries in token-major order, outputs spread out: the rows of the contiguous call
    w = _w(dtype="f16", seq_len=[400, 311], win=[8, 24], top_p=[8, 12], k_windows=[6, 3])
    st = P.DeviceState(w, device); st.compress()
    B, H, Hq, d, T = 2, 2, 4, 128, 400
    nk = st.dims.nkeep_max
    p = W.Problem(n_q_heads=Hq, n_kv_heads=H, head_dim=d, w_obs=8, seq_len=w.seq_len, win=w.win, top_p=w.top_p, k_windows=w.k_windows, dtype=W.WKV_F16,
                  max_seq_len=T, kv_strides=(T * H * d, d, H * d), q_strides=(8 * Hq * d, d, Hq * d), out_strides=(nk * H * 2 * d, 2 * d, H * 2 * d))
    major = lambda x: x.transpose(1, 2).contiguous()
    outs = [[torch.full((B, nk, H, 2 * d), 7.0, dtype=torch.float16, device=device) for _ in range(2)] for _ in range(2)]
    idx = [torch.empty_like(st.win_idx), torch.empty_like(st.tok_idx), torch.empty_like(st.n_keep)]
    W.wkv_compress_groups(p, 1, 2, [major(st.q[0])], None, [major(x) for x in st.k], [major(x) for x in st.v], outs[0], outs[1], *idx,
                          torch.empty(W.wkv_workspace_bytes(p, 1), dtype=torch.uint8, device=device))
    torch.cuda.synchronize()
    assert torch.equal(idx[1], st.tok_idx)
    for l in range(2):
        assert torch.equal(outs[0][l][..., :d].transpose(1, 2), st.k_out[l]) and torch.equal(outs[1][l][..., :d].transpose(1, 2), st.v_out[l])
        assert bool((outs[0][l][..., d:] == 7.0).all())


@pytest.mark.parametrize("offset", [0.0, -2048.0])
def test_keys_that_weigh_nothing(offset, device):
    # a stretch of keys, whole tiles of some waves, with logits of -inf, beside ordinary logits and beside ones far below zero: they score zero, the
    # others as by the stage calls
    w = _w(dtype="f32", head_dim=64, seq_len=[500], win=[4], top_p=[4], k_windows=[6])
    st = P.DeviceState(w, device)
    st.q[0][..., 0] = 1.0
    st.k[0][..., 0] = offset
    st.k[0][:, :, 100:333, 0] = -float("inf")
    st.compress()
    t, s, wi, ti, nk = st.stages(0)
    _, got = batched_intermediates(st)
    want = s.cpu().numpy()
    assert np.isfinite(got).all() and (got[0, :, :, 25:83] == 0).all() and (want[:, :, 25:83] == 0).all()
    # a product is summed in 64 steps, each rounded to half a unit in the last place of at most 2^12 (2^-12), times 1/8 in the exponent: at random signs
    # 8 * 2^-12 / 8 for either side
    np.testing.assert_allclose(got[0], want, rtol=5e-4 if offset else 2e-5, atol=1e-30)
    assert torch.equal(ti, st.tok_idx[0])
