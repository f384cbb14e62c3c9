"""GPU parity of the merged selection and gather of small calls: on both sides of the sizes that choose it, with budgets of
their own, padding kept or filled, and every row width."""
import pytest
import torch

import paper_2503_17922_amd as W
import wkv_synth as S
from tests import parity as P
from tests.test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(name="small", seed=411, dtype="bf16", n_groups=1, gamma=1, n_q_heads=8, n_kv_heads=2, head_dim=128, w_obs=16,
                seq_len=[700], win=[8], top_p=[8], k_windows=[10])
    base.update(kw)
    return S.Workload(**base)


@pytest.mark.parametrize("kw", [
    dict(n_groups=8, gamma=1, seq_len=[300, 40]),                              # eight groups, the most one launch takes
    dict(n_groups=3, gamma=3, seq_len=[300]),                                  # nine layers: two launches
    dict(n_groups=2, gamma=4, seq_len=[500] * 8),                              # 256 pairs
    dict(n_groups=1, gamma=8, n_q_heads=32, n_kv_heads=32, w_obs=8, seq_len=[200]),          # 512 pairs: one workgroup each
    dict(n_groups=1, gamma=2, seq_len=[200] * 9),                              # nine sequences: two launches
    dict(seq_len=[8192 + 16], win=[1], top_p=[1], k_windows=[8000]),           # the most windows one launch takes
    dict(seq_len=[8193 + 16], win=[1], top_p=[1], k_windows=[8193]),           # one more, all of them kept
    dict(head_dim=64, seq_len=[900, 16], win=[128, 8], top_p=[100, 8]),        # 128-byte rows, a sequence without windows
    dict(dtype="f32", head_dim=128, seq_len=[900], win=[7], top_p=[3]),        # 512-byte rows
])
def test_sizes_that_choose_the_merged_launch(kw, device):
    n = len(kw.get("seq_len", [0]))
    full = dict(kw)
    for key, val in (("win", 8), ("top_p", 8), ("k_windows", 3)):
        full.setdefault(key, [val] * n)
    full["k_windows"] = [min(k, -(-(L - kw.get("w_obs", 16)) // w)) for k, L, w in zip(full["k_windows"], full["seq_len"], full["win"])]
    run_and_check(_w(**full), device)


def test_merged_launch_with_budgets_and_kept_padding(device):
    w = _w(n_groups=4, gamma=2, seq_len=[1000, 333], win=[8, 32], top_p=[4, 32], k_windows=[20, 5])
    budgets = [[20, 0], [3, 5], [0, 0], [11, 2]]
    ref = P.DeviceState(w, device); ref.compress(k_groups=budgets)
    st = P.DeviceState(w, device, flags=W.WKV_KEEP_PADDING); st.compress(k_groups=budgets)
    assert torch.equal(ref.tok_idx, st.tok_idx) and torch.equal(ref.win_idx, st.win_idx) and torch.equal(ref.n_keep, st.n_keep)
    # stage by stage, with the largest budgets: the same windows first come out of the selection's own launch
    for g in range(4):
        for b in range(2):
            assert int(ref.n_keep[g, b, 0]) >= w.w_obs and int((ref.win_idx[g, b, 0] >= 0).sum()) == budgets[g][b]
        for l in range(g * 2, g * 2 + 2):
            for b in range(2):
                for h in range(2):
                    n = int(ref.n_keep[g, b, h])
                    rows = ref.tok_idx[g, b, h, :n].to(torch.int64)
                    assert torch.equal(ref.k_out[l][b, h, :n], ref.k[l][b, h].index_select(0, rows))
                    assert torch.equal(st.v_out[l][b, h, :n], st.v[l][b, h].index_select(0, rows))
                    assert not ref.v_out[l][b, h, n:].any() and bool((st.k_out[l][b, h, n:] == 7.0).all())
