"""GPU tests of what the score passes do before their first key tile (queries by whole rows, the fold of the statistics by the
workgroups of the second pass) and of row counts that leave a row tile of the last row group empty."""
import pytest
import torch

import paper_2503_17922_amd as W
import wkv_synth as S
from tests import parity as P
from tests.test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(name="prologue", seed=523, dtype="bf16", n_groups=1, gamma=1, n_q_heads=8, n_kv_heads=2, head_dim=128, w_obs=32,
                seq_len=[901, 430], win=[24, 8], top_p=[9, 8], k_windows=[7, 20])
    base.update(kw)
    return S.Workload(**base)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f32", 128)])
@pytest.mark.parametrize("q_heads,w_obs", [(2, 5), (8, 32), (14, 31), (16, 32)])
def test_query_layouts(dtype, d, q_heads, w_obs, device):
    # rows of a KV head's queries at equal distances (contiguous, and spread out), and not (token-major): the same scores
    w = _w(dtype=dtype, head_dim=d, n_q_heads=q_heads, w_obs=w_obs)
    st = P.DeviceState(w, device)
    q, k = st.q[0], st.k[0]
    B, n_review = len(w.seq_len), max(w.seq_len) - w_obs

    def scores(q, strides):
        p = W.Problem(n_q_heads=q_heads, n_kv_heads=w.n_kv_heads, head_dim=d, w_obs=w_obs, seq_len=w.seq_len, win=w.win, top_p=w.top_p,
                      k_windows=w.k_windows, dtype={"bf16": W.WKV_BF16, "f16": W.WKV_F16, "f32": W.WKV_F32}[dtype], q_strides=strides)
        t = torch.zeros((B, w.n_kv_heads, n_review), dtype=torch.float32, device=device)
        W.wkv_score(p, q, k, None, t, torch.empty(W.wkv_workspace_bytes(p, 1), dtype=torch.uint8, device=device))
        torch.cuda.synchronize()
        return t

    want = scores(q, (q_heads * w_obs * d, w_obs * d, d))
    assert want.abs().max() > 0
    spread = torch.empty((B, q_heads, w_obs, 3 * d), dtype=q.dtype, device=device).fill_(float("nan"))
    spread[..., :d] = q
    assert torch.equal(scores(spread, (q_heads * w_obs * 3 * d, w_obs * 3 * d, 3 * d)), want)
    token_major = q.transpose(1, 2).contiguous()
    assert torch.equal(scores(token_major, (q_heads * w_obs * d, d, q_heads * d)), want)


@pytest.mark.parametrize("L", [2050, 4200, 8192, 8290])
def test_statistics_folded_by_the_second_pass(L, device):
    # two KV heads in chunks of 128 keys: 17 to 64 chunks a row, in one or two batches a thread; 65 fold in a launch of their own
    run_and_check(_w(seq_len=[L], win=[24], top_p=[9], k_windows=[30]), device)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("q_heads,w_obs", [(5, 32), (5, 31), (7, 31), (7, 32)])
@pytest.mark.parametrize("heads,L", [(1, 700), (8, 16397)])
def test_rows_that_leave_a_tile_out(dtype, d, q_heads, w_obs, heads, L, device):
    # 155 to 224 rows: five to seven tiles of 32 rows for two row groups of three or four, in rings of every wave's own or (128 channels up to 9 MB and
    # above 112 MB) shared
    groups = 1 if L < 1000 else 5 if d == 128 else 9
    w = S.scaled_workload(S.make_workload("c4"), name="left_out", dtype=dtype, head_dim=d, n_q_heads=q_heads * heads, n_kv_heads=heads, w_obs=w_obs,
                          n_groups=groups, gamma=1, seq_len=[L], win=[24], top_p=[9], k_windows=[20])
    run_and_check(w, device, n_oracle=2, n_gather_cpu=1, stage_groups=[groups - 1])
