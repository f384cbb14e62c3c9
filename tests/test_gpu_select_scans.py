"""Top-k at window counts around waves, workgroups and the scores that a thread requests together, with spread, equal, few-valued and infinite
scores, against a stable sort."""
import numpy as np
import pytest
import torch

import paper_2503_17922_amd as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw", [1, 2, 63, 64, 65, 255, 256, 257, 511, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 16385])
def test_top_k_by_window_count(nw, device):
    H, win, w_obs = 6, 3, 2
    L = nw * win - 1 + w_obs                       # the last window is partial
    rng = np.random.default_rng(nw)
    s = rng.standard_normal((1, H, nw)).astype(np.float32)
    s[0, 1] = 0.25                                 # ties everywhere: lower indices win
    s[0, 2] = rng.integers(0, 3, nw)
    s[0, 3] = np.abs(s[0, 3]) * 1e-30
    s[0, 4, rng.integers(0, nw)] = np.inf
    s[0, 5, rng.integers(0, nw, max(nw // 2, 1))] = -np.inf
    for k in sorted({1, (nw + 1) // 2, nw}):
        p = W.Problem(n_q_heads=H, n_kv_heads=H, head_dim=64, w_obs=w_obs, seq_len=[L], win=[win], top_p=[win], k_windows=[k], dtype=W.WKV_BF16)
        wi = torch.full((1, H, k), -7, dtype=torch.int32, device=device)
        ti = torch.full((1, H, k * win + w_obs), -7, dtype=torch.int32, device=device)
        nk = torch.zeros((1, H), dtype=torch.int32, device=device)
        W.wkv_topk_windows(p, torch.from_numpy(s).to(device), wi, ti, nk)
        torch.cuda.synchronize()
        for h in range(H):
            want = np.sort(np.argsort(-s[0, h], kind="stable")[:k])
            assert np.array_equal(wi[0, h].cpu().numpy(), want), (nw, k, h)
            tok = np.concatenate([np.arange(w * win, min((w + 1) * win, L - w_obs)) for w in want] + [np.arange(L - w_obs, L)])
            assert int(nk[0, h]) == len(tok) and np.array_equal(ti[0, h, : len(tok)].cpu().numpy(), tok)
            assert bool((ti[0, h, len(tok):] == -1).all())


@pytest.mark.parametrize("nw", [1, 100, 2047, 2048, 4096])
def test_room_past_the_windows_of_a_sequence(nw, device):
    # a thread's first scores are requested before its sequence is known: what lies past the windows of a shorter one counts for nothing
    H, w_obs, room = 2, 1, 4200
    rng = np.random.default_rng(nw)
    s = rng.standard_normal((3, H, room)).astype(np.float32)
    s[1, :, nw:] = np.nan
    s[1, 1, nw:] = np.inf
    k = [7, (nw + 1) // 2, 0]
    p = W.Problem(n_q_heads=H, n_kv_heads=H, head_dim=64, w_obs=w_obs, seq_len=[room + w_obs, nw + w_obs, w_obs], win=[1] * 3, top_p=[1] * 3,
                  k_windows=k, dtype=W.WKV_BF16)
    d = W.wkv_get_dims(p)
    wi = torch.full((3, H, d.k_max), -7, dtype=torch.int32, device=device)
    ti = torch.full((3, H, d.nkeep_max), -7, dtype=torch.int32, device=device)
    nk = torch.zeros((3, H), dtype=torch.int32, device=device)
    W.wkv_topk_windows(p, torch.from_numpy(s).to(device), wi, ti, nk)
    torch.cuda.synchronize()
    for b, n in enumerate((room, nw, 0)):
        for h in range(H):
            want = np.sort(np.argsort(-s[b, h, :n], kind="stable")[: k[b]])
            assert np.array_equal(wi[b, h, : k[b]].cpu().numpy(), want) and bool((wi[b, h, k[b]:] == -1).all())
            assert int(nk[b, h]) == k[b] + w_obs and np.array_equal(ti[b, h, : k[b]].cpu().numpy(), want)


@pytest.mark.parametrize("seq_len,k", [([9000], 476), ([9000], 477), ([5200, 4000], 156), ([5200, 4000], 157)])
def test_compact_caches_around_the_limit_of_one_launch(seq_len, k, device):
    # 60 MB (one sequence) and 40 MB (two) exactly, and a window more: one launch, and two
    import wkv_synth as S
    from tests.test_gpu_parity import run_and_check
    n = len(seq_len)
    nkeep = k * 8 + 32
    limit = (60 if n == 1 else 40) << 20
    assert (64 * n * nkeep * 256 <= limit) == (k in (476, 156)) and abs(64 * n * nkeep * 256 - limit) <= 64 * n * 8 * 256
    w = S.scaled_workload(S.make_workload("c4"), name="limit", n_groups=1, gamma=4, seq_len=seq_len, win=[8] * n, top_p=[8] * n, k_windows=[k] + [k // 2] * (n - 1))
    run_and_check(w, device, n_oracle=2, n_gather_cpu=1, stage_groups=[0])
