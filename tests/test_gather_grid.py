"""The gather's workgroups: the grid and the rule of their size (host code, no GPU), and parity of batches on every side of that rule, with
rows beyond a sequence's budget where the caller's own index lists have them."""
import os
import subprocess

import pytest
import torch

import paper_2503_17922_amd as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_grid_and_rule(tmp_path):
    from paper_2503_17922_amd import build as B
    exe = B.build_host_sanitized(str(tmp_path), [os.path.join(ROOT, "tests", "c", "gather_grid.cpp"),
                                                 os.path.join(ROOT, "tests", "c", "launch_stubs.cpp")], exe_name="gather_grid")
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)          # the sanitizer runtime must come first in the link order of the process
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f16", 128), ("f32", 128)])
@pytest.mark.parametrize("keep_padding", [False, True])
@pytest.mark.parametrize("budgets", [[257, 60, 3, 0], [257, 120, 100, 0], [66, 2, 1, 1], [15, 1, 0, 2]])     # 0.32, 0.47, 0.28, 0.35 of the room
def test_budgets_of_their_own(dtype, d, keep_padding, budgets, device):
    H, L, w_obs, layers, B = 3, 600, 1, 2, len(budgets)
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    nk = max(budgets) + w_obs
    p = W.Problem(n_q_heads=H, n_kv_heads=H, head_dim=d, w_obs=w_obs, seq_len=[L] * B, win=[1] * B, top_p=[1] * B, k_windows=budgets,
                  dtype={"bf16": W.WKV_BF16, "f16": W.WKV_F16, "f32": W.WKV_F32}[dtype], flags=W.WKV_KEEP_PADDING if keep_padding else 0)
    gen = torch.Generator(device=device).manual_seed(nk + d)
    k, v = ([torch.randn((B, H, L, d), device=device, generator=gen).to(tdt) for _ in range(layers)] for _ in range(2))
    idx = torch.randint(0, L, (B, H, nk), device=device, generator=gen, dtype=torch.int32)
    keep = torch.tensor([[n + w_obs, max(n, 1), nk] for n in budgets], dtype=torch.int32, device=device)        # the last: all the room
    ko, vo = ([torch.full((B, H, nk, d), 7.0, device=device, dtype=tdt) for _ in range(layers)] for _ in range(2))
    W.wkv_gather_group(p, k, v, idx, keep, ko, vo)
    torch.cuda.synchronize()
    for src, dst in zip(k + v, ko + vo):
        for b in range(B):
            for h in range(H):
                n = int(keep[b, h])
                assert torch.equal(dst[b, h, :n], src[b, h][idx[b, h, :n].long()])
                assert bool((dst[b, h, n:] == (7.0 if keep_padding else 0.0)).all())
