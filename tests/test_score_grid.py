"""The launch grid and the argument block of the score passes (host code, no GPU), and parity of batches whose sequences lie on both sides
of what a workgroup reads of the block at once."""
import os
import subprocess

import pytest
import torch

import paper_2503_17922_amd as W
import wkv_synth as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_grid_and_arguments(tmp_path):
    from paper_2503_17922_amd import build as B
    exe = B.build_host_sanitized(str(tmp_path), [os.path.join(ROOT, "tests", "c", "score_grid.cpp"),
                                                 os.path.join(ROOT, "tests", "c", "launch_stubs.cpp")], exe_name="score_grid")
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)          # the sanitizer runtime must come first in the link order of the process
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,groups", [(7, 3, 1), (8, 8, 1), (9, 2, 3), (17, 4, 1), (16, 1, 2), (64, 1, 1)])
def test_batches_and_rows(batch, heads, groups, device):
    # 1 to 8 rows an XCD and rows that do not divide them; the first block of the sequences' ends, exactly, and one more of them
    from tests.test_gpu_parity import run_and_check
    lens = [40 + 97 * ((5 * b) % batch) for b in range(batch)]
    w = S.scaled_workload(S.make_workload("c4"), name="score_grid", n_q_heads=4 * heads, n_kv_heads=heads, n_groups=groups, gamma=1, seq_len=lens,
                          win=[8, 24] * (batch // 2) + [16] * (batch % 2), top_p=[5] * batch, k_windows=[1] * batch, planted_spans=0)
    run_and_check(w, device, n_oracle=4, n_gather_cpu=1, stage_groups=[groups - 1])


@pytest.mark.gpu
def test_as_many_heads_as_a_call_may_have(device):
    # two groups of 65535 KV heads: more rows than the grid of XCDs takes; each group as by a call of its own
    heads, L, d = 65535, 25, 64
    gen = torch.Generator(device=device).manual_seed(65535)
    mk = lambda *shape: torch.randn(shape, device=device, dtype=torch.float32, generator=gen).to(torch.bfloat16)
    q, k, v = [mk(1, heads, 1, d) for _ in range(2)], [mk(1, heads, L, d) for _ in range(2)], [mk(1, heads, L, d) for _ in range(2)]
    p = W.Problem(n_q_heads=heads, n_kv_heads=heads, head_dim=d, w_obs=1, seq_len=[L], win=[4], top_p=[4], k_windows=[2], dtype=W.WKV_BF16)
    nk = W.wkv_get_dims(p).nkeep_max
    ws = torch.empty(W.wkv_workspace_bytes(p, 2), dtype=torch.uint8, device=device)

    def call(groups):
        n = len(groups)
        out = [[torch.full((1, heads, nk, d), 7.0, dtype=torch.bfloat16, device=device) for _ in groups] for _ in range(2)]
        idx = [torch.full(shape, -7, dtype=torch.int32, device=device) for shape in ((n, 1, heads, 2), (n, 1, heads, nk), (n, 1, heads))]
        pick = lambda xs: [xs[g] for g in groups]
        W.wkv_compress_groups(p, n, 1, pick(q), None, pick(k), pick(v), out[0], out[1], *idx, ws)
        torch.cuda.synchronize()
        return out, idx

    out, idx = call([0, 1])
    for g in range(2):
        alone, own = call([g])
        for a, b in zip(idx, own):
            assert torch.equal(a[g], b[0])
        rows = idx[1][g, 0].to(torch.int64)[..., None].expand(-1, -1, d)
        for i, full in enumerate((k[g], v[g])):
            assert torch.equal(out[i][g], alone[i][0]) and torch.equal(out[i][g][0], full[0].gather(1, rows))
