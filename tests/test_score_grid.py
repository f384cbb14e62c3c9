"""The launch grid and the argument block of the score passes (host code, no GPU), and parity of batches whose sequences lie on both sides
of what a workgroup reads of the block at once."""
import os
import subprocess

import pytest

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
