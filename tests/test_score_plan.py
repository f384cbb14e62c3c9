"""The score passes' choice of kernels: what the launch plan asks for on both sides of its lines (host code, no GPU), and GPU parity of
the row counts that only such a choice reaches."""
import os
import subprocess

import pytest

import wkv_synth as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lines_of_the_plan(tmp_path):
    from paper_2503_17922_amd import build as B
    exe = B.build_host_sanitized(str(tmp_path), [os.path.join(ROOT, "tests", "c", "score_plan.cpp"),
                                                 os.path.join(ROOT, "tests", "c", "launch_stubs.cpp")], exe_name="score_plan")
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)          # the sanitizer runtime must come first in the link order of the process
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,q_heads,w_obs,n_groups,L", [
    ("bf16", 128, 28, 16, 1, 4099),         # 112 rows in chunks of 128 keys: tiles of 32 rows
    ("bf16", 128, 28, 14, 1, 12011),        # 98 rows in larger ones: of 16
    ("f16", 128, 28, 16, 2, 16397),
    ("f16", 64, 28, 16, 8, 16397),          # 64 channels, two workgroups a compute unit: of 16
    ("bf16", 128, 28, 16, 17, 16397),       # the same by nontemporal loads
    ("bf16", 64, 28, 16, 33, 16397),
    ("bf16", 64, 32, 16, 33, 16397),        # 128 rows by nontemporal loads: of 32
    ("f16", 64, 12, 16, 33, 16397),         # 48
])
def test_row_counts_and_tiles(dtype, d, q_heads, w_obs, n_groups, L, device):
    from tests.test_gpu_parity import run_and_check
    w = S.scaled_workload(S.make_workload("c4"), name="row_counts", dtype=dtype, head_dim=d, n_q_heads=q_heads, n_kv_heads=4, w_obs=w_obs,
                          n_groups=n_groups, gamma=1, seq_len=[L], win=[24], top_p=[9], k_windows=[80])
    run_and_check(w, device, n_oracle=3, n_gather_cpu=1, stage_groups=[n_groups - 1])
