"""Launch planning (host code, no GPU): the chunk lengths of the score passes and what picking them costs, the order of the
decode step's key ranges."""
import os
import subprocess
import time

import pytest

import paper_2503_17922_amd as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("program", ["launch_plan", "decode_ranges"])
def test_plans(program, tmp_path):
    # chunk lengths are those of a search of every length; every key range is taken once, with the rows of a batch spread over the chip
    from paper_2503_17922_amd import build as B
    exe = B.build_host_sanitized(str(tmp_path), [os.path.join(ROOT, "tests", "c", program + ".cpp"),
                                                 os.path.join(ROOT, "tests", "c", "launch_stubs.cpp")], exe_name=program)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)          # the sanitizer runtime must come first in the link order of the process
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


def _microseconds(f, calls=100):
    t = time.perf_counter()
    for _ in range(calls):
        f()
    return (time.perf_counter() - t) / calls * 1e6


def test_planning_a_large_batch_costs_little_more_than_validating_it():
    lens = [4096 + 37 * i for i in range(64)]
    p = W.Problem(n_q_heads=32, n_kv_heads=8, head_dim=128, w_obs=32, seq_len=lens, win=[8] * 64, top_p=[8] * 64, k_windows=[64] * 64,
                  dtype=W.WKV_BF16)
    for groups in (1, 8):
        # one after the other, as the processor's clock changes: validation alone, then validation and planning
        pairs = [(_microseconds(lambda: W.wkv_get_dims(p)), _microseconds(lambda: W.wkv_workspace_bytes(p, groups))) for _ in range(40)]
        validation, planning = min(pairs, key=lambda x: x[1] / x[0])
        assert planning < 5 * validation, f"{groups} groups: {planning:.1f} us, validation alone {validation:.1f} us"
