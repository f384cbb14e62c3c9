"""GPU parity of the score passes on streams of keys large enough for each way of fetching them, in the types and row
widths that the other tests take through small streams only: from 9 to 112 MB of scored keys (64 channels: up to 192 MB) every wave fetches its own tiles
where there are two row groups of 16-bit inputs, else the waves of a slot share them, above 256 MB by nontemporal loads.  16-bit inputs of
one row group take tiles of 16 rows on nontemporal streams of 128 channels and where 97 to 112 rows have much to compute, else of 32
(test_score_plan has the rule).  Chunks hold several segments of pooled token scores (1024 of them with four row groups, else 2048)."""
import pytest

import wkv_synth as S
from tests.test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.mark.parametrize("dtype,d,q_heads,n_groups,least,most", [
    ("f32", 128, 8, 5, 256, 512),           # 32 rows, one row group, nontemporal
    ("f32", 128, 32, 5, 256, 512),          # 128 rows, two
    ("f32", 128, 64, 3, 0, 256),            # 256 rows, four: two segments, plain loads
    ("f32", 128, 64, 5, 256, 512),          # the same, nontemporal
    ("f32", 64, 32, 9, 256, 512),           # 128 rows, one row group of eight tiles
    ("f32", 64, 64, 9, 256, 512),           # 256 rows, two
    ("bf16", 64, 64, 3, 0, 192),            # rings of their own
    ("bf16", 64, 64, 10, 0, 192),
    ("f16", 64, 64, 10, 0, 192),
    ("bf16", 64, 64, 14, 192, 256),         # shared
    ("f16", 64, 48, 14, 192, 256),          # 192 rows, shared
    ("bf16", 128, 48, 2, 9, 112),           # 192 rows, rings of their own
    ("bf16", 128, 56, 6, 112, 256),         # 224 rows, shared
    ("f16", 64, 64, 17, 256, 512),          # shared, nontemporal
    ("f16", 64, 32, 17, 256, 512),          # one row group, nontemporal
    ("f16", 128, 56, 9, 256, 512),          # 224 rows, shared, nontemporal
])
def test_key_streams(dtype, d, q_heads, n_groups, least, most, device):
    L = 16397
    keys = n_groups * 8 * L * d * (4 if dtype == "f32" else 2)
    assert least * MB < keys <= most * MB, "the size does not choose the kernel it is meant to"
    w = S.scaled_workload(S.make_workload("c4"), name="streams", dtype=dtype, head_dim=d, n_q_heads=q_heads, n_groups=n_groups, gamma=1,
                          seq_len=[L], win=[24], top_p=[9], k_windows=[80])
    run_and_check(w, device, n_oracle=3, n_gather_cpu=1, stage_groups=[1])


@pytest.mark.parametrize("dtype,d,q_heads,w_obs,n_groups,least,most", [
    # 16-row tiles by nontemporal loads: one to eight of them
    ("bf16", 128, 8, 5, 9, 256, 512),
    ("f16", 128, 8, 16, 9, 256, 512),
    ("bf16", 128, 8, 31, 9, 256, 512),
    ("f16", 128, 16, 32, 9, 256, 512),
    ("bf16", 128, 24, 31, 9, 256, 512),
    ("f16", 128, 56, 16, 9, 256, 512),
    ("bf16", 128, 56, 15, 9, 256, 512),
    ("bf16", 128, 32, 31, 9, 256, 512),
    # 32-row tiles by nontemporal loads: one to four of them; two row groups, the last tile of the second without rows
    ("bf16", 64, 8, 5, 17, 256, 512),
    ("f16", 64, 8, 32, 17, 256, 512),
    ("bf16", 64, 16, 31, 17, 256, 512),
    ("f16", 64, 24, 32, 17, 256, 512),
    ("bf16", 64, 40, 31, 17, 256, 512),
    ("bf16", 128, 40, 31, 9, 256, 512),
    ("f16", 128, 48, 31, 9, 256, 512),
])
def test_row_counts(dtype, d, q_heads, w_obs, n_groups, least, most, device):
    L = 16397
    keys = n_groups * 8 * L * d * 2
    assert least * MB < keys <= most * MB, "the size does not choose the kernel it is meant to"
    w = S.scaled_workload(S.make_workload("c4"), name="rows", dtype=dtype, head_dim=d, n_q_heads=q_heads, n_groups=n_groups, gamma=1, w_obs=w_obs,
                          seq_len=[L], win=[24], top_p=[9], k_windows=[80])
    run_and_check(w, device, n_oracle=2, n_gather_cpu=1, stage_groups=[1])
