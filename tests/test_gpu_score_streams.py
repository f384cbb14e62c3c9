"""GPU parity of the score passes on streams of keys large enough for each way of fetching them, in the types and row
widths that the other tests take through small streams only: up to 128 MB of scored keys every wave fetches its own tiles where
there are two row groups of 16-bit inputs, above that the waves of a slot share them, above 256 MB by nontemporal loads.  Chunks
hold several segments of pooled token scores (1024 of them with four row groups, else 2048)."""
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
    ("bf16", 64, 64, 3, 0, 128),            # rings of their own
    ("bf16", 64, 64, 10, 128, 256),         # shared
    ("f16", 64, 64, 10, 128, 256),
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
