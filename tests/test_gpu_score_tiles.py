"""GPU parity of the score passes where their tiling can go wrong: every count of row tiles and row groups a wave
or workgroup can have, lengths around tiles, chunks and segments, windows that straddle them, and key rows too far
apart for 32-bit offsets."""
import pytest
import torch

import paper_2503_17922_amd as W
import wkv_synth as S
from tests import parity as P
from tests.test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(name="tiles", seed=311, dtype="bf16", n_groups=1, gamma=1, n_q_heads=8, n_kv_heads=2, head_dim=128, w_obs=16,
                seq_len=[700], win=[8], top_p=[8], k_windows=[10])
    base.update(kw)
    return S.Workload(**base)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("q_heads,w_obs", [(2, 5), (2, 32), (4, 32), (6, 32), (14, 16), (8, 32), (12, 32), (14, 32), (16, 32)])
def test_row_tiles(dtype, d, q_heads, w_obs, device):
    # 5 .. 256 softmax rows on two KV heads: one to eight row tiles a wave, one, two and four row groups
    run_and_check(_w(dtype=dtype, head_dim=d, n_q_heads=q_heads, w_obs=w_obs, seq_len=[901, 430], win=[24, 8], top_p=[9, 8], k_windows=[7, 20]), device)


@pytest.mark.parametrize("heads", [8, 16])
def test_lengths_around_tiles_and_chunks(heads, device):
    lens = [16, 17, 31, 32, 33, 79, 80, 81, 143, 144, 145, 207, 208, 271, 272, 273]
    w = _w(n_q_heads=heads, w_obs=16, seq_len=lens, win=[8, 100] * 8, top_p=[5, 30] * 8, k_windows=[min(2, -(-(n - 16) // wn)) for n, wn in zip(lens, [8, 100] * 8)])
    run_and_check(w, device)


@pytest.mark.parametrize("win,top_p", [(24, 7), (100, 40)])
def test_windows_across_segments(win, top_p, device):
    # chunks of 2048 keys and more: their token scores are pooled in several segments of whole windows
    w = S.scaled_workload(S.make_workload("c4"), name="segments", n_groups=4, gamma=1, win=[win], top_p=[top_p], k_windows=[4096 // win])
    run_and_check(w, device, n_oracle=5, n_gather_cpu=2, stage_groups=[1])


def test_key_rows_too_far_apart_for_32_bit_offsets(device):
    w = _w(w_obs=8, seq_len=[30], win=[4], top_p=[3], k_windows=[2], n_kv_heads=2, n_q_heads=8)
    st = P.DeviceState(w, device)
    st.compress()
    stride = (1 << 26) + 512                               # elements between tokens: 16 of them span more than 2 GiB
    flat = torch.zeros(stride * 29 + 512, dtype=torch.bfloat16, device=device)
    far = flat.as_strided((1, 2, 30, 128), (256, 128, stride, 1))
    k, v = far, far
    problem = P.make_problem(w, kv_strides=(256, 128, stride))
    k.copy_(st.k[0])
    wi, ti, nk = torch.empty_like(st.win_idx), torch.empty_like(st.tok_idx), torch.empty_like(st.n_keep)
    ko, vo = torch.empty_like(st.k_out[0]), torch.empty_like(st.v_out[0])
    W.wkv_compress_groups(problem, 1, 1, st.q, None, [k], [v], [ko], [vo], wi, ti, nk, st.workspace)
    torch.cuda.synchronize()
    assert torch.equal(wi, st.win_idx) and torch.equal(ti, st.tok_idx) and torch.equal(ko, st.k_out[0]) and torch.equal(vo, st.k_out[0])


@pytest.mark.parametrize("n_groups", [3, 5, 8])
def test_two_row_groups_by_size_of_the_key_stream(n_groups, device):
    # 256 softmax rows: key tiles fetched by every wave (101 MB of keys), by the waves of a slot together (168 MB), and
    # so by nontemporal loads (269 MB)
    w = S.scaled_workload(S.make_workload("c4"), name="streams", n_groups=n_groups, gamma=1, n_q_heads=64, seq_len=[16397], win=[24], top_p=[9],
                          k_windows=[80])
    run_and_check(w, device, n_oracle=4, n_gather_cpu=2, stage_groups=[1])
