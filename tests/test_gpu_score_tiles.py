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
    # 5 .. 256 softmax rows on two KV heads: one to four tiles of 32 rows a wave and one or two row groups with 16-bit inputs, one to eight
    # tiles of 16 rows and one, two or four groups with fp32 (16-row tiles of 16-bit inputs: test_gpu_score_streams)
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


def _compress_far_apart(w, device, stride):
    """Compresses ``w`` with ``stride`` elements from token to token, the same keys and values for all groups (the storage of
    sequences and heads lies between two tokens), and compares with contiguous caches."""
    B, H, L, d, n = w.batch, w.n_kv_heads, max(w.seq_len), w.head_dim, w.n_groups
    assert B * H * d <= stride and w.gamma == 1
    near = 0.05 * torch.randn((B, H, L, d), dtype=torch.float32, device=device, generator=torch.Generator(device=device).manual_seed(w.seed))
    near = near.to(torch.bfloat16)
    flat = torch.zeros(stride * (L - 1) + B * H * d, dtype=torch.bfloat16, device=device)
    far = flat.as_strided((B, H, L, d), (H * d, d, stride, 1))
    far.copy_(near)
    st = P.DeviceState(w, device)
    outs = []
    for kv, strides in ((near, None), (far, (H * d, d, stride))):
        problem = P.make_problem(w, kv_strides=strides) if strides else P.make_problem(w)
        wi, ti, nk = (torch.full_like(t, -7) for t in (st.win_idx, st.tok_idx, st.n_keep))
        ko, vo = [torch.zeros_like(t) for t in st.k_out], [torch.zeros_like(t) for t in st.v_out]
        W.wkv_compress_groups(problem, n, 1, st.q, None, [kv] * n, [kv] * n, ko, vo, wi, ti, nk, st.workspace)
        torch.cuda.synchronize()
        outs.append([wi, ti, nk, *ko, *vo])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# a tile's rows lie within 32-bit offsets of its 16 rows while 16 of them span less than 2 GiB: from 2^26 elements of two bytes on they do not
@pytest.mark.parametrize("stride", [(1 << 26) + 512, 1 << 26, (1 << 26) - 8])
def test_key_rows_far_apart(stride, device):
    # whole 32-row tiles and the tail of one
    _compress_far_apart(_w(w_obs=8, seq_len=[70], win=[4], top_p=[3], k_windows=[5]), device, stride)


def test_key_rows_far_apart_in_shared_tiles(device):
    # two row groups of 128 channels fetch a tile of 32 rows together above 112 MB of scored keys, and the offsets of the second reach over 31 rows: nearly 4 GiB
    B, n, stride = 64, 32, (1 << 26) - 8
    w = _w(n_groups=n, n_q_heads=20, w_obs=31, n_kv_heads=4, seq_len=[70] * B, win=[4] * B, top_p=[3] * B, k_windows=[5] * B)
    assert B * n * w.n_kv_heads * 70 * 256 > 112 << 20
    _compress_far_apart(w, device, stride)


@pytest.mark.parametrize("n_groups", [3, 5, 8])
def test_two_row_groups_by_size_of_the_key_stream(n_groups, device):
    # 256 softmax rows: key tiles fetched by every wave (101 MB of keys), by the waves of a slot together (168 MB), and
    # so by nontemporal loads (269 MB)
    w = S.scaled_workload(S.make_workload("c4"), name="streams", n_groups=n_groups, gamma=1, n_q_heads=64, seq_len=[16397], win=[24], top_p=[9],
                          k_windows=[80])
    run_and_check(w, device, n_oracle=4, n_gather_cpu=2, stage_groups=[1])
