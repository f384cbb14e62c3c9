"""Decode steps over long ranges by row counts: caches of every length around the ranges' ends, empty, full and with counts that are no counts, a
length of its own for every KV head; and counts of one sequence that change while the step runs."""
import numpy as np
import pytest
import torch

import paper_2503_17922_amd as W
from oracle import wkv_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,G,d", [("bf16", 4, 128), ("f16", 7, 64)])
@pytest.mark.parametrize("B,H,cap,chunk", [
    (2, 1, 70000, 320),         # two caches, 219 ranges each
    (21, 3, 6300, 320),         # 63 caches of 20 ranges, 65 of them
    (13, 5, 6300, 320),
    (16, 16, 1700, 320),        # 256 of six
    (64, 8, 1100, 384),         # 512 of three
])
def test_ranges_by_count(dtype, G, d, B, H, cap, chunk, device):
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    edges = [1, 0, cap - 1, chunk, -1, chunk + 1, cap, chunk - 1, 2 * chunk, 17, cap - chunk, 2 * chunk + 65, cap + 5, 3 * chunk - 63, 64]
    n = [edges[i % len(edges)] + (i // len(edges) if 0 < edges[i % len(edges)] < cap - 70 else 0) for i in range(B * H)]
    gen = torch.Generator(device=device).manual_seed(cap + G)
    mk = lambda *shape: torch.randn(shape, device=device, dtype=torch.float32, generator=gen).to(tdt)
    kc, vc, q, kn, vn = mk(B, H, cap, d), mk(B, H, cap, d), 2 * mk(B, G * H, d), mk(B, H, d), mk(B, H, d)
    for i, rows in enumerate(n):                    # what lies past the retained rows must not matter
        if 0 <= rows < cap:
            kc[i // H, i % H, rows:] = float("nan")
            vc[i // H, i % H, rows:] = float("nan")
    n_valid = torch.tensor(n, dtype=torch.int32, device=device).view(B, H).contiguous()
    shape = W.DecodeShape(batch=B, n_q_heads=G * H, n_kv_heads=H, head_dim=d, capacity=cap, dtype={"bf16": W.WKV_BF16, "f16": W.WKV_F16}[dtype])
    ws_bytes = W.wkv_decode_workspace_bytes(shape)
    assert ws_bytes == B * H * -(-cap // chunk) * G * (d + 2) * 4, "the caches are not divided as this case means them to be"
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device=device)     # NaNs
    out = torch.zeros((B, G * H, d), dtype=torch.float32, device=device)
    some = range(0, B * H, max(1, B * H // 75))
    f64 = lambda t: t.to("cpu").to(torch.float64).numpy()
    want = {}
    for i in some:
        b, h, rows = i // H, i % H, n[i]
        if 0 <= rows < cap:
            want[i], *_ = O.decode_step(f64(q[b, h * G:(h + 1) * G]), f64(kc[b, h, :rows]), f64(vc[b, h, :rows]), f64(kn[b, h]), f64(vn[b, h]))
    W.wkv_decode_step(shape, q, kn, vn, kc, vc, n_valid, out, ws)
    torch.cuda.synchronize()
    got, counts = f64(out), n_valid.cpu().flatten().tolist()
    for i in some:
        b, h, rows = i // H, i % H, n[i]
        mine = got[b, h * G:(h + 1) * G]
        if i in want:
            # products of 16-bit inputs, sums in fp32: about 1e-6 of the largest value; 1e-3 is what the other decode tests ask for
            np.testing.assert_allclose(mine, want[i], rtol=1e-3, atol=2e-5, err_msg=f"rows {rows} h{h}")
            assert torch.equal(kc[b, h, rows], kn[b, h]) and torch.equal(vc[b, h, rows], vn[b, h])
        else:
            assert np.isnan(mine).all(), f"rows {rows}"
    assert counts == [r + (0 <= r < cap) for r in n]


@pytest.mark.parametrize("dtype,G,d", [("bf16", 4, 128), ("f16", 7, 64)])
def test_counts_of_another_sequence_that_change_meanwhile(dtype, G, d, device):
    # a slot of the batch is filled anew on another stream while the step runs: its own output may be of either count, the others' are theirs
    B, H, cap, slot, steps = 16, 4, 6300, 3, 24
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device=device).manual_seed(G)
    mk = lambda *shape: torch.randn(shape, device=device, dtype=torch.float32, generator=gen).to(tdt)
    kc, vc, q, kn, vn = mk(B, H, cap, d), mk(B, H, cap, d), 2 * mk(B, G * H, d), mk(B, H, d), mk(B, H, d)
    n_valid = (400 + 5800 * torch.rand((B, H), device=device, generator=gen)).to(torch.int32)
    shape = W.DecodeShape(batch=B, n_q_heads=G * H, n_kv_heads=H, head_dim=d, capacity=cap, flags=W.WKV_DECODE_KEEP_COUNT,
                          dtype={"bf16": W.WKV_BF16, "f16": W.WKV_F16}[dtype])
    ws = torch.empty(W.wkv_decode_workspace_bytes(shape), dtype=torch.uint8, device=device)
    out = torch.zeros((steps + 1, B, G * H, d), dtype=torch.float32, device=device)
    W.wkv_decode_step(shape, q, kn, vn, kc, vc, n_valid, out[steps], ws)
    # (what a range that nobody takes would leave to the merge: NaN, from the workspace)
    clean = torch.full_like(ws, 0xFF)
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    for i in range(steps):
        ws.copy_(clean)
        W.wkv_decode_step(shape, q, kn, vn, kc, vc, n_valid, out[i], ws)
        with torch.cuda.stream(other):
            for j in range(8):
                n_valid[slot].fill_((500, 6200)[j % 2])
    torch.cuda.synchronize()
    rest = [b for b in range(B) if b != slot]
    for i in range(steps):
        assert torch.equal(out[i, rest], out[steps, rest]), f"step {i}"
