"""The decode step's blocks of 16 rows: row counts around the ends of single and paired blocks, in ranges of one block for each of eight
waves and of 1 to 9 pairs for each of four; and the divisions by multiplication that find a workgroup's head."""
import os
import subprocess

import numpy as np
import pytest
import torch

import paper_2503_17922_amd as W
from oracle import wkv_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_divisions_by_multiplication(tmp_path):
    from paper_2503_17922_amd import build as B
    exe = B.build_host_sanitized(str(tmp_path), [os.path.join(ROOT, "tests", "c", "division_magic.cpp"),
                                                 os.path.join(ROOT, "tests", "c", "launch_stubs.cpp")], exe_name="division_magic")
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)          # the sanitizer runtime must come first in the link order of the process
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,G,d", [("bf16", 4, 128), ("f16", 8, 128), ("f16", 2, 64)])
@pytest.mark.parametrize("B,cap,ranges", [
    (96, 130, 2),           # ranges of 128 rows: a block for each of eight waves with 4 heads of 128 channels, else a pair for each of four
    (40, 770, 4),           # 256 rows: two pairs a wave; with 128 channels 126 MB, of which the values are streamed
    (96, 770, 2),           # 448 rows: three pairs and a block; with 128 channels 303 MB, keys streamed too
    (96, 2300, 2),          # 1152 rows: nine pairs
])
def test_pairs_of_blocks(dtype, G, d, B, cap, ranges, device):
    H, tdt = 8, {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    edges = [0, 1, 15, 16, 17, 63, 64, 65, 80, 112, 113, 127, 128, 129, 191, 192, 193, 240, 255, 256, 257, 319, 320, 321, 383, 384, 385]
    rows = [n for n in edges if n < cap]
    rows = (rows + [cap - 1 - n for n in rows] * 8)[:B]
    gen = torch.Generator(device=device).manual_seed(cap + G)
    mk = lambda *shape: torch.randn(shape, device=device, dtype=torch.float32, generator=gen).to(tdt)
    kc, vc, q, kn, vn = mk(B, H, cap, d), mk(B, H, cap, d), 2 * mk(B, G * H, d), mk(B, H, d), mk(B, H, d)
    for b, n in enumerate(rows):                    # what lies past the retained rows must not matter
        kc[b, :, n:] = float("nan")
        vc[b, :, n:] = float("nan")
    n_valid = torch.tensor(rows, dtype=torch.int32, device=device)[:, None].repeat(1, H).contiguous()
    shape = W.DecodeShape(batch=B, n_q_heads=G * H, n_kv_heads=H, head_dim=d, capacity=cap,
                          dtype={"bf16": W.WKV_BF16, "f16": W.WKV_F16}[dtype])
    ws_bytes = W.wkv_decode_workspace_bytes(shape)
    assert ws_bytes == B * H * ranges * G * (d + 2) * 4, "the caches are not divided as this case means them to be"
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device=device)     # NaNs
    out = torch.zeros((B, G * H, d), dtype=torch.float32, device=device)
    f64 = lambda t: t.to("cpu").to(torch.float64).numpy()
    k0, v0 = f64(kc), f64(vc)
    W.wkv_decode_step(shape, q, kn, vn, kc, vc, n_valid, out, ws)
    torch.cuda.synchronize()
    got, qh, knh, vnh = f64(out), f64(q), f64(kn), f64(vn)
    for b, n in enumerate(rows):
        h = b % H
        want, *_ = O.decode_step(qh[b, h * G:(h + 1) * G], k0[b, h, :n], v0[b, h, :n], knh[b, h], vnh[b, h])
        # products of 16-bit inputs, sums in fp32: about 1e-6 of the largest value; 1e-3 is what the other decode tests ask for
        np.testing.assert_allclose(got[b, h * G:(h + 1) * G], want, rtol=1e-3, atol=2e-5, err_msg=f"rows {n} h{h}")


@pytest.mark.gpu
@pytest.mark.parametrize("G", [2, 7])
def test_rows_more_than_4_gib_apart(G, device):
    # keys and values of one buffer, a row's bytes past 32 bits; ranges of a block for each of eight waves, and of pairs
    d, cap, n, st = 128, 4, 3, (1 << 31) + 1024
    buf = torch.empty(3 * st + 1024, dtype=torch.bfloat16, device=device)
    row = lambda i, at: buf[i * st + at: i * st + at + d]
    gen = torch.Generator(device=device).manual_seed(5)
    mk = lambda *shape: torch.randn(shape, device=device, dtype=torch.float32, generator=gen).to(torch.bfloat16)
    k, v, q, kn, vn = mk(n, d), mk(n, d), 2 * mk(1, G, d), mk(1, 1, d), mk(1, 1, d)
    for i in range(n):
        row(i, 0).copy_(k[i])
        row(i, 512).copy_(v[i])
    shape = W.DecodeShape(batch=1, n_q_heads=G, n_kv_heads=1, head_dim=d, capacity=cap, dtype=W.WKV_BF16, cache_strides=(d, d, st))
    n_valid = torch.tensor([[n]], dtype=torch.int32, device=device)
    out = torch.zeros((1, G, d), dtype=torch.float32, device=device)
    W.wkv_decode_step(shape, q, kn, vn, buf, buf[512:], n_valid, out, torch.empty(W.wkv_decode_workspace_bytes(shape), dtype=torch.uint8, device=device))
    torch.cuda.synchronize()
    f64 = lambda t: t.to("cpu").to(torch.float64).numpy()
    want, *_ = O.decode_step(f64(q[0]), f64(k), f64(v), f64(kn[0, 0]), f64(vn[0, 0]))
    np.testing.assert_allclose(f64(out[0]), want, rtol=1e-3, atol=2e-5)
    assert torch.equal(row(n, 0), kn[0, 0]) and torch.equal(row(n, 512), vn[0, 0])
