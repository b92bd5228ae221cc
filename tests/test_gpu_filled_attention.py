"""Attention over a filled cache (``ham_op_decode_attention``) on both sides of its split rule: rows and lengths where
it splits, does not, and leaves splits without slots; other group sizes and kv-head counts; fp32.

Against softmax attention in float64 on the stored values.  Tolerance: outputs are averages of unit normals, held as 16
significant bits (bf16 pairs) or fp32, with scores of the same precision: 2e-3 and 1e-5.

Marked ``gpu``: needs an MI355X and ``libham.so`` built in-tree.
"""
import pytest

from synth.configs import BF16, F32
from tests.gpu_util import act_rows, from_act, tiled_v

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,Hk,hd,lens", [
    (BF16, 32, 8, 128, [511]), (BF16, 32, 8, 128, [512]), (BF16, 32, 8, 128, [4097, 1]),
    (BF16, 32, 8, 64, [1023] * 2), (BF16, 32, 8, 64, [1024, 0, 33]), (BF16, 9, 3, 64, [2000, 40, 1999, 65]),
    (BF16, 8, 8, 128, [700] * 40), (BF16, 4, 2, 128, [9000]), (F32, 32, 8, 64, [511, 513, 700]), (F32, 6, 2, 128, [3001]),
    (BF16, 32, 8, 128, [4096] + [700] * 16), (BF16, 8, 2, 128, [500, 33, 0] * 5 + [8192]), (F32, 4, 2, 128, [4100, 16, 15])])
def test_filled_attention_splits(dtype, H, Hk, hd, lens):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_20438_amd import ham
    dev, R, S = "cuda:0", len(lens), (max(lens) + 63) // 64 * 64
    g = torch.Generator(device=dev).manual_seed(11)
    t = torch.bfloat16 if dtype == BF16 else torch.float32
    q = torch.randn(R, H * hd, generator=g, device=dev)
    K = torch.randn(R, Hk, S, hd, generator=g, device=dev).to(t)
    V = torch.randn(R, Hk, S, hd, generator=g, device=dev).to(t)
    n = torch.tensor(lens, dtype=torch.int32, device=dev)
    for r in range(R):   # nothing past a row's length may reach its output
        V[r, :, lens[r]:] = float("nan")
    qa = act_rows(torch, q, dtype)
    out = torch.full_like(qa, 7.0)
    ws = torch.empty(ham.ham_op_attention_workspace_bytes(R, H, Hk, hd), dtype=torch.uint8, device=dev)
    ham.ham_op_decode_attention(dtype, qa, K, tiled_v(torch, V), n, torch.ones_like(n), max(lens), out, ws,
                                torch.cuda.current_stream().cuda_stream, H, Hk, hd, S)
    got = from_act(torch, out, H * hd, dtype).double().cpu().view(R, H, hd)
    qd = from_act(torch, qa, H * hd, dtype).double().cpu().view(R, H, hd)
    for r in range(R):
        if lens[r] == 0:
            assert torch.all(got[r] == 0)
            continue
        for h in range(H):
            k, v = (x[r, h * Hk // H, :lens[r]].double().cpu() for x in (K, V))
            ref = torch.softmax(k @ qd[r, h] / hd ** 0.5, 0) @ v
            assert (got[r, h] - ref).abs().max() <= (2e-3 if dtype == BF16 else 1e-5), (r, h)
