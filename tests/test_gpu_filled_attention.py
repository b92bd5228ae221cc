"""Attention over a filled cache (``ham_op_decode_attention``) on both sides of its split rule, against softmax attention
in float64 on the stored values, row by row within FILLED_TOL of the output's root mean square.

Marked ``gpu``: needs an MI355X and ``libham.so`` built in-tree.
"""
import pytest

from synth.configs import BF16
from tests.attention_bounds import FILLED, FILLED_TOL
from tests.gpu_util import act_rows, from_act, tiled_v

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,Hk,hd,lens", FILLED)
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
    worst = 0.0
    for r in range(R):
        if lens[r] == 0:
            assert torch.all(got[r] == 0)
            continue
        for h in range(H):
            k, v = (x[r, h * Hk // H, :lens[r]].double().cpu() for x in (K, V))
            ref = torch.softmax(k @ qd[r, h] / hd ** 0.5, 0) @ v
            e = float((got[r, h] - ref).abs().max() / ref.square().mean().sqrt())
            worst = max(worst, e)
            assert e <= FILLED_TOL[dtype], (r, h, e)
    print("worst error over RMS", worst, flush=True)
