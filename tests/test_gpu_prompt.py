"""The prompt kernels at the edges of their tiles: every layer's K and V of every row of a prefill, and its
decision, against the float64 oracle.

The model's widths end inside the GEMM tiles of 128 and 256 columns (q/k/v 768, d 544, gate/up 2112 columns, k-ranges
of 17, 16 and 33 fragments); the prompt lengths end inside its tiles of 128 rows and the attention's tiles of 32 (fp32:
16).
Tolerance: the largest difference over the largest value, at most 2e-2 in bf16 (the decisions' tolerance) and 1e-4 in
fp32; a wrong row or column is off by the order of the value itself.  Attention alone is held to a closer bound, on inputs
small enough that its output decides the next layer's K and V (ATTN_TOL).

Marked ``gpu``: needs an MI355X and ``libham.so`` built in-tree.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import OracleHam
from synth.configs import BF16, F32
from tests.gpu_util import SMALL16, TOL, config_for, run_gpu
from tests.attention_bounds import ATTN_TOL, FORMS, attention_inputs, attention_shape, row_error
from tests.rules_util import rules

pytestmark = pytest.mark.gpu

EDGES = dataclasses.replace(SMALL16, n_layers=3, d_model=544, ffn_dim=1056, vocab=1024, micro_layers=1)


def _check(shp, B, P, rows, seed=301):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_20438_amd import ham
    prompts = synth.prompt_ids(seed + 1, B, P, shp.vocab)
    sched = 1 + (np.arange(B, dtype=np.int32)[:, None] + np.array([[3, 0]], dtype=np.int32)) % 4   # 4, 1, 2, 3, ...
    om = OracleHam(shp, seed)
    rt = ham.HamRuntime(config_for(shp, B, P, 1), seed)
    orc, caches = {}, {}
    for b in rows:
        orc[b] = om.generate(prompts[b], 0, 0, forced=lambda st, b=b: int(sched[b, st]), record=True)
        caches[b] = om.last_caches
    teacher = [orc[b].groups if b in orc else [[(7 * b + j) % shp.vocab for j in range(sched[b, 0])]] for b in range(B)]
    res = run_gpu(rt, prompts, [0] * B, 0, sched, teacher=teacher, debug_steps=1)
    tol = TOL[shp.dtype]
    kv = [[t.cpu().numpy().astype(np.float64) for t in rt.kv_cache(l, P)] for l in range(shp.n_layers)]
    for b in rows:
        for dec in orc[b].decisions:   # the first from the base model, the others through the context rows
            assert np.max(np.abs(res.logits[(b, 0, dec.k)] - dec.logits)) <= tol, (b, dec.k)
            assert np.max(np.abs(res.hidden[(b, 0, dec.k)] - dec.h)) <= tol, (b, dec.k)
        for l in range(shp.n_layers):
            for i, name in enumerate("KV"):
                ref = np.transpose(caches[b][l][i], (1, 0, 2))
                err = np.max(np.abs(kv[l][i][b] - ref), axis=(0, 2)) / np.max(np.abs(ref))
                assert err.max() <= tol, (b, l, name, int(err.argmax()), float(err.max()))
    assert all(s["kv_len"] == P and s["device_error"] == 0 for s in rt.kv_stats())


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("prompt", [65, 130, 257, 300, 513])   # the batched GEMM's last row count, whole and cut tiles
def test_prompt_rows_past_a_tile(dtype, prompt):
    _check(dataclasses.replace(EDGES, dtype=dtype), 1, prompt, [0])


# Batches run as one stream of rows in chunks: several prompts in a chunk, prompts cut by a chunk's end (1100 rows: 3
# chunks of 1152 for 3 prompts; 700: 2 of 1792), chunks that end exactly at a prompt's end, one-token prompts.
@pytest.mark.parametrize("shape,batch,prompt,rows", [
    (EDGES, 5, 1, [0, 4]), (EDGES, 3, 77, [0, 1, 2]), (EDGES, 17, 16, [0, 8, 16]), (EDGES, 4, 64, [0, 3]),
    (EDGES, 3, 1100, [0, 1, 2]), (EDGES, 5, 700, [1, 2, 4]), (EDGES, 2, 2048, [1]),
    (dataclasses.replace(EDGES, n_layers=1), 3, 70, [0, 2]),
    (dataclasses.replace(EDGES, n_layers=3, ctx_layer_set=(1, 2)), 3, 70, [0, 2]),
    (dataclasses.replace(EDGES, dtype=F32), 3, 77, [0, 1, 2]), (dataclasses.replace(EDGES, dtype=F32), 3, 1100, [1])])
def test_prompts_share_chunks(shape, batch, prompt, rows):
    _check(shape, batch, prompt, rows)


# 9 to 33 rows: the kernel of small row counts (row tiles of 16, eight waves that share 128 columns and split k) as a
# prompt's plain rows and as the normed rows of the first micro step (4 rows a sequence), at widths that end inside its
# 128 columns and give its waves unequal shares of the fragments (20 of d = 640); q/k/v 768, gate/up 2112 columns.
@pytest.mark.parametrize("batch,prompt", [(1, 9), (4, 4), (3, 6), (8, 4), (11, 3)])
def test_small_row_counts(batch, prompt):
    _check(dataclasses.replace(EDGES, d_model=640), batch, prompt, sorted({0, batch // 2, batch - 1}))


# the same row counts at a width whose second round of 128-column groups is nearly empty (gate/up 33,280 columns: 260
# groups), where the batched kernel takes them
@pytest.mark.parametrize("batch,prompt", [(3, 4), (7, 4)])
def test_small_row_counts_wide(batch, prompt):
    _check(dataclasses.replace(EDGES, n_layers=2, d_model=256, ffn_dim=16640), batch, prompt, [0, batch - 1])


# The prompt attention's two forms (rows, keys) at every group size, in chunks that hold several sequences, cut sequences and
# end inside a tile; positions skip as those of fused inputs do.
@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("grp,hk,hd,batch,prompt,keys", FORMS)
def test_prompt_attention_forms(dtype, grp, hk, hd, batch, prompt, keys):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_20438_amd import ham
    shp = attention_shape(grp, hk, hd, dtype)
    total = batch * prompt
    chunk = min(2048, -(-(-(-total // -(-total // 2048))) // 128) * 128)   # equal chunks of whole 128 rows, at most 2,048
    assert rules().prompt_keys(min(chunk, total), 0, prompt, shp.n_heads, shp.n_kv_heads) == keys
    X, pos = attention_inputs(batch, prompt, shp)
    rt = ham.HamRuntime(config_for(shp, batch, 4 * prompt, 1), 5)
    rt.prefill_embeds(torch.from_numpy(X).to("cuda:0"), torch.from_numpy(pos).to("cuda:0"), [0] * batch,
                      torch.ones(batch, dtype=torch.int32, device="cuda:0"))
    kv = [[t.cpu().numpy().astype(np.float64) for t in rt.kv_cache(l, prompt)] for l in range(shp.n_layers)]
    om = OracleHam(shp, 5)
    worst = 0.0
    for b in sorted({0, batch // 2, batch - 1}):
        caches = om.new_caches(shp.n_layers)
        om.forward_rows(om.layers[:shp.n_layers], X[b], pos[b], caches)
        for l in range(shp.n_layers):
            for i in range(2):
                e = row_error(np.transpose(kv[l][i][b], (1, 0, 2)), caches[l][i])
                worst = max(worst, e.max())
                assert e.max() <= ATTN_TOL[dtype], (b, l, "KV"[i], int(e.argmax()), float(e.max()))
    print("worst row", worst, flush=True)
    assert all(s["device_error"] == 0 for s in rt.kv_stats())
