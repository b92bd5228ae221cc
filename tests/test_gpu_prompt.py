"""The prompt kernels at the edges of their tiles: every layer's K and V of every row of a prefill, and its
decision, against the float64 oracle.

The model's widths end inside the GEMM tiles of 128 and 256 columns (q/k/v 768, d 544, gate/up 2112 columns, k-ranges
of 17, 16 and 33 fragments); the prompt lengths end inside its tiles of 128 rows and the attention's tiles of 16.
Tolerance: the largest difference over the largest value, at most 2e-2 in bf16 (the decisions' tolerance) and 1e-4 in
fp32; a wrong row or column is off by the order of the value itself.

Marked ``gpu``: needs an MI355X and ``libham.so`` built in-tree.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import OracleHam
from synth.configs import BF16, F32
from tests.gpu_util import SMALL16, TOL, config_for, run_gpu

pytestmark = pytest.mark.gpu

EDGES = dataclasses.replace(SMALL16, n_layers=3, d_model=544, ffn_dim=1056, vocab=1024, micro_layers=1)


def _check(shp, B, P, rows, seed=301):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_20438_amd import ham
    prompts = synth.prompt_ids(seed + 1, B, P, shp.vocab)
    sched = synth.group_schedule(seed + 2, B, 2, 4)
    om = OracleHam(shp, seed)
    rt = ham.HamRuntime(config_for(shp, B, P, 1), seed)
    teacher = [[[(7 * b + j) % shp.vocab for j in range(sched[b, s])] for s in range(2)] for b in range(B)]
    res = run_gpu(rt, prompts, [0] * B, 0, sched, teacher=teacher, debug_steps=1)
    tol = TOL[shp.dtype]
    kv = [[t.cpu().numpy().astype(np.float64) for t in rt.kv_cache(l, P)] for l in range(shp.n_layers)]
    for b in rows:
        o = om.generate(prompts[b], 0, 0, forced=lambda st: 1, record=True)
        dec = o.decisions[0]
        assert np.max(np.abs(res.logits[(b, 0, 0)] - dec.logits)) <= tol, b
        assert np.max(np.abs(res.hidden[(b, 0, 0)] - dec.h)) <= tol, b
        for l in range(shp.n_layers):
            for i, name in enumerate("KV"):
                ref = np.transpose(om.last_caches[l][i], (1, 0, 2))
                err = np.max(np.abs(kv[l][i][b] - ref), axis=(0, 2)) / np.max(np.abs(ref))
                assert err.max() <= tol, (b, l, name, int(err.argmax()), float(err.max()))
    assert all(s["kv_len"] == P and s["device_error"] == 0 for s in rt.kv_stats())


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("prompt", [65, 130, 257, 300, 513])   # the batched GEMM's last row count, whole and cut tiles
def test_prompt_rows_past_a_tile(dtype, prompt):
    _check(dataclasses.replace(EDGES, dtype=dtype), 1, prompt, [0])
