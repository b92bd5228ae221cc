"""Cases of the attention tests and the bounds that their results are held to (test_attention_bounds.py: a lost key exceeds
them).

Prompt attention: the input rows are small (0.004) against the attention's output (about 0.4 / sqrt(slots) of 8 heads of 64, more of more
heads), so the next layer's K and V depend on the attention in full.

Bound, per row over all kv heads of a layer, 2-norm of the difference over 2-norm of the row.  bf16: K and V are rounded
to 8 significant bits on both sides, so a value near a rounding boundary differs by one unit, at most 2^-8 of itself:
3.9e-3 if every value did, and the error before rounding (about 1e-3: hi/lo operands, and the rounding of the layer
before) comes on top.  fp32: sums of up to 2,000 products, twice per layer, at 2^-24 each.

Attention over a filled cache: largest difference of a (row, q-head) over the root mean square of its output.  bf16:
probabilities and outputs are hi/lo pairs (2^-17 of the value), scores fp32 sums over the head dim (about 1e-5 absolute),
together below 1e-4; fp32: scores and sums at 2^-24, below 1e-5.  A lost slot of n changes the output by about 1 / sqrt(n) of it.
"""
import dataclasses

import numpy as np

from synth.configs import BF16, F32
from tests.gpu_util import SMALL16

ATTN_TOL = {BF16: 5e-3, F32: 2e-5}
FILLED_TOL = {BF16: 3e-4, F32: 3e-5}

# dtype, q-heads, kv heads, head dim, slots of each row: rows and lengths where the op splits, does not, and leaves splits
# without slots; other group sizes and kv-head counts; one long row among short ones
FILLED = [
    (BF16, 32, 8, 128, [511]), (BF16, 32, 8, 128, [512]), (BF16, 32, 8, 128, [4097, 1]),
    (BF16, 32, 8, 64, [1023] * 2), (BF16, 32, 8, 64, [1024, 0, 33]), (BF16, 9, 3, 64, [2000, 40, 1999, 65]),
    (BF16, 8, 8, 128, [700] * 40), (BF16, 4, 2, 128, [9000]), (F32, 32, 8, 64, [511, 513, 700]), (F32, 6, 2, 128, [3001]),
    (BF16, 32, 8, 128, [4096] + [700] * 16), (BF16, 8, 2, 128, [500, 33, 0] * 5 + [8192]), (F32, 4, 2, 128, [4100, 16, 15])]

# q-heads per kv head, kv heads, head dim, batch, prompt, whether the keys form takes the first chunk
FORMS = [
    (1, 8, 64, 17, 77, 0), (1, 8, 64, 3, 1100, 1), (1, 8, 128, 1, 65, 1), (2, 8, 64, 17, 77, 0), (2, 8, 128, 3, 300, 1),
    (3, 8, 64, 16, 77, 0), (3, 8, 64, 1, 300, 1), (3, 8, 128, 2, 129, 1), (4, 8, 64, 16, 77, 0), (4, 8, 64, 3, 1100, 0),
    (4, 2, 64, 2, 161, 1), (4, 8, 128, 9, 130, 0)]


def attention_shape(grp, hk, hd, dtype):
    return dataclasses.replace(SMALL16, n_layers=2, d_model=256, n_heads=grp * hk, n_kv_heads=hk, head_dim=hd, ffn_dim=256,
                               vocab=256, micro_layers=1, dtype=dtype)


def attention_inputs(batch, prompt, shp):
    rng = np.random.default_rng(7)
    X = (0.004 * rng.standard_normal((batch, prompt, shp.d_model))).astype(np.float32)
    pos = (np.cumsum(rng.integers(1, 5, (batch, prompt)), axis=1) - 1).astype(np.int32)
    return X, pos


def row_error(a, b):
    """a, b [slots][kv heads][head dim] -> relative 2-norm error of each slot."""
    n = a.shape[0]
    d = np.linalg.norm((np.asarray(a, np.float64) - b).reshape(n, -1), axis=1)
    return d / np.linalg.norm(np.asarray(b, np.float64).reshape(n, -1), axis=1)
