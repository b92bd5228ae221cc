"""A lost key exceeds the bounds of the attention tests: planted in the float64 reference, on the CPU."""
import numpy as np
import pytest

from oracle import OracleHam
from oracle.ham import attend
from synth.configs import BF16, F32
from tests.attention_bounds import ATTN_TOL, FILLED, FILLED_TOL, FORMS, attention_inputs, attention_shape, row_error


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("grp,hk,hd,prompt", sorted({(g, hk, hd, p) for g, hk, hd, _, p, _ in FORMS}))
def test_lost_key_of_a_prompt(dtype, grp, hk, hd, prompt):
    # the rows of the last tile of 32 miss one slot of their attention in the first layer, in every head
    shp = attention_shape(grp, hk, hd, dtype)
    X, pos = attention_inputs(1, prompt, shp)
    om = OracleHam(shp, 5)
    good, bad = om.new_caches(2), om.new_caches(2)
    om.forward_rows(om.layers[:2], X[0], pos[0], good)
    first = (prompt - 1) // 32 * 32

    def lossy(q, K, V, n_valid):
        out = attend(q, K, V, n_valid, hk)
        keep = np.delete(np.arange(K.shape[0]), first // 2)   # a slot that these rows all see
        out[first:] = attend(q[first:], K[keep], V[keep], np.asarray(n_valid)[first:] - 1, hk)
        return out
    om.attend = lossy
    om.forward_rows(om.layers[:2], X[0], pos[0], bad)
    for i in range(2):
        assert np.all(row_error(bad[1][i], good[1][i])[:first] == 0)
        e = row_error(bad[1][i], good[1][i])[first:]
        assert e.min() > 2 * ATTN_TOL[dtype]


@pytest.mark.parametrize("dtype,n,hd", sorted({(t, n, hd) for t, _, _, hd, lens in FILLED for n in lens if n > 1}))
def test_lost_slot_of_a_filled_cache(dtype, n, hd):
    rng = np.random.default_rng(n)
    q, K, V = rng.standard_normal((1, 4, hd)), rng.standard_normal((n, 1, hd)), rng.standard_normal((n, 1, hd))
    ref = attend(q, K, V, [n], 1)[0]
    for j in (0, n // 2, n - 1):
        keep = np.delete(np.arange(n), j)
        d = np.abs(attend(q, K[keep], V[keep], [n - 1], 1)[0] - ref).max(axis=1) / np.sqrt((ref ** 2).mean(axis=1))
        assert d.max() > 2 * FILLED_TOL[dtype], (j, d)   # some head of the row shows it
