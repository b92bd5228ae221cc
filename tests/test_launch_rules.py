"""The launch rules that pick a kernel's split or form from sizes alone (``csrc/launch_rules.h``), on the CPU."""
import pytest

from synth.configs import BF16, F32
from tests.rules_util import rules

CUS = 256


@pytest.mark.parametrize("dtype,hd,kv", [(BF16, 128, 4096), (BF16, 128, 8192), (BF16, 128, 32768), (BF16, 64, 16384), (F32, 128, 4096)])
def test_filled_attention_keeps_the_gpu_busy(dtype, hd, kv):
    # one workgroup runs per CU: their number fills at least 7/10 of the rounds that it takes, at every row count
    for hk in (2, 8):
        for rows in range(1, 65):
            wgs = rows * hk * rules().splits(dtype, rows, hk, hd, kv)
            assert wgs >= 0.7 * CUS * -(-wgs // CUS) or wgs == rows * hk * 64, (hk, rows, wgs)


@pytest.mark.parametrize("dtype,hd,kv", [(BF16, 128, 8192), (BF16, 128, 32768), (BF16, 64, 16384), (F32, 128, 4096), (F32, 64, 9000)])
def test_long_rows_are_shared(dtype, hd, kv):
    # a row's slots are shared by its own splits alone, and the batch may be ragged: from 2 MB of keys a row has up to 8
    # splits while two rounds of workgroups hold them
    for hk in (1, 2, 3, 8, 32):
        for rows in range(1, 65):
            assert rules().splits(dtype, rows, hk, hd, kv) >= min(8, -(-2 * CUS // (rows * hk))), (hk, rows)


def test_filled_attention_split_limits():
    for dtype, hd, kb, es in ((BF16, 64, 32, 2), (BF16, 128, 32, 2), (F32, 64, 16, 4), (F32, 128, 16, 4)):
        for rows in (1, 2, 7, 40, 64, 1000):
            for hk in (1, 8, 64):
                for kv in (1, 31, 128 * 1024 // (hd * es) - 1, 128 * 1024 // (hd * es), 1000, 5000, 1 << 24):
                    s = rules().splits(dtype, rows, hk, hd, kv)
                    assert 1 <= s <= max(1, min(64, (-(-kv // kb) + 1) // 2))   # two key blocks or more each
                    assert s == 1 or kv * hd * es >= 128 * 1024


@pytest.mark.parametrize("rows,kv,splits", [(1, 512, 8), (2, 1999, 16), (1, 2048, 32), (8, 2048, 4), (8, 4096, 4), (32, 4096, 1),
                                            (64, 4096, 1), (1, 32768, 32), (4, 32768, 8)])
def test_filled_attention_splits_where_one_round_is_full(rows, kv, splits):
    assert rules().splits(BF16, rows, 8, 128, kv) == splits


# q/k/v 6,144 columns, the embedder 12,288, gate/up 28,672 and (wider models) beyond one round of 256 x 128 columns
@pytest.mark.parametrize("rows,cols,takes", [(9, 6144, 1), (32, 12288, 1), (32, 28672, 1), (32, 32768, 1), (8, 28672, 0), (33, 28672, 0),
                                             (32, 32800, 0), (32, 33280, 0), (16, 33280, 0), (16, 36864, 1), (17, 36864, 0), (32, 40960, 1),
                                             (32, 57344, 1), (32, 65536, 1), (32, 99840, 0), (16, 99840, 1)])
def test_row_kernel_takes_well_filled_rounds(rows, cols, takes):
    assert rules().rows_takes(rows, cols) == takes


@pytest.mark.parametrize("grp", [1, 2, 3, 4])
def test_prompt_attention_blocks_cover_every_tile(grp):
    # the tiles of 32 rows that the workgroups of a sequence take, by the kernel's own mapping, are each taken once
    for rows, s0, T in ((1, 0, 1), (31, 0, 31), (33, 0, 33), (77, 0, 77), (300, 0, 300), (1232, 0, 77), (1664, 500, 1100), (2048, 0, 4096)):
        for hk in (1, 2, 8, 32):
            keys, blocks = rules().prompt_keys(rows, s0, T, grp * hk, hk), rules().prompt_blocks(rows, s0, T, grp * hk, hk)
            for z in range((s0 + rows - 1) // T + 1):
                lo, hi = max(z * T - s0, 0), min(z * T - s0 + T, rows)
                nt, groups = -(-(hi - lo) // 32), 8 // grp
                taken = []
                for x in range(blocks):
                    if keys:
                        n = groups // 2
                        taken += [t for t in range(x * n, x * n + n) if t < nt]
                    else:
                        half = groups // 2
                        for t in range(x * half, x * half + half):
                            taken += ([t] if 2 * t < nt else []) + ([nt - 1 - t] if 2 * t < nt - 1 else [])
                assert sorted(taken) == list(range(nt)), (rows, s0, T, hk, keys, z)
