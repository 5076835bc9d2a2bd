"""Which schedule the automatic choice takes below 4096 rows, told by its
workspace (no GPU): rows are grouped by key block where rows of one (batch, KV
head) share its blocks, and decode batches never are."""
import pytest

from paper_2609_31093_amd import pisa

AUTO, TWO, FUSED, SPLIT = range(4)


def _ws(schedule, B, H, Hkv, Nq, N, d=128, C=64, g=2, K=16, dtype="bf16"):
    return pisa.pisa_select_workspace_bytes(pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, 1, dtype, schedule))


@pytest.mark.parametrize("shape", [
    # (B, H, Hkv, Nq, N): one token of each of many sequences
    (64, 32, 8, 1, 131072),
    (128, 32, 8, 1, 20011),
    (255, 32, 8, 1, 4096),
    (256, 8, 8, 1, 20011),
    (64, 8, 8, 4, 20011),   # a few drafted tokens each
    (16, 32, 8, 8, 131072),
    # few rows over their own keys, or little work
    (1, 1, 1, 2048, 2048),
    (1, 4, 1, 1024, 8192),
    (1, 8, 2, 256, 1000),   # no more blocks than are kept
    (1, 16, 1, 2048, 60000),  # more than four heads
    # pairs per key block, and work, just below the line
    (2, 1, 1, 1024, 128 * 8193, 64, 128, 2, 16),
    (2, 8, 2, 512, 64 * 2049, 64, 64, 2, 4),
    (1, 2, 1, 1025, 32768, 64, 64, 3, 13),
])
def test_split_below_2048_rows(shape):
    assert _ws(AUTO, *shape) == _ws(SPLIT, *shape) != _ws(TWO, *shape)


@pytest.mark.parametrize("shape", [
    (300, 8, 8, 1, 131072),
    (1, 4, 4, 1000, 4000, 64, 64, 2, 8),    # short lists
    (1, 4, 1, 3000, 8192, 128, 64, 2, 4),
    (1, 16, 1, 3000, 8192, 128, 64, 2, 4),
    (1, 1, 1, 4000, 16384, 64, 32, 2, 16),  # little work
    (300, 8, 2, 4, 64 * 129),               # half a pair per key block
    (2100, 16, 1, 1, 64 * 385, 64, 64, 2, 8),
])
def test_fused_above(shape):
    assert _ws(AUTO, *shape) == 0 < _ws(TWO, *shape)


@pytest.mark.parametrize("shape", [
    (1, 32, 8, 256, 8192),
    (1, 8, 8, 256, 32768),
    (8, 4, 1, 64, 30000),
    (64, 4, 1, 32, 8192),
    (1, 16, 4, 600, 30000),
    (1, 8, 2, 1500, 30000),
    (1, 16, 1, 2049, 6000, 64, 64, 2, 8),
    (1, 4, 2, 1100, 20000, 128, 128, 4, 32),
    # few KV heads, or few blocks, with long lists or wide blocks
    (1, 4, 1, 804, 452031, 128, 128, 4, 32),
    (1, 1, 1, 3000, 262144, 128, 256, 2, 16),
    (2, 4, 1, 1500, 8192, 128, 128, 4, 32),
    (64, 2, 1, 32, 2048, 128, 256, 8, 4),
    (1, 8, 8, 3000 // 8, 2300),
    # pairs per key block, and work, at the line
    (2, 1, 1, 1024, 128 * 8192, 64, 128, 2, 16),
    (1, 2, 1, 1025, 32768, 64, 64, 3, 14),
    (1, 4, 1, 1025, 8192),
    (600, 4, 1, 4, 64 * 128),
    (2100, 16, 1, 1, 64 * 384, 64, 64, 2, 8),
])
def test_grouped(shape):
    assert _ws(AUTO, *shape) == _ws(TWO, *shape)
