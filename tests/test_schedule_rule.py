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
    # few rows over their own keys, or on one KV head
    (1, 4, 1, 512, 2048),
    (1, 1, 1, 2048, 2048),
    (1, 8, 2, 256, 1000),   # no more blocks than are kept
])
def test_split_below_2048_rows(shape):
    assert _ws(AUTO, *shape) == _ws(SPLIT, *shape) != _ws(TWO, *shape)


@pytest.mark.parametrize("shape", [
    (300, 8, 8, 1, 131072),
    (1, 1, 1, 3000, 3000),
    (1, 4, 4, 1000, 4000, 64, 64, 2, 8),
    (1, 4, 1, 3000, 8192, 128, 64, 2, 4),
    (1, 16, 1, 3000, 8192, 128, 64, 2, 4),
    (2, 4, 1, 1500, 4096, 128, 128, 4, 32),
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
])
def test_grouped(shape):
    assert _ws(AUTO, *shape) == _ws(TWO, *shape)
