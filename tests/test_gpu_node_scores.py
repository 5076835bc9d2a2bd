"""Split selection from node scores computed up front (few rows): the walks of
one and of two candidates per lane, at the sizes where a level is just ranked
or just not, against the float64 oracle and against the level-by-level walk
that a caller with the smaller workspace gets."""
import numpy as np
import pytest
import torch

from paper_2609_31093_amd import inputs
from tests.helpers import check_selection_rows, check_selection_valid, dev

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2609_31093_amd import pisa
else:
    pisa = None


def _small_ws(p):
    """a1, counts and scores of the split schedule, 256-byte aligned each: the workspace without node scores."""
    rows, gK = p.B * p.Hkv * p.Nq, p.fanout * p.K
    up = lambda n: (n + 255) // 256 * 256
    return 2 * up(rows * gK * 4) + up(rows * 4)


@pytest.mark.parametrize("shape", [
    # (B, H, Hkv, Nq, N, d, C, g, K, causal, dtype, score)
    (1, 2, 2, 1, 40000, 128, 64, 2, 16, 1, "bf16", 0),
    (1, 1, 1, 3, 32 * 65, 64, 32, 2, 16, 1, "bf16", 0),    # 65 leaves: level 3 holds 17, one over the budget
    (1, 1, 1, 3, 32 * 64, 64, 32, 2, 16, 1, "bf16", 0),    # 64 leaves: level 3 is not ranked
    (2, 6, 2, 2, 9000, 128, 32, 2, 13, 0, "bf16", 0),      # three heads, no forced blocks, a ragged last node
    (1, 4, 1, 2, 20000, 64, 32, 2, 32, 1, "f32", 0),       # 64 candidates
    (1, 8, 2, 1, 100000, 128, 128, 4, 32, 1, "bf16", 0),   # 128 candidates: two per lane
    (1, 2, 1, 5, 60000, 64, 32, 4, 30, 0, "bf16", 0),      # 120 of them, no forced blocks
    (1, 2, 1, 2, 30000, 64, 32, 3, 25, 1, "f32", 0),       # fan-out 3, 75 candidates
    (1, 16, 1, 1, 20000, 64, 64, 2, 8, 1, "bf16", 1),      # sixteen heads, the mean
    (1, 1, 1, 4, 30000, 128, 32, 4, 12, 1, "bf16", 2),     # the mean and the variance
])
def test_split_from_node_scores(shape):
    B, H, Hkv, Nq, N, d, C, g, K, causal, dtype, score = shape
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, dtype, seed=51)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, causal, dtype, schedule=pisa.PISA_SCHEDULE_SPLIT, score=score)
    q, k = dev(x["q"], dtype), dev(x["k"], dtype)
    pyr = pisa.build_pyramid(p, k)
    idx, sc = pisa.select(p, q, k, pyr, with_score=True)
    small = torch.empty(_small_ws(p), dtype=torch.uint8, device="cuda")
    idx2 = torch.empty_like(idx)
    pisa.pisa_select(p, q, k, pyr, idx2, None, small, small.numel())
    with pytest.raises(pisa.PisaError):
        pisa.pisa_select(p, q, k, pyr, idx2, None, small, small.numel() - 1)
    torch.cuda.synchronize()
    idx, idx2, sc = idx.cpu().numpy(), idx2.cpu().numpy(), sc.cpu().numpy()
    rows = np.arange(Nq)
    kind = ("lse", "mean", "mean_var")[score]
    check_selection_valid(idx, N, Nq, C, K, bool(causal))
    check_selection_rows(x["q"], x["k"], C, g, K, bool(causal), idx, rows, gpu_score=sc, score=kind)
    check_selection_rows(x["q"], x["k"], C, g, K, bool(causal), idx2, rows, score=kind)


def test_small_workspace_is_smaller():
    p = pisa.make_problem(1, 2, 2, 1, 40000, 128, 64, 2, 16, 1, "bf16")
    assert pisa.pisa_select_workspace_bytes(p) > _small_ws(p)


@pytest.mark.parametrize("shape", [
    # (B, H, Hkv, Nq, N, d, C, g, K, causal): rows where the automatic schedule may group
    (1, 4, 1, 512, 9001, 128, 64, 2, 16, 1),     # split: few rows of one KV head
    (1, 1, 1, 2047, 6000, 64, 64, 2, 8, 1),      # split, one below and at the line of single heads: little work
    (1, 1, 1, 2048, 6000, 64, 64, 2, 8, 1),
    (1, 16, 1, 2049, 6000, 64, 64, 2, 8, 1),     # grouped: sixteen heads, above the split range
    (1, 4, 2, 1100, 20000, 128, 128, 4, 32, 0),  # grouped, 128 candidates
    (3, 3, 1, 800, 3000, 64, 32, 3, 7, 1),       # grouped, three heads
])
def test_middle_rows(shape):
    """The schedule that the full workspace gets, grouped by key block where that
    pays, and the one of callers with the least workspace (none, or the split
    schedule's smallest)."""
    B, H, Hkv, Nq, N, d, C, g, K, causal = shape
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=52)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, causal, "bf16")
    q, k = dev(x["q"], "bf16"), dev(x["k"], "bf16")
    pyr = pisa.build_pyramid(p, k)
    idx, sc = pisa.select(p, q, k, pyr, with_score=True)
    idx2 = torch.empty_like(idx)
    small = torch.empty(_small_ws(p), dtype=torch.uint8, device="cuda")
    if B * Hkv * Nq > 2048:
        pisa.pisa_select(p, q, k, pyr, idx2)
    else:
        pisa.pisa_select(p, q, k, pyr, idx2, None, small, small.numel())
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(4), np.linspace(0, Nq - 1, 12).astype(int), np.arange(Nq - 4, Nq)]))
    for got, score in ((idx, sc), (idx2, None)):
        got = got.cpu().numpy()
        check_selection_valid(got, N, Nq, C, K, bool(causal))
        check_selection_rows(x["q"], x["k"], C, g, K, bool(causal), got[:, :, rows], rows,
                             gpu_score=None if score is None else score.cpu().numpy()[:, :, rows])
