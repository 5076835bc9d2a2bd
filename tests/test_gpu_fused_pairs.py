"""The fused selection's row-pair kernel (fan-out 2, g*K <= 32, up to four
heads per KV head, more than 2048 rows): sizes where its halves, key passes
and blocks end, against the float64 oracle under the selection parity bar."""
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


@pytest.mark.parametrize("shape", [
    # (B, H, Hkv, Nq, N, d, C, K, causal, dtype, score)
    (1, 1, 1, 2049, 2049, 64, 32, 4, 1, "f32", 0),     # an odd row alone in its wavefront, 32-key blocks
    (1, 2, 2, 1025, 3333, 64, 96, 7, 0, "f32", 0),     # 96-key blocks; a ragged last block is scored
    (1, 1, 1, 2100, 8101, 128, 256, 16, 0, "f32", 0),  # the widest block, the widest list, a 165-key last block
    (1, 3, 1, 2050, 2050, 128, 64, 5, 1, "f32", 0),    # three heads per KV head
    (2, 4, 1, 1030, 1500, 64, 64, 3, 1, "bf16", 0),    # forced blocks only
    (1, 4, 1, 2055, 2055, 128, 160, 4, 1, "bf16", 1),  # the mean, 160 keys
    (1, 1, 1, 2051, 2051, 128, 32, 16, 1, "bf16", 2),  # the mean and the variance
    (1, 1, 1, 2060, 2060, 64, 256, 16, 1, "f32", 0),   # every row keeps all of its blocks
])
def test_fused_pair_sizes(shape):
    B, H, Hkv, Nq, N, d, C, K, causal, dtype, score = shape
    assert B * Hkv * Nq > 2048
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, dtype, seed=41)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, causal, dtype, schedule=pisa.PISA_SCHEDULE_FUSED, score=score)
    q, k = dev(x["q"], dtype), dev(x["k"], dtype)
    idx, sc = pisa.select(p, q, k, pisa.build_pyramid(p, k), with_score=True)
    torch.cuda.synchronize()
    idx, sc = idx.cpu().numpy(), sc.cpu().numpy()
    check_selection_valid(idx, N, Nq, C, K, bool(causal))
    rows = np.unique(np.concatenate([np.arange(6), np.linspace(0, Nq - 1, 20).astype(int), np.arange(Nq - 6, Nq)]))
    check_selection_rows(x["q"], x["k"], C, 2, K, bool(causal), idx[:, :, rows], rows, gpu_score=sc[:, :, rows],
                         score=("lse", "mean", "mean_var")[score])
