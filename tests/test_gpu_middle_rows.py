"""The automatic schedule below 4096 bf16 rows where it groups the leaf pairs by
key block: each stage 1 that serves these rows, against the float64 oracle, and
what callers get who bring another workspace."""
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
    # (B, H, Hkv, Nq, N, d, C, g, K, causal)
    (1, 16, 4, 131, 5000, 128, 64, 2, 16, 1),    # up to 64 candidates, at most 2048 rows
    (2, 8, 2, 160, 9001, 64, 64, 2, 32, 0),      # 64 of them, no forced blocks
    (1, 8, 2, 300, 20001, 128, 64, 4, 32, 1),    # 128
    (4, 8, 2, 300, 3001, 128, 64, 2, 16, 1),     # more rows: row pairs, fan-out 2
    (8, 4, 1, 300, 3001, 128, 64, 3, 10, 1),     # fan-out 3
    (2, 8, 2, 600, 9001, 128, 32, 2, 40, 1),     # 80 candidates
    (1, 16, 1, 2051, 2051, 64, 64, 2, 8, 1),     # sixteen heads
])
def test_grouped_rows(shape):
    B, H, Hkv, Nq, N, d, C, g, K, causal = shape
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=71)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, causal, "bf16")
    two = pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, causal, "bf16", schedule=pisa.PISA_SCHEDULE_TWO_STAGE)
    assert B * Hkv * Nq < 4096 and pisa.pisa_select_workspace_bytes(p) == pisa.pisa_select_workspace_bytes(two)
    q, k = dev(x["q"], "bf16"), dev(x["k"], "bf16")
    idx, sc = pisa.select(p, q, k, pisa.build_pyramid(p, k), with_score=True)
    torch.cuda.synchronize()
    idx, sc = idx.cpu().numpy(), sc.cpu().numpy()
    check_selection_valid(idx, N, Nq, C, K, bool(causal))
    rows = np.unique(np.concatenate([np.arange(2), np.linspace(0, Nq - 1, 6).astype(int), np.arange(Nq - 2, Nq)]))
    check_selection_rows(x["q"], x["k"], C, g, K, bool(causal), idx[:, :, rows], rows, gpu_score=sc[:, :, rows])


def test_workspaces_of_no_use():
    """Rows that the fused schedule serves without a workspace take any: none,
    a small one, or one that is not aligned, whose bytes stay as they are.  The
    split schedule, which needs one, refuses it."""
    B, H, Hkv, Nq, N, d, C, g, K = 1, 16, 4, 600, 9001, 64, 64, 2, 16
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=72)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, 1, "bf16")
    q, k = dev(x["q"], "bf16"), dev(x["k"], "bf16")
    pyr = pisa.build_pyramid(p, k)
    need = pisa.pisa_select_workspace_bytes(p)
    assert need > 0
    want = torch.empty((B, Hkv, Nq, K), dtype=torch.int32, device="cuda")
    pisa.pisa_select(p, q, k, pyr, want)
    ws = torch.full((need + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    idx = torch.empty_like(want)
    pisa.pisa_select(p, q, k, pyr, idx, None, ws[16:], need)
    torch.cuda.synchronize()
    assert torch.equal(idx, want) and bool((ws == 0x5A).all())
    few = pisa.make_problem(B, H, Hkv, 300, N, d, C, g, K, 1, "bf16")
    with pytest.raises(pisa.PisaError) as e:
        pisa.pisa_select(few, q[:, :, :300].contiguous(), k, pyr, idx, None, ws[16:], need)
    assert e.value.status == pisa.PISA_ERR_INVALID_ARG
