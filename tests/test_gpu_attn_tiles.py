"""Causal attention of several heads per KV head on the row-tile kernel: every
block size and group against the oracle, at budgets on both sides of the slots
that a column's lanes read ahead (8 or 16) and of a multiple of four."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_31093_amd import inputs
from tests.helpers import dev

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2609_31093_amd import pisa
else:
    pisa = None


def _lists(BH, Nq, N, C, K, seed):
    """[BH, Nq, K]: the first, previous and own block and random earlier ones, ascending, -1 padded."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    M1 = -(-N // C)
    c = (N - Nq + torch.arange(Nq, device="cuda")) // C
    s = torch.rand((BH, Nq, M1), generator=gen, device="cuda")
    blocks = torch.arange(M1, device="cuda")
    s = s.masked_fill(blocks > c[:, None], -1.0)
    for f in (torch.zeros_like(c), (c - 1).clamp(min=0), c):
        s[:, torch.arange(Nq, device="cuda"), f] = 2.0
    w, i = s.topk(min(K, M1), dim=-1)
    i = torch.where(w < 0, M1, i).sort(-1).values
    out = torch.full((BH, Nq, K), -1, dtype=torch.int32, device="cuda")
    out[..., :i.shape[-1]] = torch.where(i == M1, -1, i).int()
    return out


@pytest.mark.parametrize("d,C", [(64, 32), (64, 96), (64, 128), (128, 32), (128, 64), (128, 96), (128, 128)])
@pytest.mark.parametrize("G,K", [(2, 16), (4, 5), (4, 13), (4, 16), (4, 17), (8, 9), (8, 20), (16, 8), (16, 16), (4, 33)])
def test_tiles_match_oracle(d, C, G, K):
    B, Hkv, Nq = 1, 2, 2060
    N = max(Nq, (K + 6) * C)
    H = Hkv * G
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=81)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, 1, "bf16")
    q, k, v = (dev(x[n], "bf16") for n in "qkv")
    idx = _lists(Hkv, Nq, N, C, K, 82).view(B, Hkv, Nq, K)
    o, lse = pisa.sparse_attn_fwd(p, q, k, v, idx)
    torch.cuda.synchronize()
    T = 128 // G
    rows = np.unique(np.concatenate([np.arange(0, Nq, 97), [T - 1, T, Nq - Nq % T, Nq - 1]]))
    want_o, want_lse = O.sparse_attention(x["q"], x["k"], x["v"], idx.cpu().numpy()[:, :, rows], C, True, rows=rows)
    assert np.abs(o.float().cpu().numpy()[:, :, rows] - want_o).max() <= 2e-2
    assert np.abs(lse.cpu().numpy()[:, :, rows] - want_lse).max() <= 1e-3
