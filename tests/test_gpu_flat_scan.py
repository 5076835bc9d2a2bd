"""Flat block selection on the scan kernels (bf16): the sizes where their tiles
end, budgets at the edges of what a lane or a list holds, ties that fill a
list, and scores that send a tile to the exact list kernel.

Rows are held to the parity bar of the other selection tests: identical to the
float64 oracle where its margin exceeds 1e-3, admissible elsewhere (scores are
fp32 sums over bf16 hi and lo means, off by at most 2^-17 of sum |q_i m_i|)."""
import numpy as np
import pytest
import torch

from paper_2609_31093_amd import inputs
from tests.helpers import check_flat_bsa_rows, check_selection_valid, dev

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2609_31093_amd import pisa
else:
    pisa = None


def _run(x, B, H, Hkv, Nq, N, d, C, K, causal):
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, causal, "bf16")
    q, k = dev(x["q"], "bf16"), dev(x["k"], "bf16")
    idx = pisa.select_flat_bsa(p, q, pisa.build_pyramid(p, k))
    torch.cuda.synchronize()
    return idx.cpu().numpy()


def _check(x, idx, N, Nq, C, K, causal, rows):
    check_selection_valid(idx, N, Nq, C, K, bool(causal))
    st = check_flat_bsa_rows(x["q"], x["k"], C, K, bool(causal), idx[:, :, rows], rows)
    assert st["rows"] > 0
    return st


@pytest.mark.parametrize("shape", [
    # (B, H, Hkv, Nq, N, d, C, K, causal); C = 32 makes many blocks
    (1, 1, 1, 128, 1024, 128, 32, 16, 1),      # one workgroup of 128 rows, 32 blocks: one tile
    (1, 2, 2, 129, 1056, 64, 32, 13, 1),       # a row past a workgroup, a block past a tile
    (1, 1, 1, 63, 2048, 128, 32, 16, 0),       # rows end inside a wavefront's half, no forced blocks
    (1, 1, 1, 33, 640, 64, 32, 3, 1),          # causal budget of the forced blocks alone
    (1, 1, 1, 40, 640, 128, 32, 1, 0),         # one block kept
    (64, 1, 1, 2049, 2049, 64, 64, 8, 1),      # 512 or more workgroups: 256 rows each
    (1, 2, 1, 31, 1024, 128, 32, 16, 1),       # several heads: less than a 32-row tile
    (1, 4, 1, 65, 4128, 128, 32, 32, 1),       # several heads, budget 32: lists of up to 64
    (1, 3, 1, 32, 4096, 64, 32, 17, 0),
    (1, 16, 1, 33, 2080, 64, 32, 16, 0),       # sixteen heads
    (1, 5, 1, 34, 2080, 128, 32, 32, 1),       # more than four heads, d = 128: the largest LDS
    (1, 2, 1, 40, 640, 64, 32, 3, 1),
])
def test_tile_edges(shape):
    B, H, Hkv, Nq, N, d, C, K, causal = shape
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=31)
    idx = _run(x, B, H, Hkv, Nq, N, d, C, K, causal)
    rows = np.arange(Nq) if B * Nq <= 200 else np.array([0, 5, 511, 512, 1279, Nq - 2, Nq - 1])
    if B > 1:  # the oracle walks every batch entry: the first and the last
        check_selection_valid(idx, N, Nq, C, K, bool(causal))
        for b in (0, B - 1):
            one = {n: a[b:b + 1] for n, a in x.items()}
            check_flat_bsa_rows(one["q"], one["k"], C, K, bool(causal), idx[b:b + 1][:, :, rows], rows)
    else:
        _check(x, idx, N, Nq, C, K, causal, rows)


@pytest.mark.parametrize("H,every,d", [(1, 3, 128), (1, 40, 64), (4, 3, 64), (4, 40, 128)])
def test_equal_blocks_at_the_cut(H, every, d):
    """Many blocks with exactly equal scores beside others above and below
    them: the smaller ones are kept, also when more are equal than a query's
    list holds."""
    B, Hkv, Nq, N, C, K = 1, 1, 96, 16384, 32, 16
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=32)
    for j in range(1, N // C, every):
        x["k"][:, :, j * C:(j + 1) * C] = x["k"][:, :, :1]
    idx = _run(x, B, H, Hkv, Nq, N, d, C, K, 1)
    _check(x, idx, N, Nq, C, K, 1, np.arange(Nq))


@pytest.mark.parametrize("H", [1, 4])
def test_one_class_holds_the_best(H):
    """The best blocks 128 apart, which the scans count as one class each: more
    of them reach the cut than a class keeps."""
    B, Hkv, Nq, N, d, C, K = 1, 1, 64, 65536, 64, 32, 16
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=33)
    u = x["q"][0, 0, 0] / np.linalg.norm(x["q"][0, 0, 0])
    x["q"] = inputs.round_to_bf16(x["q"] * 0.25 + 4 * u.astype(np.float32))
    for n, j in enumerate(range(5, N // C, 128)):
        x["k"][:, :, j * C:(j + 1) * C] = inputs.round_to_bf16((3 + 0.25 * n) * u.astype(np.float32))
    idx = _run(x, B, H, Hkv, Nq, N, d, C, K, 1)
    _check(x, idx, N, Nq, C, K, 1, np.arange(Nq))


@pytest.mark.parametrize("B,H,Hkv,Nq,K,equal", [
    (8, 4, 1, 4100, 8, "all"),     # 520 tiles of 64 rows, each marked: two to some workgroups of the exact kernel
    (8, 2, 1, 8300, 16, "all"),    # 1040 of them
    (8, 4, 1, 4100, 8, "some"),    # the tiles of every other batch entry
    (8, 1, 1, 4100, 8, "all"),     # one head: the scans decide ties
])
def test_marked_tiles(B, H, Hkv, Nq, K, equal):
    """Keys that are all equal: every block scores the same and the smaller
    ones are kept, beside the forced ones."""
    N, d, C = Nq, 64, 64
    gen = torch.Generator(device="cuda").manual_seed(34)
    q, k = (torch.randn((B, h, N, d), generator=gen, device="cuda").bfloat16() for h in (H, Hkv))
    marked = slice(None) if equal == "all" else slice(1, None, 2)
    k[marked] = 0.5
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, 1, "bf16")
    idx = pisa.select_flat_bsa(p, q, pisa.build_pyramid(p, k))
    c = (torch.arange(Nq, device="cuda") // C)[:, None]
    j = torch.arange(K, device="cuda")[None]
    want = torch.where(c < K, torch.where(j <= c, j, -1), torch.where(j < K - 2, j, c - (K - 1) + j))
    assert torch.equal(idx[marked], want.int().expand_as(idx[marked]))
    if equal == "some":
        rows = np.array([0, 63, 64, 2000, Nq - 1])
        x = {"q": q[:1].float().cpu().numpy(), "k": k[:1].float().cpu().numpy()}
        check_flat_bsa_rows(x["q"], x["k"], C, K, True, idx[:1, :, rows].cpu().numpy(), rows)


@pytest.mark.parametrize("H", [1, 4])
@pytest.mark.parametrize("K", [16, 24])
def test_nan(H, K):
    """A block of NaN keys and a few NaN queries: rows that see neither select
    what they would without them, the other rows what can be ranked (with one
    head: every other block) and their forced blocks, padded with -1."""
    B, Hkv, Nq, N, d, C = 1, 1, 200, 8192, 64, 32
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, "bf16", seed=35)
    j = 253  # of 256; rows 0-103 end before it, and it is no row's forced block from row 168 on
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, 1, "bf16")
    q, k = dev(x["q"], "bf16"), dev(x["k"], "bf16")
    clean = pisa.select_flat_bsa(p, q, pisa.build_pyramid(p, k)).cpu().numpy()[0, 0]
    k[:, :, j * C:(j + 1) * C] = float("nan")
    q[:, :, 40:200:50] = float("nan")
    idx = pisa.select_flat_bsa(p, q, pisa.build_pyramid(p, k)).cpu().numpy()[0, 0]
    nan_q = np.isin(np.arange(Nq), np.arange(40, 200, 50))
    for r in range(Nq):
        c = (N - Nq + r) // C
        row = idx[r]
        got = row[row >= 0]
        assert np.all(np.diff(got) > 0) and {0, c - 1, c} <= set(got) and np.all(row[len(got):] == -1)
        if nan_q[r]:
            assert list(got) == [0, c - 1, c]
        elif c < j:
            assert np.array_equal(row, clean[r])
        elif c > j + 1 and H == 1:
            assert len(got) == K and j not in got and set(clean[r]) - {j} <= set(got)
    rows = np.array([0, 1, 39, 41, 88, 91, 103])
    check_flat_bsa_rows(x["q"], x["k"], C, K, True, idx[None, None, rows], rows)
