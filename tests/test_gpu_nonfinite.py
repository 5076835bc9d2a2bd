"""Selection over keys that hold NaN or infinities: every row still selects
min(K, eligible) distinct blocks, the forced ones among them, and rows that see
none of those keys select what they would without them (float64 oracle)."""
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

SPLIT, FUSED, TWO = 3, 2, 1


def poison(k, C, first, what):
    """Every other block from block `first` on: NaN of either sign in every
    value ("nan", "-nan"), or an infinity in one dimension ("inf": scores of
    +inf or -inf by the query's sign, NaN where they meet)."""
    k = k.clone()
    blocks = torch.arange(first, -(-k.shape[2] // C), 2)
    rows = (blocks[:, None] * C + torch.arange(C)).flatten().cuda()
    rows = rows[rows < k.shape[2]]
    if what == "inf":
        k[:, :, rows, 3] = float("inf")
    else:
        k[:, :, rows] = float("nan")
        if what == "-nan":
            bits = k.view(torch.int16 if k.dtype == torch.bfloat16 else torch.int32)
            bits[:, :, rows] |= torch.iinfo(bits.dtype).min
    return k


def check(B, H, Hkv, Nq, N, d, C, g, K, causal, dtype, schedule, score, what, workspace=None):
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, dtype, seed=61)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, g, K, causal, dtype, schedule=schedule, score=score)
    q, clean = dev(x["q"], dtype), dev(x["k"], dtype)
    M1 = -(-N // C)
    first = M1 // 3
    k = poison(clean, C, first, what)
    nb = pisa.pisa_select_workspace_bytes(p) if workspace is None else workspace(p)
    ws = torch.empty(max(nb, 1), dtype=torch.uint8, device="cuda")
    idx = torch.empty((B, Hkv, Nq, K), dtype=torch.int32, device="cuda")
    pisa.pisa_select(p, q, k, pisa.build_pyramid(p, k), idx, None, ws if nb else None, nb)
    torch.cuda.synchronize()
    idx = idx.cpu().numpy()
    check_selection_valid(idx, N, Nq, C, K, bool(causal))
    before = min(Nq, first * C - (N - Nq))  # rows that see none of the poisoned blocks
    if causal and before > 0:
        rows = np.unique(np.linspace(0, before - 1, 12).astype(int))
        check_selection_rows(x["q"], x["k"], C, g, K, True, idx[:, :, rows], rows,
                             score=("lse", "mean", "mean_var")[score])


def split_floor(p):
    """The split schedule's workspace without node scores: its candidates, counts and scores."""
    rows, gK = p.B * p.Hkv * p.Nq, p.fanout * p.K
    up = lambda n: (n + 255) // 256 * 256
    return 2 * up(rows * gK * 4) + up(rows * 4)


@pytest.mark.parametrize("what", ["nan", "-nan", "inf"])
@pytest.mark.parametrize("shape", [
    # ranked by counting the candidates that come before one
    (1, 2, 1, 40, 16000, 128, 64, 2, 48, 1, "bf16", SPLIT, 0, split_floor),  # 96 candidates, a workgroup per row
    (1, 2, 1, 40, 16000, 64, 32, 4, 32, 0, "f32", SPLIT, 1, split_floor),    # no forced blocks
    (1, 1, 1, 300, 9001, 64, 32, 2, 16, 1, "bf16", FUSED, 1, None),          # up to the raw keys
    (1, 1, 1, 2100, 21000, 64, 32, 4, 50, 1, "bf16", FUSED, 0, None),        # 200 candidates, a wavefront per row
    (1, 1, 1, 2100, 21000, 64, 32, 4, 50, 1, "bf16", TWO, 0, None),          # ... and in the final Top-K
    (1, 4, 1, 2100, 21000, 128, 64, 4, 32, 1, "bf16", 0, 0, None),           # the automatic schedule
])
def test_counting_rank(shape, what):
    *problem, workspace = shape
    check(*problem, what, workspace)


@pytest.mark.parametrize("what", ["nan", "-nan", "inf"])
@pytest.mark.parametrize("shape", [
    # ranked by sorts across 32 or 64 lanes
    (1, 1, 1, 2101, 9001, 64, 64, 2, 4, 1, "f32", FUSED, 0, None),          # row pairs up to the raw keys
    (1, 1, 1, 2101, 9001, 128, 32, 2, 16, 1, "f32", FUSED, 1, None),        # ... with the sort that stops early
    (1, 4, 1, 2060, 9001, 128, 64, 2, 7, 1, "bf16", FUSED, 0, None),
    (1, 1, 1, 2060, 9001, 64, 32, 2, 9, 0, "f32", FUSED, 2, None),          # no forced blocks
    (1, 1, 1, 5000, 9001, 128, 64, 2, 16, 1, "bf16", TWO, 0, None),         # row pairs, then the final Top-K
    (1, 4, 1, 4500, 9001, 64, 64, 2, 5, 1, "bf16", TWO, 1, None),
    (1, 2, 1, 300, 9001, 64, 32, 3, 7, 1, "bf16", TWO, 0, None),            # fan-out 3
    (1, 8, 1, 200, 9001, 128, 64, 2, 16, 1, "bf16", TWO, 0, None),          # matrix cores, up to 32 candidates
    (1, 2, 1, 300, 9001, 64, 32, 2, 20, 1, "bf16", TWO, 1, None),           # ... over the union of four rows
    (1, 2, 1, 5, 20000, 128, 32, 2, 16, 1, "bf16", SPLIT, 0, split_floor),  # few rows, level by level
    (1, 2, 1, 5, 20000, 128, 32, 2, 30, 1, "f32", SPLIT, 1, split_floor),
    (1, 2, 1, 5, 20000, 128, 32, 2, 16, 1, "bf16", SPLIT, 0, None),         # ... from node scores
    (1, 2, 1, 5, 20000, 128, 32, 2, 30, 1, "f32", SPLIT, 1, None),
    (1, 2, 1, 5, 60000, 64, 32, 4, 30, 1, "bf16", SPLIT, 0, None),          # two candidates per lane
])
def test_forced_blocks_first(shape, what):
    *problem, workspace = shape
    check(*problem, what, workspace)


@pytest.mark.parametrize("dtype,H,Hkv", [("f32", 3, 3), ("bf16", 12, 3)])
def test_blocks_of_minus_infinity_rank_last(dtype, H, Hkv):
    """Blocks whose every logit is -inf (keys of -inf in a dimension where the
    queries are positive) score -inf and are kept only where nothing else is
    left; only the leaf level is ranked here."""
    B, d, C, K = 1, 64, 32, 16
    N = Nq = 1024  # 32 blocks under 16 nodes
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, dtype, seed=62)
    x["q"][..., 3] = np.abs(x["q"][..., 3]) + 0.25
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, 1, dtype, schedule=FUSED)
    q, k = dev(x["q"], dtype), dev(x["k"], dtype)
    clean = k.double()
    bad = torch.arange(1, N // C, 4)
    rows = (bad[:, None] * C + torch.arange(C)).flatten().cuda()
    k[:, :, rows, 3] = float("-inf")
    idx, sc = pisa.select(p, q, k, pisa.build_pyramid(p, k), with_score=True)
    torch.cuda.synchronize()
    check_selection_valid(idx.cpu().numpy(), N, Nq, C, K, True)
    z = torch.matmul(q.double().view(B, Hkv, H // Hkv, Nq, d), clean.transpose(2, 3)[:, :, None]) / d ** 0.5
    want = z.view(B, Hkv, H // Hkv, Nq, N // C, C).logsumexp(-1).sum(2)  # [B, Hkv, Nq, blocks]
    want[..., bad.cuda()] = float("-inf")
    kept = idx.clamp(min=0).long()
    scored = torch.isfinite(sc) | torch.isneginf(sc) & (idx >= 0)
    ref = want.gather(-1, kept)
    assert bool(scored.any())
    ok = (sc.double() - ref).abs() < 1e-3
    assert bool((ok | (torch.isneginf(ref) & torch.isneginf(sc)))[scored].all())
    # no finite block is left out for one of -inf
    t = torch.arange(Nq, device="cuda")
    eligible = torch.arange(N // C, device="cuda") <= (t // C)[:, None]
    taken = (idx[..., None] == torch.arange(N // C, device="cuda")).any(-2)
    left_finite = (eligible & torch.isfinite(want) & ~taken).any(-1)
    forced = torch.stack([torch.zeros_like(t), (t // C - 1).clamp(min=0), t // C], -1)
    is_forced = (kept[..., None] == forced[None, None, :, None]).any(-1)
    took_bad = (torch.isneginf(ref) & (idx >= 0) & ~is_forced).any(-1)
    assert bool(left_finite.any()) and not bool((left_finite & took_bad).any())


@pytest.mark.parametrize("dtype,H,K", [("f32", 1, 7), ("f32", 4, 5), ("f32", 5, 40), ("bf16", 1, 40)])
@pytest.mark.parametrize("what", ["nan", "-inf"])
def test_flat_rows_with_nothing_left_to_rank(dtype, H, K, what):
    """The flat baseline row by row, with fewer blocks that can be ranked than
    are kept: the forced ones and those, ascending, then -1."""
    B, Hkv, Nq, N, d, C = 1, 1, 70, 3000, 64, 32
    x = inputs.random_qkv(B, H, Hkv, Nq, N, d, dtype, seed=64)
    p = pisa.make_problem(B, H, Hkv, Nq, N, d, C, 2, K, 1, dtype)
    q, k = dev(x["q"], dtype), dev(x["k"], dtype)
    if what == "nan":
        k[:, :, 3 * C:] = float("nan")
    else:
        q[..., 0] = 1.0
        k[:, :, 3 * C:, 0] = float("-inf")
    idx = pisa.select_flat_bsa(p, q, pisa.build_pyramid(p, k)).cpu().numpy()[0, 0]
    for r in range(Nq):
        c = (N - Nq + r) // C
        got = idx[r][idx[r] >= 0]
        assert np.all(np.diff(got) > 0) and np.all(idx[r][len(got):] == -1)
        assert {0, c - 1, c} <= set(got) <= {0, 1, 2, c - 1, c}
        if H == 1:
            assert len(got) == 5


def test_quality_of_masses_that_cannot_be_ranked():
    """Rows of NaN queries have NaN masses: their reference is the forced
    blocks; the other rows' is what it is without the NaN."""
    B, H, Hkv, N, d, C, K = 1, 2, 1, 2000, 64, 32, 6
    x = inputs.random_qkv(B, H, Hkv, N, N, d, "bf16", seed=65)
    p = pisa.make_problem(B, H, Hkv, N, N, d, C, 2, K, 1, "bf16")
    q, k = dev(x["q"], "bf16"), dev(x["k"], "bf16")
    idx = pisa.select(p, q, k, pisa.build_pyramid(p, k))
    rows = torch.tensor([0, 500, 959, 960, 1500, 1999], dtype=torch.int32, device="cuda")
    met, want = pisa.selection_quality(p, q, k, idx, rows)
    q[:, :, 960:] = float("nan")
    met2, ref = pisa.selection_quality(p, q, k, idx, rows)
    torch.cuda.synchronize()
    assert torch.equal(ref[0, 0, :3], want[0, 0, :3]) and torch.equal(met2[0, 0, :3], met[0, 0, :3])
    for i in range(3, 6):
        c = int(rows[i]) // C
        assert ref[0, 0, i].tolist() == [0, c - 1, c] + [-1] * (K - 3)
