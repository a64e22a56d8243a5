"""Top-k rows at the edges of the kernel's row kinds (rows held in registers, streamed rows, rows cut
into ranges) and with values that make the sampled bracket hard: everything large in one stretch, far
outliers, plateaus of equal values around the k-th, infinities.  The selection is integer work on given
scores: compared bit for bit with the oracle's top-k (ties: lower index)."""
import numpy as np
import pytest

from oracle import misa_oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def misa():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2605_07363_amd import misa as m
    return m


def rows_of(rng, L, k):
    """One row per kind of values."""
    x = rng.standard_normal((7, L)).astype(np.float32)
    x[1] -= 3.0
    x[1, L // 3:L // 3 + min(L, 2048)] += 4.0                 # the top in one stretch
    x[2, rng.choice(L, max(L // 500, 1), replace=False)] *= 1e4   # far outliers
    x[3] = np.where(rng.random(L) < 0.5, np.float32(0.0), np.minimum(x[3], 0))  # k-th on a plateau of zeros (-0.0 too)
    x[3, ::7] = -0.0
    x[4] = np.round(x[4] * 8) / 8                             # few distinct values
    x[5, rng.choice(L, min(L, 40), replace=False)] = np.inf
    x[5, rng.choice(L, min(L, 40), replace=False)] = -np.inf
    x[6] = -np.exp(6 * x[6])                                  # all negative, many binades
    return x


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("L,k", [(4096, 256), (4097, 4000), (8192, 2048), (8193, 1), (16387, 2048), (65536, 2048),
                                 (65537, 2048), (70001, 8192), (131072, 8192), (140000, 2048), (40000, 16384)])
def test_rows_match_the_oracle(misa, L, k, many):
    x = rows_of(np.random.default_rng(L + k), L, k)
    # causal prefixes around the row end and inside the row; with `many`, over 512 rows (they repeat)
    pos = np.array([L - 1, L - 2, (2 * L) // 3, min(L - 1, k), min(L - 1, max(k - 1, 0)), 8192 % L, L // 2], dtype=np.int32)
    rows, rep = len(x), (75 if many else 1)
    S = torch.from_numpy(x).cuda().repeat(rep, 1).contiguous()
    q_pos = torch.from_numpy(pos).cuda().repeat(rep).contiguous()
    p = misa.Problem(1, L, rows * rep, 64, 64, 8, misa.BF16, misa.BF16, q_pos, None)
    idx = torch.full((1, rows * rep, k), -9, dtype=torch.int32, device="cuda")
    val = torch.full((1, rows * rep, k), -9.0, dtype=torch.float32, device="cuda")
    misa.topk(p, S, k, idx, val, misa.alloc_workspace(p, misa.OP_TOPK, k))
    torch.cuda.synchronize()
    got, v = idx[0].cpu().numpy(), val[0].cpu().numpy()
    for t in range(rows):
        n = int(pos[t]) + 1
        ref = O.topk(x[t, :n].astype(np.float64), k)
        assert np.array_equal(got[t, :len(ref)], ref), (L, k, t)
        assert np.all(got[t, len(ref):] == -1)
        assert np.array_equal(v[t, :len(ref)], x[t, ref])
    for r in range(1, rep):
        assert np.array_equal(got[r * rows:(r + 1) * rows], got[:rows])


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("L,n,k,first,last", [(4096, 4000, 3976, 384, 413), (8192, 8100, 8080, 1280, 1320),
                                              (4096, 4095, 4090, 100, 163), (4096, 4000, 3950, 3900, 3959)])
def test_lowest_finite_values_below_a_prefix(misa, L, n, k, first, last, many):
    """The k-th largest is one of a few entries of the lowest finite value (a usual mask), the row ends
    before the buffer does: only visible keys, and of the masked ones the first."""
    x = np.random.default_rng(L + n + k).standard_normal(L).astype(np.float32)
    x[first:last + 1] = np.finfo(np.float32).min
    rows = 600 if many else 1
    S = torch.from_numpy(np.tile(x, (rows, 1))).cuda()
    seq_len = torch.full((rows,), n, dtype=torch.int32, device="cuda")
    p = misa.Problem(rows, L, 1, 64, 64, 8, misa.BF16, misa.BF16, None, seq_len)
    idx = torch.full((rows, 1, k), -9, dtype=torch.int32, device="cuda")
    val = torch.full((rows, 1, k), -9.0, dtype=torch.float32, device="cuda")
    misa.topk(p, S, k, idx, val, misa.alloc_workspace(p, misa.OP_TOPK, k))
    torch.cuda.synchronize()
    got, v = idx[:, 0].cpu().numpy(), val[:, 0].cpu().numpy()
    ref = O.topk(x[:n].astype(np.float64), k)
    assert len(ref) == k
    for t in range(rows):
        assert np.array_equal(got[t], ref), t
        assert np.array_equal(v[t], x[ref]), t
