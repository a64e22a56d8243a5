"""How many elements of a row the sampled top-k takes into its list.  Results do not depend on it (a row
whose list does not do is selected by the general path), time does.  Few rows above 65536 elements are
listed by a first kernel in segments of the workspace: its headers (elements listed, or -1 where the
sample gave no bracket) are what these tests read.  The list lengths are those of the bracket's own rule:
r ls elements for one line sampled of every ls, r = k / ls + 6 sqrt(k / ls) + 8."""
import numpy as np
import pytest

from oracle import misa_oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SEG_INTS = 64 + 2 * 7000     # a segment of the workspace: header, then entries
UNTOUCHED = -77


@pytest.fixture(scope="module")
def misa():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2605_07363_amd import misa as m
    return m


def expected_list(k, n, lines):
    ls = -(-(-(-n // 16)) // lines)
    return ls * (k / ls + 6 * (k / ls) ** 0.5 + 8)


def listed(misa, x, k, n=None):
    """Selects the top k of the rows of x (their first n elements), checks them and returns how many
    elements of each row were listed (-1: no bracket; UNTOUCHED: the row was not listed at all)."""
    rows, L = x.shape
    n = L if n is None else n
    S = torch.from_numpy(x).cuda()
    p = misa.Problem(rows, L, 1, 64, 64, 8, misa.BF16, misa.BF16, None,
                     torch.full((rows,), n, dtype=torch.int32, device="cuda"))
    idx = torch.full((rows, 1, k), -9, dtype=torch.int32, device="cuda")
    ws = misa.alloc_workspace(p, misa.OP_TOPK, k)
    ws.view(torch.int32).fill_(UNTOUCHED)
    misa.topk(p, S, k, idx, None, ws)
    torch.cuda.synchronize()
    got = idx[:, 0].cpu().numpy()
    for t in range(rows):
        assert np.array_equal(got[t], O.topk(x[t, :n].astype(np.float64), k)), t
    seg = ws.view(torch.int32)
    fills = seg[:seg.numel() // SEG_INTS * SEG_INTS].view(rows, -1, SEG_INTS)[:, :, 0].cpu().numpy()
    out = []
    for f in fills:
        f = f[f != UNTOUCHED]
        out.append(UNTOUCHED if f.size == 0 else -1 if (f < 0).any() else int(f.sum()))
    return np.array(out)


def test_the_longest_rows_are_listed(misa):
    got = listed(misa, np.random.default_rng(9).standard_normal((4, 524288)).astype(np.float32), 2048)
    assert (got >= 2048).all(), got


def test_rows_that_end_early_are_sampled_as_finely_as_the_list_expects(misa):
    x = np.random.default_rng(3).standard_normal((48, 140000)).astype(np.float32)
    k = 2048
    got = listed(misa, x, k, n=131072)
    assert (got >= k).all()
    assert got.mean() <= expected_list(k, 140000, 512), got.mean()
