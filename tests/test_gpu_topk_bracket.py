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


def rows_with(kind, rng, rows, L):
    x = rng.standard_normal((rows, L)).astype(np.float32)
    if kind == "masked":
        x[:, int(L * 0.7):] = np.finfo(np.float32).min
    elif kind == "outliers":
        x[:, ::997] *= np.float32(1e4)
    elif kind == "heavy":
        x = np.exp(4 * x)
    return x


@pytest.mark.parametrize("kind", ["masked", "outliers", "heavy"])
@pytest.mark.parametrize("L,k,lines", [(131072, 512, 256), (131072, 2048, 256), (200003, 2048, 512)])
def test_far_values_leave_the_bracket_narrow(misa, kind, L, k, lines):
    """Values far from the rest make the sample's histogram coarse; the rows are listed all the same, and
    not many more elements than the rank calls for (the elements of one bin with 64 samples in it)."""
    got = listed(misa, rows_with(kind, np.random.default_rng(L + k), 8, L), k)
    assert (got >= k).all(), got
    ls = -(-(-(-L // 16)) // lines)
    assert got.mean() <= expected_list(k, L, lines) + 64 * ls, got.mean()


def test_the_longest_rows_are_listed(misa):
    got = listed(misa, rows_with("gauss", np.random.default_rng(9), 4, 524288), 2048)
    assert (got >= 2048).all(), got


def test_rows_that_end_early_are_sampled_as_finely_as_the_list_expects(misa):
    x = np.random.default_rng(3).standard_normal((48, 140000)).astype(np.float32)
    k = 2048
    got = listed(misa, x, k, n=131072)
    assert (got >= k).all()
    assert got.mean() <= expected_list(k, 140000, 512), got.mean()


def values(kind, rng, rows, L):
    x = rng.standard_normal((rows, L)).astype(np.float32)
    low = np.finfo(np.float32).min
    if kind == "masked tail":
        x[:, int(L * 0.7):] = low
    elif kind == "masked":
        x[rng.random(x.shape) < 0.3] = low
    elif kind == "outliers":
        x[:, ::997] *= np.float32(1e4)
    elif kind == "largest finite":
        x[:, ::997] = np.finfo(np.float32).max
        x[:, 5::997] = low
    elif kind == "heavy":
        x = np.exp(4 * x)
    elif kind == "tiny":                                   # subnormal numbers and both zeros
        x = (x * np.float32(1e-40)).astype(np.float32)
        x[:, ::3] = -0.0
    elif kind == "zeros":                                  # the k-th largest on a plateau of nearly the whole row
        x = np.where(rng.random(x.shape) < 0.005, np.abs(x), np.float32(0))
        x[:, ::2] = np.where(x[:, ::2] == 0, np.float32(-0.0), x[:, ::2])
    elif kind == "plateau edge":                           # a plateau that ends around the k-th largest
        x = np.where(x > 1.85, x, np.float32(1.5))
    elif kind == "constant":
        x[:] = 1.5
    elif kind == "masked constant":
        x[:] = low
        x[:, ::50] = 2.0
    elif kind == "runs":                                   # 16 neighbours are nearly alike: the sample's lines are
        x = np.repeat(rng.standard_normal((rows, -(-L // 16))).astype(np.float32), 16, axis=1)[:, :L] + x * np.float32(0.01)
    elif kind == "steps":
        x = np.repeat(rng.standard_normal((rows, -(-L // 64))).astype(np.float32), 64, axis=1)[:, :L]
    elif kind == "infinite":
        x[:, ::11] = np.inf
        x[:, 1::3] = -np.inf
    elif kind == "nan":
        x[:, 7::1000] = np.nan
    return np.ascontiguousarray(x)


KINDS = ["masked tail", "masked", "outliers", "largest finite", "heavy", "tiny", "zeros", "plateau edge", "constant",
         "masked constant", "runs", "steps", "infinite", "nan"]


def reference(x, k):
    """Top k by value (NaN above all, as the order of the integer images has it), lower index first."""
    y = np.where(np.isnan(x), np.inf, x.astype(np.float64))
    o = np.lexsort((np.arange(len(x)), -y, ~np.isnan(x)))
    return np.sort(o[:k])


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("rows,L,k", [(3, 4096, 256), (600, 4095, 2000), (2, 8192, 2048), (40, 20011, 2048), (5, 65536, 8192),
                                      (600, 9001, 512), (32, 131072, 2048), (2, 140001, 512), (2, 524288, 2048),
                                      (2, 524287, 16384)])
def test_hard_values_match_a_sort(misa, kind, rows, L, k):
    distinct = min(rows, 32 if L <= 131072 else 2)
    x = values(kind, np.random.default_rng(L + k), distinct, L)
    S = torch.from_numpy(x).cuda()[torch.arange(rows) % distinct].contiguous()
    p = misa.Problem(rows, L, 1, 64, 64, 8, misa.BF16, misa.BF16, None, None)
    idx = torch.full((rows, 1, k), -9, dtype=torch.int32, device="cuda")
    val = torch.full((rows, 1, k), -9.0, dtype=torch.float32, device="cuda")
    misa.topk(p, S, k, idx, val, misa.alloc_workspace(p, misa.OP_TOPK, k))
    torch.cuda.synchronize()
    got, v = idx[:, 0].cpu().numpy(), val[:, 0].cpu().numpy()
    for t in range(distinct):
        ref = reference(x[t], k)
        assert np.array_equal(got[t], ref), t
        assert np.array_equal(v[t].view(np.int32), x[t, ref].view(np.int32)), t
        assert np.array_equal(got[t::distinct], np.broadcast_to(got[t], got[t::distinct].shape)), t


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("rows,L,k", [
    (255, 45056, 4000),      # 1024 threads
    (256, 8193, 2048),       # 512 threads, two rows per CU: the shortest row,
    (300, 45056, 4000),      # the longest one with a list beyond 53 KB,
    (511, 20011, 5000),      # and one between
    (256, 45057, 4000),      # 1024 threads again
    (511, 45056, 9000),      # a list that does not fit twice
    (512, 45056, 4000),      # more rows: lists of up to 53 KB only
])
def test_hard_values_of_less_than_two_rows_per_cu(misa, kind, rows, L, k):
    test_hard_values_match_a_sort(misa, kind, rows, L, k)
