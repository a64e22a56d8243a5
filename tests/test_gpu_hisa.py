"""GPU parity tests of the comparison indexers misa_hisa_select and
misa_block_sparse_select (Eq. block_score, Eq. final_topk; "Baselines") against the
fp64 oracle: chosen blocks by the margin rule on the oracle's block scores (first and last
block always present), final tokens by the margin rule on the dense scores inside the
blocks the GPU chose, values within the score tolerance."""
import numpy as np
import pytest
import torch

from oracle import misa_oracle as O
from paper_2605_07363_amd import workloads as WL
from helpers import oracle_view, assert_scores_close, check_index_set

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def misa():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2605_07363_amd import misa as m
    return m


def small(base, **kw):
    return WL.scaled(WL.WORKLOADS[base], **kw)


CASES = {
    # name: (workload, m)
    "bf16_decode": (small("c1", n_seq=3, L=5000, B=128, k=300), 6),
    "fp8_decode": (small("c3", n_seq=2, L=4133, B=128, k=512, needles=16), 8),
    "f32_decode": (small("c0", L=1500, B=64, k=100), 4),
    "bf16_prefill": (small("c2", L=3000, n_q=37, B=64, k=200), 9),
    "fp8_prefill": (small("c4", L=2500, n_q=20, B=32, k=128, k_cand=0, needles=16), 12),
    "all_blocks": (small("c1", n_seq=2, L=1000, B=100, k=64), 16),       # m >= M: the dense indexer
    "two_blocks": (small("c2", L=2000, n_q=9, B=50, k=60), 2),           # only the forced blocks
}


def _random_case(i):
    rng = np.random.default_rng(7000 + i)
    decode = bool(rng.integers(0, 2))
    H = int(rng.choice([1, 8, 17, 32, 64]))
    L = int(rng.integers(60, 4000))
    B = int(rng.choice([1, 5, 16, 64, 128, 700]))
    m = int(rng.integers(2, max(3, min(16384 // B, 40))))
    k = int(rng.integers(1, min(m * B, 400) + 1))
    wl = WL.scaled(WL.WORKLOADS["c3" if decode else "c2"], n_seq=int(rng.integers(1, 4)), L=L,
                   n_q=1 if decode else int(rng.integers(2, 40)), H=H, h=int(rng.integers(1, H + 1)), B=B, k=k,
                   k_cand=0, k_dtype=["f32", "bf16", "e4m3"][i % 3], q_dtype=["bf16", "e4m3", "f32"][(i // 3) % 3],
                   needles=int(rng.integers(0, 9)), name=f"random{i}")
    return wl, m


RANDOM = {f"random{i}": _random_case(i) for i in range(18)}
CASES.update(RANDOM)


def forced_scores(J):
    J = J.copy()
    if J.shape[0]:
        J[0] = np.inf
        J[-1] = np.inf
    return J


def run(misa, name, seq_len=None, q_pos=None, page_size=0):
    wl, m = CASES[name]
    inp = WL.make_inputs(wl, seed=300 + sum(map(ord, name)), seq_len=seq_len)
    if q_pos is not None:
        inp["q_pos"] = np.asarray(q_pos, dtype=np.int32)
    dv = misa.to_device(inp)
    if page_size:
        dv = misa.paginate(dv, page_size, seed=3)
    p = dv["problem"]
    rows = (wl.n_seq, wl.n_q)
    Kp = torch.empty((wl.n_seq, p.M, wl.d), dtype=torch.float32, device="cuda")
    misa.pool_keys(p, dv["K"], dv["kscale"], Kp, misa.alloc_workspace(p, misa.OP_POOL))
    blocks = torch.full(rows + (m,), -9, dtype=torch.int32, device="cuda")
    idx = torch.full(rows + (wl.k,), -9, dtype=torch.int32, device="cuda")
    val = torch.full(rows + (wl.k,), 9.0, dtype=torch.float32, device="cuda")
    ws = misa.alloc_workspace(p, misa.OP_HISA, m)
    misa.hisa_select(p, dv["Q"], dv["W"], Kp, dv["K"], dv["kscale"], m, wl.k, idx, val, blocks, ws)
    bs_blocks = torch.full(rows + (m,), -9, dtype=torch.int32, device="cuda")
    bs_idx = torch.full(rows + (m * wl.B,), -9, dtype=torch.int32, device="cuda")
    misa.block_sparse_select(p, dv["Q"], dv["W"], Kp, m, bs_idx, bs_blocks, ws)
    torch.cuda.synchronize()
    assert torch.equal(blocks, bs_blocks)
    return inp, wl, m, blocks.cpu().numpy(), idx.cpu().numpy(), val.cpu().numpy(), bs_idx.cpu().numpy()


def check(inp, wl, m, blocks, idx, val, bs_idx):
    exact = 0
    for s in range(wl.n_seq):
        for t in range(wl.n_q):
            K, q, w, n = oracle_view(inp, s, t)
            what = f"{wl.name} row {s},{t} (n={n})"
            J = O.block_scores(q, w, K, wl.B, n)
            M = J.shape[0]
            got_blocks = blocks[s, t]
            check_index_set(got_blocks, forced_scores(J), m, "blocks " + what)
            chosen = got_blocks[got_blocks >= 0]
            if M:
                assert chosen[0] == 0 and chosen[-1] == M - 1, what
            exact += np.array_equal(chosen, O.select_blocks(J, m)) if M else 1
            omega = O.block_tokens(chosen, wl.B, n)
            # Block-Sparse: the tokens of the chosen blocks at their slots
            expect = np.full(m * wl.B, -1, dtype=np.int64)
            for i, b in enumerate(chosen.tolist()):
                toks = np.arange(b * wl.B, min((b + 1) * wl.B, n))
                expect[i * wl.B:i * wl.B + toks.shape[0]] = toks
            np.testing.assert_array_equal(bs_idx[s, t], expect, err_msg=what)
            # HISA fine stage on the GPU's blocks
            dense = O.dsa_scores(q, w, K, n)
            final = idx[s, t][idx[s, t] >= 0]
            assert set(final.tolist()) <= set(omega.tolist()), what
            pos = np.searchsorted(omega, final)
            padded = np.concatenate([pos, np.full(wl.k - pos.shape[0], -1, dtype=pos.dtype)])
            check_index_set(padded, dense[omega], wl.k, "tokens " + what)
            assert_scores_close(val[s, t, :final.shape[0]], dense[final], "values " + what)
            assert np.all(np.isneginf(val[s, t, final.shape[0]:]))
    return exact


@pytest.mark.parametrize("name", [n for n in CASES if n not in RANDOM])
def test_hisa_and_block_sparse_match_oracle(misa, name):
    inp, wl, m, blocks, idx, val, bs_idx = run(misa, name)
    exact = check(inp, wl, m, blocks, idx, val, bs_idx)
    assert exact >= 0.9 * wl.n_seq * wl.n_q


@pytest.mark.parametrize("name", list(RANDOM))
def test_hisa_random_problems(misa, name):
    # seeded random shapes, storage types, ragged batches, unsorted query positions, paged keys
    wl, m = CASES[name]
    rng = np.random.default_rng(sum(map(ord, name)))
    seq_len = rng.integers(0, wl.L + 1, wl.n_seq).astype(np.int32) if rng.integers(0, 2) else None
    q_pos = rng.integers(0, wl.L, wl.n_q) if (not wl.decode and rng.integers(0, 2)) else None
    inp, wl, m, blocks, idx, val, bs_idx = run(misa, name, seq_len=seq_len, q_pos=q_pos,
                                               page_size=int(rng.choice([0, 16, 128])))
    check(inp, wl, m, blocks, idx, val, bs_idx)


def test_hisa_with_all_blocks_is_the_dense_indexer(misa):
    inp, wl, m, blocks, idx, val, _ = run(misa, "all_blocks")
    for s in range(wl.n_seq):
        K, q, w, n = oracle_view(inp, s, 0)
        dense = O.dsa_scores(q, w, K, n)
        check_index_set(idx[s, 0], dense, wl.k, f"dense seq {s}")


def test_hisa_ragged_and_early_queries(misa):
    wl, m = CASES["bf16_prefill"]
    q_pos = sorted([0, 1, 63, 64, 65, 127, 128, 500, 1279, 1280, 1281] + list(range(2974, 3000)))
    assert len(q_pos) == wl.n_q
    inp, wl, m, blocks, idx, val, bs_idx = run(misa, "bf16_prefill", seq_len=np.array([2100], dtype=np.int32),
                                               q_pos=q_pos)
    check(inp, wl, m, blocks, idx, val, bs_idx)


def test_hisa_argument_checks(misa):
    wl, _ = CASES["bf16_decode"]
    dv = misa.to_device(WL.make_inputs(wl, seed=1))
    p = dv["problem"]
    Kp = torch.zeros((wl.n_seq, p.M, wl.d), dtype=torch.float32, device="cuda")
    idx = torch.zeros((wl.n_seq, 1, 64), dtype=torch.int32, device="cuda")
    ws = misa.alloc_workspace(p, misa.OP_HISA, 4)
    for m, k in ((1, 64), (129, 64), (4, 0), (4, 4 * 128 + 1)):
        with pytest.raises(misa.MisaError):
            misa.hisa_select(p, dv["Q"], dv["W"], Kp, dv["K"], dv["kscale"], m, k, idx, None, None, ws)
    with pytest.raises(misa.MisaError):
        misa.hisa_select(p, dv["Q"], dv["W"], Kp, dv["K"], dv["kscale"], 4, 64, idx, None, None, None)


@pytest.mark.parametrize("n_q,H,L,B", [(1, 64, 4100, 32), (2, 32, 4096, 31), (3, 33, 2050, 16), (17, 32, 9000, 64),
                                       (40, 64, 16500, 128), (5, 1, 130, 1), (2100, 64, 1030, 8), (64, 8, 600, 600)])
def test_block_scores_on_the_matrix_core(misa, n_q, H, L, B):
    """Block scores of bf16 queries against fp64, at the edges of the query steps, head slots and block
    tiles.  They are the first rows of the workspace.  Bound: products are exact, about 128 + H fp32
    additions of terms whose absolute sum is A: 2^-24 * sqrt(128 + H) * A at one standard deviation of
    independent roundings; eight are allowed."""
    g = torch.Generator(device="cuda").manual_seed(n_q * H)
    M = -(-L // B)
    Kp = torch.randn(2, M, 128, generator=g, device="cuda") * 0.05
    Q = (torch.randn(2, n_q, H, 128, generator=g, device="cuda") * 0.09).to(torch.bfloat16)
    W = torch.randn(2, n_q, H, generator=g, device="cuda")
    pos = torch.randint(0, L, (n_q,), generator=g, device="cuda", dtype=torch.int32)
    p = misa.Problem(2, L, n_q, H, B, 1, misa.BF16, misa.BF16, pos)
    m = 2
    idx = torch.empty(2, n_q, m * B, dtype=torch.int32, device="cuda")
    ws = misa.alloc_workspace(p, misa.OP_HISA, m)
    misa.block_sparse_select(p, Q, W, Kp, m, idx, None, ws)
    torch.cuda.synchronize()
    J = ws[:2 * n_q * M * 4].view(torch.float32).view(2, n_q, M).double()
    for s in range(2):
        dots = (Q[s].double().reshape(-1, 128) @ Kp[s].double().T).relu().view(n_q, H, M)
        ref = (W[s].double()[..., None] * dots).sum(1)
        size = (W[s].double().abs()[..., None] * (Q[s].double().abs().reshape(-1, 128) @ Kp[s].double().abs().T).view(n_q, H, M)).sum(1)
        Mn = (pos.long()[:, None] + B) // B
        b = torch.arange(M, device="cuda")[None]
        forced, none = (b == 0) | (b == Mn - 1), b >= Mn
        assert bool((J[s][none] == -np.inf).all()) and bool((J[s][forced & ~none] == np.inf).all())
        inner = ~forced & ~none
        tol = 8 * 2.0 ** -24 * (128 + H) ** 0.5 * size
        assert bool(((J[s] - ref).abs() <= tol)[inner].all())


@pytest.mark.parametrize("H", [64, 40, 32, 24])
@pytest.mark.parametrize("what", ["key", "negative_gates", "large_key", "query", "large_product"])
def test_block_scores_of_infinite_components(misa, H, what):
    """A block with an infinite component (or one above the largest bf16), a query with an infinite
    component and a finite product above the largest fp32 score as their products say; every other block and
    query as without them.  One such component per block or query, so that no dot product is infinity minus
    infinity (large_product: all components of a block have the sign of the query's and one is large)."""
    n_q, L, B = 5, 1000, 20
    g = torch.Generator().manual_seed(H)
    M = L // B
    Kp = torch.randn(M, 128, generator=g) * 0.05
    Q = (torch.randn(n_q, H, 128, generator=g) * 0.09).to(torch.bfloat16)
    W = torch.rand(n_q, H, generator=g) + 0.1
    if what == "query":
        Q[2, 3, 17] = float("inf")
        Q[4, H - 1, 100] = -float("inf")
    elif what == "large_product":                # the key's nearest bf16 is above it: its second piece is negative
        Q, Kp, W = Q.abs(), Kp.abs(), W * 0.05
        Q[2] *= 1e6
        Kp[7, 5] = Kp[31, 17] = 1.0085e38
    else:
        for i, b in enumerate((1, 7, 31, 32, 40, 48)):
            Kp[b, (37 * i) % 128] = 3.4e38 if what == "large_key" else float("inf") if i % 2 else -float("inf")
    if what == "negative_gates":
        W = -W
    if what == "large_key":
        W *= 0.05                                # (the sums stay finite)
    p = misa.Problem(1, L, n_q, H, B, 1, misa.BF16, misa.BF16, torch.full((n_q,), L - 1, dtype=torch.int32, device="cuda"))
    idx = torch.empty(1, n_q, 2 * B, dtype=torch.int32, device="cuda")
    ws = misa.alloc_workspace(p, misa.OP_HISA, 2)
    misa.block_sparse_select(p, Q[None].cuda(), W[None].cuda().contiguous(), Kp[None].cuda(), 2, idx, None, ws)
    torch.cuda.synchronize()
    J = ws[:n_q * M * 4].view(torch.float32).view(n_q, M).double().cpu()
    products = Q.double()[:, :, None, :] * Kp.double()[None, None]
    terms = W.double()[:, :, None] * products.sum(-1).relu()
    ref, size = terms.sum(1), (W.double().abs()[:, :, None] * products.abs().sum(-1)).sum(1)
    assert not ref[:, 1:-1].isnan().any()
    assert what == "large_key" or (ref[:, 1:-1].abs() > 3.4e38).any()
    for q in range(n_q):
        for b in range(1, M - 1):
            r, got = ref[q, b].item(), J[q, b].item()
            if abs(r) > 3.4e38:                  # infinite in fp32
                assert got == float("inf") * np.sign(r), (q, b, got, r)
            else:
                assert abs(got - r) <= 8 * 2.0 ** -24 * (128 + H) ** 0.5 * size[q, b].item(), (q, b, got, r)


MANY = {
    # from 704 rows on the dense scores of 2048 to 8192 candidates (m blocks of B) and their top-k are one kernel
    "bf16": (small("c2", L=3001, n_q=1024, B=64, k=200, H=32, h=8), 9),
    "fp8_keys": (small("c4", L=2500, n_q=1100, B=32, k=128, k_cand=0, H=64, needles=16), 12),
    "two_sequences": (small("c2", n_seq=2, L=2777, n_q=513, B=100, k=300, H=40, h=8), 7),
    "fp8_queries": (small("c4", n_seq=2, L=2000, n_q=512, B=64, k=64, k_cand=0, H=17, h=8, q_dtype="e4m3", needles=4), 5),
    "2560_candidates": (small("c2", L=3001, n_q=1024, B=64, k=200, H=32, h=8), 40),
    "2048_candidates_fp8_keys": (small("c4", L=2500, n_q=1100, B=32, k=128, k_cand=0, H=64, needles=16), 64),
    "2100_candidates_of_two": (small("c2", n_seq=2, L=2777, n_q=513, B=100, k=300, H=40, h=8), 21),
    "2112_candidates_fp8_queries": (small("c4", n_seq=2, L=2500, n_q=512, B=64, k=64, k_cand=0, H=17, h=8, q_dtype="e4m3", needles=4), 33),
    "8192_candidates": (small("c2", L=9000, n_q=1030, B=128, k=2048, H=8, h=8), 64),
    "8256_candidates": (small("c2", L=9000, n_q=1030, B=129, k=2048, H=8, h=8), 64),
    "k_of_all": (small("c2", L=600, n_q=1024, B=50, k=250, H=16, h=8), 5),
}


@pytest.mark.parametrize("name", list(MANY))
def test_many_rows_equal_their_queries_by_themselves(misa, name):
    """All rows of a call, from queries that see one key to those that see all and of sequences of several
    lengths, bit for bit against calls of at most 500 rows, and some rows against the oracle."""
    wl, m = MANY[name]
    n_q, seq_len = wl.n_q, (None if wl.n_seq == 1 else [wl.L, wl.L // 3])
    inp = WL.make_inputs(wl, seed=41, seq_len=seq_len)
    q_pos = np.unique(np.concatenate([np.arange(8), np.linspace(0, wl.L - 1, n_q - 8).astype(int)]))
    q_pos = np.sort(np.concatenate([q_pos, np.full(n_q - len(q_pos), wl.L - 1)])).astype(np.int32)
    inp["q_pos"] = q_pos
    dv = misa.to_device(inp)
    p = dv["problem"]
    Kp = torch.empty((wl.n_seq, p.M, wl.d), dtype=torch.float32, device="cuda")
    misa.pool_keys(p, dv["K"], dv["kscale"], Kp, misa.alloc_workspace(p, misa.OP_POOL))

    def select(p, Q, W, Kp, K, kscale):
        rows = (p.n_seq, p.n_q)
        blocks = torch.full(rows + (m,), -9, dtype=torch.int32, device="cuda")
        idx = torch.full(rows + (wl.k,), -9, dtype=torch.int32, device="cuda")
        val = torch.full(rows + (wl.k,), 9.0, dtype=torch.float32, device="cuda")
        misa.hisa_select(p, Q, W, Kp, K, kscale, m, wl.k, idx, val, blocks, misa.alloc_workspace(p, misa.OP_HISA, m))
        torch.cuda.synchronize()
        return blocks, idx, val

    blocks, idx, val = select(p, dv["Q"], dv["W"], Kp, dv["K"], dv["kscale"])
    for s in range(wl.n_seq):
        one = None if p.seq_len is None else p.seq_len[s:s + 1].contiguous()
        for t in range(0, n_q, 500):
            part = misa.Problem(1, p.L, min(500, n_q - t), p.H, p.B, p.h, p.k_dtype, p.q_dtype, p.q_pos[t:t + 500].contiguous(), one)
            b1, i1, v1 = select(part, dv["Q"][s:s + 1, t:t + 500].contiguous(), dv["W"][s:s + 1, t:t + 500].contiguous(), Kp[s:s + 1].contiguous(),
                                dv["K"][s:s + 1].contiguous(), None if dv["kscale"] is None else dv["kscale"][s:s + 1].contiguous())
            assert torch.equal(blocks[s:s + 1, t:t + 500], b1), (s, t)
            assert torch.equal(idx[s:s + 1, t:t + 500], i1), (s, t)
            assert torch.equal(val[s:s + 1, t:t + 500].view(torch.int32), v1.view(torch.int32)), (s, t)
    some = np.unique(np.concatenate([[0, 1, 7, n_q - 1], np.random.default_rng(5).integers(0, n_q, 6)]))
    few = dict(inp, wl=WL.scaled(wl, n_q=len(some)), Q=inp["Q"][:, some], W=inp["W"][:, some], q_pos=q_pos[some])
    sel = lambda x: x.cpu().numpy()[:, some]
    bs = np.full((wl.n_seq, len(some), m * wl.B), -1, dtype=np.int64)
    for s in range(wl.n_seq):
        for i, t in enumerate(some):
            n = oracle_view(few, s, i)[3]
            for j, b in enumerate(sel(blocks)[s, i]):
                toks = np.arange(max(b, 0) * wl.B, min((b + 1) * wl.B, n)) if b >= 0 else np.arange(0)
                bs[s, i, j * wl.B:j * wl.B + len(toks)] = toks
    check(few, few["wl"], m, sel(blocks), sel(idx), sel(val), bs)
