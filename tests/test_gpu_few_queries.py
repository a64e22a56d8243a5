"""Scoring of a few queries per sequence, which share one read of the keys: every row must equal, bit for
bit, the decode call (one query per sequence) on the cache truncated to what the query sees; the decode
call is held against the oracle in the stage tests."""
from dataclasses import replace

import pytest

from paper_2605_07363_amd import workloads as WL

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def misa():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2605_07363_amd import misa as m
    return m


@pytest.mark.parametrize("k_dtype", ["bf16", "e4m3"])
@pytest.mark.parametrize("n_q,h,L,page", [(2, 8, 1023, 0), (3, 8, 4097, 64), (4, 5, 2049, 0), (5, 8, 1500, 16), (6, 1, 777, 0),
                                          (7, 8, 5000, 256), (2, 16, 2048, 0), (3, 9, 1281, 64), (4, 16, 3000, 0),
                                          (5, 12, 1024, 0), (7, 16, 4100, 16), (4, 17, 1100, 0), (6, 32, 900, 0), (2, 8, 3, 0)])
def test_rows_equal_the_decode_call(misa, k_dtype, n_q, h, L, page):
    wl = WL.scaled(WL.WORKLOADS["c1"], n_seq=3, L=L, n_q=n_q, H=32, h=h, decode=False, k_dtype=k_dtype, needles=2)
    dv = misa.to_device(WL.make_inputs(wl, seed=n_q * 100 + h, seq_len=[L, max(L - 5, 1), 2]))
    if page:
        dv = misa.paginate(dv, page, seed=1)
    # positions out of order, at the end of the cache, near its start and before it
    pos = torch.tensor([L - 1, 0, L // 2, -1, L - 2, L // 3, L + 7][:n_q], dtype=torch.int32, device="cuda")
    p = replace(dv["problem"], q_pos=pos)
    g = torch.Generator().manual_seed(h)
    heads = torch.stack([torch.randperm(32, generator=g)[:h].sort().values for _ in range(3 * n_q)])
    heads = heads.to(torch.int32).view(3, n_q, h).cuda()
    heads[0, 0, 0] = 99                      # not a head: contributes nothing
    S = torch.full((3, n_q, L), 7.0, device="cuda")
    misa.score_tokens(p, dv["Q"], dv["W"], heads, dv["K"], dv["kscale"], S)
    for t in range(n_q):
        n = (pos[t] + 1).clamp(min=0)
        one = replace(p, n_q=1, q_pos=None, seq_len=torch.minimum(dv["problem"].seq_len, n).to(torch.int32).contiguous())
        ref = torch.full((3, 1, L), 9.0, device="cuda")
        misa.score_tokens(one, dv["Q"][:, t:t + 1].contiguous(), dv["W"][:, t:t + 1].contiguous(),
                          heads[:, t:t + 1].contiguous(), dv["K"], dv["kscale"], ref)
        assert torch.equal(S[:, t], ref[:, 0]), (n_q, h, t)


@pytest.mark.parametrize("k_dtype", ["bf16", "e4m3"])
@pytest.mark.parametrize("n_q,h,L,page,more", [(n_q, h, L, page, more) for n_q, h, L, page in
                                               [(2, 8, 1023, 0), (3, 8, 4097, 64), (4, 5, 2049, 0), (5, 8, 1500, 16), (6, 1, 777, 0),
                                                (7, 8, 5000, 256), (2, 16, 2048, 0), (3, 9, 1281, 64), (4, 16, 3000, 0),
                                                (5, 12, 1024, 0), (7, 16, 4100, 16)] for more in (0, 1)])
def test_many_sequences_equal_the_decode_call(misa, k_dtype, n_q, h, L, page, more):
    """The same at both sides of the rule that lets the queries share the read: at most 256 workgroups of one
    query and 1024 keys, and more."""
    wl = WL.scaled(WL.WORKLOADS["c1"], n_seq=3, L=L, n_q=n_q, H=32, h=h, decode=False, k_dtype=k_dtype, needles=2)
    dv = misa.to_device(WL.make_inputs(wl, seed=n_q * 100 + h, seq_len=[L, max(L - 5, 1), 2]))
    N = 256 // (n_q * -(-L // 1024)) + more
    rep = lambda x: x if x is None else x[torch.arange(N, device="cuda") % 3].contiguous()
    pos = torch.tensor([L - 1, 0, L // 2, -1, L - 2, L // 3, L + 7][:n_q], dtype=torch.int32, device="cuda")
    p3 = replace(dv["problem"], q_pos=pos)
    g = torch.Generator().manual_seed(h)
    heads = torch.stack([torch.randperm(32, generator=g)[:h].sort().values for _ in range(3 * n_q)])
    heads = heads.to(torch.int32).view(3, n_q, h).cuda()
    big = {"K": rep(dv["K"]), "kscale": rep(dv["kscale"]), "problem": replace(p3, n_seq=N, seq_len=rep(p3.seq_len))}
    if page:
        big = misa.paginate(big, page, seed=1)
    S = torch.full((N, n_q, L), 7.0, device="cuda")
    misa.score_tokens(big["problem"], rep(dv["Q"]), rep(dv["W"]), rep(heads), big["K"], big["kscale"], S)
    for t in range(n_q):
        n = (pos[t] + 1).clamp(min=0)
        one = replace(p3, n_q=1, q_pos=None, seq_len=torch.minimum(p3.seq_len, n).to(torch.int32).contiguous())
        ref = torch.full((3, 1, L), 9.0, device="cuda")
        misa.score_tokens(one, dv["Q"][:, t:t + 1].contiguous(), dv["W"][:, t:t + 1].contiguous(),
                          heads[:, t:t + 1].contiguous(), dv["K"], dv["kscale"], ref)
        assert torch.equal(S[:, t], rep(ref)[:, 0]), (n_q, h, t)
