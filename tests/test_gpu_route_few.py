"""Router of decode-like problems (a few queries per sequence): head scores against fp64 at the edges of the
block tiles, partial sums and row tiles, and the chosen heads by the margin rule on them."""
import numpy as np
import pytest

from oracle import misa_oracle as O
from paper_2605_07363_amd import workloads as WL
from helpers import assert_scores_close, check_index_set, oracle_view

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def misa():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2605_07363_amd import misa as m
    return m


@pytest.mark.parametrize("q_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_q,H,L,B", [(1, 64, 1024, 16), (1, 64, 1025, 16), (1, 33, 4111, 1), (1, 16, 63, 64), (1, 17, 16 * 65, 16),
                                       (3, 64, 2000, 16), (7, 40, 1031, 8), (2, 32, 700, 7), (5, 12, 515, 4), (7, 64, 1, 1),
                                       (1, 1, 9001, 2), (4, 64, 70000, 8)])
def test_head_scores(misa, n_q, H, L, B, q_dtype):
    wl = WL.scaled(WL.WORKLOADS["c1"], n_seq=2, L=L, n_q=n_q, H=H, h=min(H, 8), B=B, decode=n_q == 1, q_dtype=q_dtype, needles=0)
    inp = WL.make_inputs(wl, seed=L + H, seq_len=[L, max(1, L - L // 3)])
    if n_q > 1:
        inp["q_pos"] = np.maximum(0, L - 1 - np.array([0, 1, 5, L // 2, L, 2, L // 4])[:n_q]).astype(np.int32)
    dv = misa.to_device(inp)
    p = dv["problem"]
    Kp = torch.empty(2, p.M, 128, device="cuda")
    misa.pool_keys(p, dv["K"], dv["kscale"], Kp, misa.alloc_workspace(p, misa.OP_POOL))
    heads = torch.empty(2, n_q, p.h, dtype=torch.int32, device="cuda")
    E = torch.empty(2, n_q, H, device="cuda")
    misa.route_heads(p, dv["Q"], dv["W"], Kp, dv["K"], dv["kscale"], heads, E, misa.alloc_workspace(p, misa.OP_ROUTE))
    torch.cuda.synchronize()
    for s in range(2):
        for t in range(n_q):
            K, q, w, n = oracle_view(inp, s, t)
            _, ref = O.route_heads(q, w, K, B, p.h, n)
            assert_scores_close(E[s, t].cpu().numpy(), ref, f"E {s} {t}")
            check_index_set(heads[s, t].cpu().numpy(), ref, p.h, f"heads {s} {t}")


@pytest.mark.parametrize("q_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_seq,n_q,H,L,B", [(128, 4, 64, 768, 4), (128, 4, 64, 772, 4), (520, 3, 32, 130, 2), (64, 1, 64, 1024, 2),
                                             (600, 1, 64, 500, 2), (96, 6, 8, 1500, 4)])
def test_head_scores_of_many_sequences(misa, n_seq, n_q, H, L, B, q_dtype):
    """Both sides of the rules that count the workgroups of all sequences: a block of queries per read of the
    pooled keys or one, and the partial sums of a query.  A few sequences, repeated."""
    wl = WL.scaled(WL.WORKLOADS["c1"], n_seq=2, L=L, n_q=n_q, H=H, h=8, B=B, decode=n_q == 1, q_dtype=q_dtype, needles=0)
    inp = WL.make_inputs(wl, seed=L + H, seq_len=[L, max(1, L - L // 3)])
    if n_q > 1:
        inp["q_pos"] = np.maximum(0, L - 1 - np.array([0, 1, 5, L // 2, L, 2, L // 4])[:n_q]).astype(np.int32)
    dv = misa.to_device(inp)
    from dataclasses import replace
    rep = lambda x: x if x is None else x[torch.arange(n_seq, device="cuda") % 2].contiguous()
    p = replace(dv["problem"], n_seq=n_seq, seq_len=rep(dv["problem"].seq_len))
    K, ks, Q, W = rep(dv["K"]), rep(dv["kscale"]), rep(dv["Q"]), rep(dv["W"])
    Kp = torch.empty(n_seq, p.M, 128, device="cuda")
    misa.pool_keys(p, K, ks, Kp, misa.alloc_workspace(p, misa.OP_POOL))
    heads = torch.empty(n_seq, n_q, p.h, dtype=torch.int32, device="cuda")
    E = torch.empty(n_seq, n_q, H, device="cuda")
    misa.route_heads(p, Q, W, Kp, K, ks, heads, E, misa.alloc_workspace(p, misa.OP_ROUTE))
    torch.cuda.synchronize()
    assert torch.equal(E[2:], rep(E[:2])[2:]) and torch.equal(heads[2:], rep(heads[:2])[2:])
    for s in range(2):
        for t in range(n_q):
            Ks, q, w, n = oracle_view(inp, s, t)
            _, ref = O.route_heads(q, w, Ks, B, p.h, n)
            assert_scores_close(E[s, t].cpu().numpy(), ref, f"E {s} {t}")
            check_index_set(heads[s, t].cpu().numpy(), ref, p.h, f"heads {s} {t}")


@pytest.mark.parametrize("k_dtype,q_dtype", [("bf16", "bf16"), ("e4m3", "bf16"), ("f32", "bf16"), ("bf16", "f32"), ("e4m3", "f32")])
@pytest.mark.parametrize("H,L,B", [(64, 1400, 300), (37, 32 * 16 * 3 + 17, 16), (64, 32 * 40, 8), (20, 5000, 1024)])
def test_head_scores_of_a_chunk_with_tails(misa, k_dtype, q_dtype, H, L, B):
    """A prefill chunk whose workgroups do not fill the chip (block tiles split down to one each), and tail blocks of
    every length at which the rounds of their loads end."""
    tails = [1, 2, 3, 4, 5, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, B - 1, B]
    tails = [t for t in tails if t <= B]
    wl = WL.scaled(WL.WORKLOADS["c1"], n_seq=1, L=L, n_q=2 * len(tails), H=H, h=8, B=B, decode=False, k_dtype=k_dtype,
                   q_dtype=q_dtype, needles=0)
    inp = WL.make_inputs(wl, seed=L + H)
    full = L // B - 1
    inp["q_pos"] = np.array([full * B + t - 1 for t in tails] + [t - 1 for t in tails], dtype=np.int32)
    dv = misa.to_device(inp)
    p = dv["problem"]
    Kp = torch.empty(1, p.M, 128, device="cuda")
    misa.pool_keys(p, dv["K"], dv["kscale"], Kp, misa.alloc_workspace(p, misa.OP_POOL))
    heads = torch.empty(1, p.n_q, p.h, dtype=torch.int32, device="cuda")
    E = torch.empty(1, p.n_q, H, device="cuda")
    misa.route_heads(p, dv["Q"], dv["W"], Kp, dv["K"], dv["kscale"], heads, E, misa.alloc_workspace(p, misa.OP_ROUTE))
    torch.cuda.synchronize()
    for t in range(p.n_q):
        K, q, w, n = oracle_view(inp, 0, t)
        _, ref = O.route_heads(q, w, K, B, p.h, n)
        assert_scores_close(E[0, t].cpu().numpy(), ref, f"E {t}")
        check_index_set(heads[0, t].cpu().numpy(), ref, p.h, f"heads {t}")
