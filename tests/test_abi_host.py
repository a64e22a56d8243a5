"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every symbol the header declares, and rejects bad arguments before launching."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def misa():
    from paper_2605_07363_amd import misa as m
    return m


def test_every_declared_symbol_is_exported(misa):
    header = open(os.path.join(ROOT, "include", "misa.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = set(re.findall(r"\b(misa_[a-z0-9_]+)\s*\(", header))
    assert {"misa_pool_keys", "misa_route_heads", "misa_score_tokens", "misa_topk", "misa_rerank", "misa_select_tokens", "misa_hisa_select", "misa_block_sparse_select", "misa_pool_keys_update", "misa_route_heads_proxy",
            "misa_probe_hbm_read", "misa_probe_mfma_bf16", "misa_probe_mfma_bf16_operands", "misa_convert_queries",
            "misa_workspace_bytes", "misa_last_error", "misa_version"} <= names
    for n in names:
        assert hasattr(misa.lib, n), f"{n} declared in misa.h but not exported"
    assert misa.version() == 1000


def _prob(misa, **kw):
    base = dict(n_seq=2, L=1000, n_q=1, H=64, B=64, h=8, k_dtype=misa.BF16, q_dtype=misa.BF16)
    base.update(kw)
    return misa.Problem(**base)


FAKE = ctypes.c_void_p(0x1000)   # 16- and 256-byte aligned, never dereferenced on the host


def _pool(misa, p, K=FAKE, kscale=None, Kp=FAKE):
    return misa.lib.misa_pool_keys(ctypes.byref(p.c()), K, kscale, Kp, None, 0, None)


def test_invalid_problem_fields_are_rejected_without_launch(misa):
    INVALID, UNSUPPORTED = 1, 2
    for kw in (dict(n_seq=0), dict(L=0), dict(n_q=0), dict(H=0), dict(B=0), dict(h=0), dict(h=65, H=64),
               dict(k_dtype=7), dict(q_dtype=-1), dict(n_q=2)):   # n_q > 1 without q_pos
        assert _pool(misa, _prob(misa, **kw)) == INVALID, kw
        assert misa.lib.misa_last_error() != b""
    for kw in (dict(d=64), dict(H=128, h=8), dict(L=1 << 20),
               dict(n_seq=70000)):
        assert _pool(misa, _prob(misa, **kw)) == UNSUPPORTED, kw
    assert misa.lib.misa_pool_keys(None, FAKE, None, FAKE, None, 0, None) == INVALID


def test_null_and_misaligned_pointers(misa):
    p = _prob(misa)
    assert _pool(misa, p, K=None) == 1
    assert _pool(misa, p, Kp=None) == 1
    assert _pool(misa, p, K=ctypes.c_void_p(0x1008)) == 1
    assert b"aligned" in misa.lib.misa_last_error()
    assert _pool(misa, _prob(misa, k_dtype=misa.FP8_E4M3), kscale=None) == 1     # fp8 needs scales
    pc = ctypes.byref(p.c())
    assert misa.lib.misa_score_tokens(pc, None, FAKE, None, FAKE, None, FAKE, None, 0, None) == 1
    assert misa.lib.misa_score_tokens(pc, FAKE, FAKE, None, FAKE, None, None, None, 0, None) == 1
    assert misa.lib.misa_topk(pc, FAKE, 0, FAKE, None, None, 0, None) == 1          # k < 1
    assert misa.lib.misa_topk(pc, FAKE, 20000, FAKE, None, None, 0, None) == 2      # k too large
    assert misa.lib.misa_topk(pc, None, 8, FAKE, None, None, 0, None) == 1
    assert misa.lib.misa_rerank(pc, FAKE, FAKE, FAKE, None, FAKE, 4, 8, FAKE, None, FAKE, 1 << 20, None) == 1  # k > k_cand
    assert misa.lib.misa_rerank(pc, FAKE, FAKE, FAKE, None, None, 8, 4, FAKE, None, FAKE, 1 << 20, None) == 1


def test_workspace_contract(misa):
    p = _prob(misa)
    pc = ctypes.byref(p.c())
    need = misa.workspace_bytes(p, misa.OP_ROUTE)
    assert need > 0 and need % 256 == 0
    assert misa.workspace_bytes(p, misa.OP_POOL) == 0
    assert misa.workspace_bytes(p, misa.OP_RERANK, 512) == 2 * 1 * 512 * 4
    assert misa.workspace_bytes(p, 9) == 0
    args = (pc, FAKE, FAKE, FAKE, FAKE, None, FAKE, None)
    assert misa.lib.misa_route_heads(*args, None, 0, None) == 3                      # NULL workspace
    assert misa.lib.misa_route_heads(*args, FAKE, need - 1, None) == 3               # too small
    assert b"too small" in misa.lib.misa_last_error()
    assert misa.lib.misa_route_heads(*args, ctypes.c_void_p(0x1010), need, None) == 3   # misaligned
    assert misa.lib.misa_rerank(pc, FAKE, FAKE, FAKE, None, FAKE, 512, 64, FAKE, None, FAKE, 100, None) == 3


def test_binding_refuses_host_tensors(misa):
    import torch
    p = _prob(misa)
    with pytest.raises(ValueError):
        misa.pool_keys(p, torch.zeros(4), None, torch.zeros(4))


def test_page_table_and_probe_arguments(misa):
    INVALID = 1
    base = _prob(misa).c()

    def paged(**kw):
        c = _prob(misa).c()
        c.page_table, c.page_size, c.max_pages = 0x2000, 64, 16          # 16 pages of 64 cover L = 1000
        for k, v in kw.items():
            setattr(c, k, v)
        return misa.lib.misa_pool_keys(ctypes.byref(c), FAKE, None, FAKE, None, 0, None)

    for kw in (dict(page_size=48), dict(page_size=8), dict(page_size=1 << 17), dict(max_pages=15),
               dict(page_table=None)):                                    # sizes without a table
        assert paged(**kw) == INVALID, kw
    assert b"page" in misa.lib.misa_last_error()
    assert base.page_table is None and base.page_size == 0 and base.max_pages == 0
    # probes: argument checks come before any launch
    assert misa.lib.misa_probe_hbm_read(None, 8192, FAKE, None) == INVALID
    assert misa.lib.misa_probe_hbm_read(FAKE, 8192, None, None) == INVALID
    assert misa.lib.misa_probe_hbm_read(FAKE, 1000, FAKE, None) == INVALID          # not a multiple of 8192
    assert misa.lib.misa_probe_hbm_read(ctypes.c_void_p(0x1004), 8192, FAKE, None) == INVALID
    assert misa.lib.misa_probe_mfma_bf16(0, 1, FAKE, None, None) == INVALID
    assert misa.lib.misa_probe_mfma_bf16(1, 0, FAKE, None, None) == INVALID
    assert misa.lib.misa_probe_mfma_bf16(1, 1, None, None, None) == INVALID
    assert misa.lib.misa_probe_mfma_bf16_operands(1, 1, None, FAKE, None, None) == INVALID
    assert misa.lib.misa_probe_mfma_bf16_operands(1, 1, ctypes.c_void_p(0x1008), FAKE, None, None) == INVALID
    assert misa.lib.misa_probe_mfma_bf16_operands(0, 1, FAKE, FAKE, None, None) == INVALID


def test_paginate_places_every_key_where_the_page_table_says(misa):
    import torch
    L, P, n_seq = 150, 16, 3
    K = torch.arange(n_seq * L * 128, dtype=torch.float32).view(n_seq, L, 128)
    ks = torch.arange(n_seq * L, dtype=torch.float32).view(n_seq, L)
    p = misa.Problem(n_seq, L, 1, 8, 16, 2, misa.F32, misa.F32)
    # (the binding only checks devices when a call is made; the layout helper works on any device)
    pg = misa.paginate({"K": K, "kscale": ks, "problem": p}, P, seed=5)
    table, pool, spool = pg["problem"].page_table, pg["K"], pg["kscale"]
    assert table.shape == (n_seq, -(-L // P)) and pg["problem"].page_size == P
    assert len(set(table.view(-1).tolist())) == table.numel()            # pages are not shared
    for i in range(n_seq):
        for s in (0, 1, 15, 16, 17, 100, L - 1):
            row = int(table[i, s // P]) * P + s % P
            assert torch.equal(pool.view(-1, 128)[row], K[i, s])
            assert spool.view(-1)[row] == ks[i, s]


def test_route_heads_static_rejects_problems_beyond_its_scratch_array(misa):
    # 300 decode sequences need 300 x 64 x 64 floats of partial sums: more than the 4 MiB array
    p = _prob(misa, n_seq=300)
    assert misa.workspace_bytes(p, misa.OP_ROUTE) > misa.ROUTE_STATIC_SCRATCH_BYTES
    st = misa.lib.misa_route_heads_static(ctypes.byref(p.c()), FAKE, FAKE, FAKE, FAKE, None, FAKE, None, None)
    assert st == 2 and b"scratch" in misa.lib.misa_last_error()
    # argument validation comes first, as in misa_route_heads
    assert misa.lib.misa_route_heads_static(ctypes.byref(_prob(misa).c()), None, FAKE, FAKE, FAKE, None, FAKE,
                                            None, None) == 1


def test_binding_without_the_raw_stream_handle_of_torch(misa, monkeypatch):
    """torch's raw stream handle is not part of its public interface: a torch without it takes the public one."""
    import importlib.util
    import sys
    import types

    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0x1230))
    spec = importlib.util.spec_from_file_location("misa_without_raw_stream", misa.__file__)
    m = importlib.util.module_from_spec(spec)
    monkeypatch.setitem(sys.modules, spec.name, m)
    spec.loader.exec_module(m)
    assert m._stream() == 0x1230
