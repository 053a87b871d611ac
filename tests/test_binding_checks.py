"""The binding's argument checks (CPU): what every entry point runs on each
tensor before its C call, so a wrong dtype, shape, layout or device raises
ValueError instead of reaching a kernel."""
import types

import pytest
import torch

from paper_2512_22492_amd import binding as B


def test_check_tensor_accepts_matching_tensors():
    t = torch.empty((4, 8, 128), dtype=torch.bfloat16)
    B._check_tensor("t", t, dtype=torch.bfloat16, shape=(4, 8, 128), device=t.device)
    B._check_tensor("t", t, dtype=(torch.uint8, torch.bfloat16), shape=(None, 8, None))
    B._check_tensor("t", t, ndim=3)
    B._check_tensor("t", t[:, :4], contiguous=False, shape=(4, 4, 128))


@pytest.mark.parametrize("kw", [
    dict(dtype=torch.float32),
    dict(dtype=(torch.uint8, torch.int32)),
    dict(shape=(4, 8, 64)),
    dict(shape=(4, 8)),
    dict(shape=(4, 8, 128, 1)),
    dict(shape=(None, 4, None)),
    dict(ndim=2),
    dict(device=torch.device("meta")),
])
def test_check_tensor_rejects(kw):
    t = torch.empty((4, 8, 128), dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        B._check_tensor("t", t, **kw)


def test_check_tensor_rejects_non_tensors_and_strided_views():
    t = torch.empty((4, 8, 128), dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        B._check_tensor("t", [1, 2, 3])
    with pytest.raises(ValueError):
        B._check_tensor("t", t[:, ::2], shape=(4, 4, 128))


def test_check_table_and_pools():
    bt = torch.zeros((3, 5), dtype=torch.int32)
    sl = torch.ones(3, dtype=torch.int32)
    B._check_table(bt, sl, 3, bt.device)
    for args in [(bt.long(), sl, 3), (bt, sl.long(), 3), (bt, sl, 2), (bt[:, ::2], sl, 3),
                 (bt, sl[:2], 3)]:
        with pytest.raises(ValueError):
            B._check_table(*args, bt.device)
    k = torch.empty((6, 2, 16, 128), dtype=torch.bfloat16)
    v = torch.empty_like(k)
    kw = dict(kv_dtype=B.RL_DA_KV_BF16, layout=B.RL_DA_LAYOUT_HND, num_kv_heads=2,
              head_dim=128, page_size=16, device=k.device)
    assert B._check_pools(k, v, None, None, **kw) == 6
    with pytest.raises(ValueError):
        B._check_pools(k, v[:5], None, None, **kw)
    with pytest.raises(ValueError):
        B._check_pools(k, v, torch.ones((6, 2)), torch.ones((6, 2)), **kw)
    with pytest.raises(ValueError):          # token-major pools checked as head-major
        B._check_pools(k.transpose(1, 2).contiguous(), v.transpose(1, 2).contiguous(),
                       None, None, **kw)
    k8 = torch.empty((6, 2, 16, 128), dtype=torch.uint8)
    kw8 = dict(kw, kv_dtype=B.RL_DA_KV_FP8_E4M3)
    assert B._check_pools(k8, k8.clone(), torch.ones((6, 2)), torch.ones((6, 2)), **kw8) == 6
    with pytest.raises(ValueError):
        B._check_pools(k8, k8.clone(), None, None, **kw8)
    with pytest.raises(ValueError):
        B._check_pools(k8, k8.clone(), torch.ones((6, 3)), torch.ones((6, 2)), **kw8)


def test_extend_divides_only_with_the_callers_workspace(monkeypatch):
    """extend_attention brings no workspace of its own, whatever the launch's size
    and table: what a sequence's rows are does not depend on the batch, the call
    allocates nothing, and the caller's workspace goes through with its size."""
    seen = []
    monkeypatch.setattr(B, "rl_extend_attn_ws",
                        lambda *a: seen.append((a[-3], a[-2])) or B.RL_DA_OK)

    def call(batch, pages, new, workspace=None):
        pool = torch.zeros((8, 2, 16, 128), dtype=torch.bfloat16)
        p = types.SimpleNamespace(
            kv_dtype="bf16", layout="hnd", num_q_heads=8, num_kv_heads=2, head_dim=128,
            page_size=16, batch=batch, num_pages=8, max_pages=pages, scale=1.0, k_pool=pool,
            v_pool=pool.clone(), k_scale=None, v_scale=None,
            block_table=torch.zeros((batch, pages), dtype=torch.int32),
            seq_lens=torch.ones(batch, dtype=torch.int32))
        q = torch.zeros((batch * new, 8, 128), dtype=torch.bfloat16)
        start = torch.arange(batch + 1, dtype=torch.int32) * new
        B.extend_attention(p, q, start, new, torch.empty_like(q), None, workspace)
        return seen.pop()

    for batch, pages, new in ((1, 4096, 3), (1, 4, 3), (300, 4096, 1), (2, 4096, 300)):
        assert call(batch, pages, new) == (None, 0)
    ws = torch.zeros(1 << 20, dtype=torch.uint8)
    assert call(1, 4096, 3, ws) == (ws, 1 << 20)
    for bad in (ws.view(torch.int32), ws[::2], ws.view(2, -1), 7):
        with pytest.raises(ValueError):
            call(1, 4096, 3, bad)
