"""Decode steps of few short heads (one workgroup per head, planned while it
streams): heads with no, one and many tiles, tiles the append starts, every
page size and group, popped pages, capacity and pool errors.  State bit-exact,
outputs within the decode tolerance (tests/dms_testlib.py)."""
import numpy as np
import pytest

from dms_testlib import SeqInputs, compare_state, to_dev
from test_decode_parity import _append_chunks, _decode_steps, _mk, _oracle_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,P,g,w,H,starts,p", [
    (64, 32, 1, 1, 1, (0,), 0.5), (128, 64, 6, 16, 2, (31, 0), 0.5), (128, 256, 16, 40, 1, (1990,), 0.0),
    (64, 128, 5, 7, 3, (500, 95, 63), 0.75), (128, 32, 7, 300, 4, (352, 351), 0.875),
    (64, 64, 2, 16, 64, (40, 33, 64, 1), 0.5)])       # 256 heads: one per compute unit
def test_steps(D, P, g, w, H, starts, p):
    steps = 6
    maxp = 2048 // P
    n = len(starts)
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=n, num_kv_heads=H, group_size=g, head_dim=D, window=w,
                               page_size=P, num_pages=H * sum(-(-(s + steps) // P) for s in starts),
                               max_pages_per_head=maxp, max_chunk_tokens=max(1, sum(starts))))
    orc = _oracle_for(cfg)
    seqs = list(range(n))
    inputs = {s: SeqInputs(11, 0, s, starts[s] + steps, H, g, D, p) for s in seqs}
    if any(starts):
        _append_chunks(dms, cache, orc, seqs, inputs, {s: 0 for s in seqs}, dict(enumerate(starts)), max(starts))
    _decode_steps(dms, cache, orc, seqs, inputs, dict(enumerate(starts)), steps, g)
    cache.close()


@pytest.mark.parametrize("P,L,pages,maxp,err", [
    (32, 32, 1, 4, "DMS_ERR_OUT_OF_PAGES"), (32, 32, 8, 1, "DMS_ERR_CAPACITY"),
    # longer page tables: the launch that plans in every workgroup
    (32, 32, 1, 65, "DMS_ERR_OUT_OF_PAGES"), (256, 2304, 10, 9, "DMS_ERR_CAPACITY")])
def test_refused_step_changes_nothing(P, L, pages, maxp, err):
    import torch
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=2, num_kv_heads=1, group_size=2, head_dim=64, window=64,
                               page_size=P, num_pages=pages, max_pages_per_head=maxp, max_chunk_tokens=L))
    orc = _oracle_for(cfg)
    inputs = {0: SeqInputs(12, 0, 0, L + 1, 1, 2, 64, 0.0)}
    _append_chunks(dms, cache, orc, [0], inputs, {0: 0}, {0: L}, L)
    x = inputs[0]
    out = torch.full((2, 2, 64), 7.0, device="cuda")

    def step(*ids):
        rep = [np.repeat(a[L][None], len(ids), 0) for a in (x.q, x.k, x.v, x.flags)]
        dms.dms_decode_step(cache.ctx, 0, len(ids), to_dev(np.array(ids, np.int32)), *map(to_dev, rep), out[:len(ids)])
        return dms.dms_status(cache.ctx)

    for _ in range(2):   # the second call finds the sticky status
        assert step(0) == getattr(dms, err)
    for ids in ((5,), (-1,), (1, 1), (0, 2)):
        dms.dms_clear_status(cache.ctx)
        assert step(*ids) == dms.DMS_ERR_BAD_SEQ
    assert bool((out == 7.0).all())
    compare_state(cache.export(0), orc, [0, 1])
    cache.close()


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("H,g,D,L,maxp", [
    (2, 6, 128, 1270, 32), (8, 5, 128, 2000, 32),     # one workgroup of eleven streams per head
    (2, 6, 128, 370, 64), (4, 7, 64, 250, 64),        # longer page tables: one workgroup of four
    (2, 6, 128, 1270, 64)])                           # four workgroups per head
def test_step_is_as_precise_as_one_wave_per_tile(H, g, D, L, maxp, fp8):
    """The weights are rounded to bf16 against a reference; a head's tiles on waves of their own (dms_decode
    over many waves: each tile's largest weight is exactly 1) are as near to 64-bit sums as it gets.  A step
    that walks several tiles a wave must not be further off."""
    import torch
    from paper_2506_05345_amd import dms
    n, w = 8, 1
    cfg = dms.make_config(1, n, H, g, D, w, 64, n * H * (-(-(L + 1) // 64)), maxp, n * L,
                          kv_format=dms.DMS_KV_FP8 if fp8 else dms.DMS_KV_BF16)
    gen = torch.Generator("cuda").manual_seed(17)
    k, v = (torch.randn((n, L + 1, H, D), generator=gen, device="cuda").bfloat16() for _ in range(2))
    q = torch.randn((n, H * g, D), generator=gen, device="cuda").bfloat16()
    if fp8:   # rows that FP8 pages hold exactly
        k, v = (torch.cat([x.float().clamp(-1.75, 1.75).mul(4).round().div(4)[..., :-1],
                           torch.full_like(x[..., :1], 1.75).float()], -1).bfloat16() for x in (k, v))
    cache = dms.DmsCache(cfg)
    sid = torch.arange(n, dtype=torch.int32, device="cuda")
    cu = (torch.arange(n + 1, device="cuda") * L).to(torch.int32)
    z = lambda *s: torch.zeros(s, dtype=torch.uint8, device="cuda")  # noqa: E731
    dms.dms_append_chunk(cache.ctx, 0, n, sid, cu, n * L, L, k[:, :L].reshape(n * L, H, D),
                         v[:, :L].reshape(n * L, H, D), z(n * L, H))
    out = [torch.empty((n, H * g, D), device="cuda") for _ in range(2)]
    dms.dms_decode_step(cache.ctx, 0, n, sid, q, k[:, L].contiguous(), v[:, L].contiguous(), z(n, H), out[0])
    dms.dms_decode(cache.ctx, 0, n, sid, q, out[1])
    assert dms.dms_status(cache.ctx) == 0
    s = torch.einsum("nhgd,nthd->nhgt", q.double().view(n, H, g, D), k.double()) / D ** 0.5
    ref = torch.einsum("nhgt,nthd->nhgd", s.softmax(-1), v.double()).reshape(n, H * g, D)
    err = [float((o.double() - ref).norm() / ref.norm()) for o in out]
    print(err)
    assert err[0] <= 1.01 * err[1], err
    cache.close()
