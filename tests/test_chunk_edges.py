"""Chunk commits where their passes' rounds end: 1 to 16 residue classes per
block (fewer for fewer heads), 1024 tokens of them per round, 4096 tokens per
scan round; sequence release with more heads than lane groups.  Bookkeeping and
stored rows are bit-exact."""
import numpy as np
import pytest

from dms_testlib import SeqInputs, bf16_to_f32, compare_pool, compare_state, to_dev
from test_decode_parity import _append_chunks, _mk, _oracle_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,lens,chunk,H", [
    (1, (130,), 65, 1),              # one class, more members than a round
    (15, (200, 31), 97, 2), (16, (1100, 16), 1060, 2), (17, (140, 1), 140, 3),
    (300, (250, 90), 250, 2),        # window longer than the chunk
    (40, (4200,), 4097, 1)])         # a scan round and one token
def test_chunk_then_release(w, lens, chunk, H):
    import torch
    maxp = -(-max(lens) // 32) + 1
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=len(lens), num_kv_heads=H, group_size=1, head_dim=64,
                               window=w, page_size=32, num_pages=H * len(lens) * maxp, max_pages_per_head=maxp,
                               max_chunk_tokens=chunk * len(lens)))
    orc = _oracle_for(cfg)
    seqs = list(range(len(lens)))
    inputs = {s: SeqInputs(7, 0, s, n, H, 1, 64, 0.5) for s, n in zip(seqs, lens)}
    for _ in range(2):   # the second time on released pages
        _append_chunks(dms, cache, orc, seqs, inputs, {s: 0 for s in seqs}, dict(zip(seqs, lens)), chunk)
        view = cache.export(0)
        compare_state(view, orc, seqs)
        compare_pool(cache, 0, view, seqs, inputs)
        dms.dms_seq_reset(cache.ctx, 0, len(seqs), to_dev(np.array(seqs, np.int32)))
        orc.seq_reset(seqs)
        compare_state(cache.export(0), orc, seqs)
    cache.close()


@pytest.mark.parametrize("w,lens,chunk,H", [
    (1, (1100,), 1100, 1),           # one class a block, more members than a round
    (70, (150,) * 8, 150, 2),        # four classes a block, the last one short
    (40, (90,) * 16, 90, 8),         # sixteen
    (9, (35,) * 12, 35, 2)])         # release: half a wave per head
def test_classes_per_block(w, lens, chunk, H):
    test_chunk_then_release(w, lens, chunk, H)


def test_release_of_many_heads():
    H, n = 24, 45   # more heads than a round of 1024 threads
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=n, num_kv_heads=H, group_size=1, head_dim=64, window=4,
                               page_size=32, num_pages=H * n * 2, max_pages_per_head=2, max_chunk_tokens=n * 40))
    orc = _oracle_for(cfg)
    seqs = list(range(n))
    lens = {s: 1 + (s * 7) % 40 for s in seqs}
    inputs = {s: SeqInputs(8, 0, s, lens[s], H, 1, 64, 0.25) for s in seqs}
    _append_chunks(dms, cache, orc, seqs, inputs, {s: 0 for s in seqs}, lens, 40)
    gone = [s for s in seqs if s != 3]
    dms.dms_seq_reset(cache.ctx, 0, len(gone), to_dev(np.array(gone, np.int32)))
    orc.seq_reset(gone)
    compare_state(cache.export(0), orc, seqs)
    cache.close()


def test_refused_prefill_leaves_no_error_behind():
    """A prefill refused for its boundaries, some of whose heads are also over
    capacity, must not make the next call fail."""
    import torch
    H, n = 2, 2
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=n, num_kv_heads=H, group_size=1, head_dim=64, window=8,
                               page_size=32, num_pages=8, max_pages_per_head=1, max_chunk_tokens=128))
    sid = to_dev(np.arange(n, dtype=np.int32))

    def prefill(cu, total, longest):
        x = torch.zeros((total, H, 64), dtype=torch.bfloat16, device="cuda")
        f = torch.zeros((total, H), dtype=torch.uint8, device="cuda")
        out = torch.empty((total, H, 64), device="cuda")
        dms.dms_prefill_chunk(cache.ctx, 0, n, sid, to_dev(np.array(cu, np.int32)), total, longest, x, x, x, f, out)
        torch.cuda.synchronize()
        return dms.dms_status(cache.ctx)

    # sequence 0 needs more slots than a head has, sequence 1 is longer than announced
    assert prefill([0, 40, 100], 100, 50) == dms.DMS_ERR_INVALID
    dms.dms_clear_status(cache.ctx)
    assert prefill([0, 20, 50], 50, 30) == 0
    assert cache.export(0).pos.tolist() == [20, 30]
    cache.close()


@pytest.mark.parametrize("left", [-5, -1, 0x7FFFFFFF])
def test_chunk_calls_read_nothing_left_in_the_workspace(left):
    """Whatever an interrupted call left in the scratch of the chunk passes (an error code among it), the
    next append or prefill is planned from its own tokens alone."""
    import torch
    H, n, T = 2, 2, 40
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=n, num_kv_heads=H, group_size=1, head_dim=64, window=8,
                               page_size=32, num_pages=16, max_pages_per_head=4, max_chunk_tokens=n * T))
    orc = _oracle_for(cfg)
    inputs = {s: SeqInputs(9, 0, s, 2 * T, H, 1, 64, 0.5) for s in range(n)}
    cache.workspace.view(torch.int32).fill_(left)
    _append_chunks(dms, cache, orc, [0, 1], inputs, {0: 0, 1: 0}, {0: T, 1: T}, T)
    compare_state(cache.export(0), orc, [0, 1])
    cache.workspace.view(torch.int32).fill_(left)
    sid, cu = to_dev(np.arange(n, dtype=np.int32)), to_dev(np.array([0, T, 2 * T], np.int32))
    x = [to_dev(np.concatenate([getattr(inputs[s], a)[T:] for s in range(n)])) for a in ("q", "k", "v", "flags")]
    out = torch.full((n * T, H, 64), float("nan"), device="cuda")
    dms.dms_prefill_chunk(cache.ctx, 0, n, sid, cu, n * T, T, *x, out)
    assert dms.dms_status(cache.ctx) == 0 and bool(torch.isfinite(out).all())
    orc.append_chunk([0, 1], [inputs[s].flags[T:] for s in range(n)],
                     [bf16_to_f32(inputs[s].k[T:]) for s in range(n)], [bf16_to_f32(inputs[s].v[T:]) for s in range(n)])
    compare_state(cache.export(0), orc, [0, 1])
    cache.close()


def test_refused_chunks_name_their_error():
    """Boundaries that disagree, too many tokens for a head's pages and an empty pool, each refused with its
    own error, nothing changed, and a valid call right after."""
    import torch
    dms, cfg, cache = _mk(dict(num_layers=1, max_seqs=2, num_kv_heads=1, group_size=1, head_dim=64, window=8,
                               page_size=32, num_pages=3, max_pages_per_head=2, max_chunk_tokens=200))

    def append(ids, cu):
        x = torch.zeros((cu[-1], 1, 64), dtype=torch.bfloat16, device="cuda")
        f = torch.zeros((cu[-1], 1), dtype=torch.uint8, device="cuda")
        n = len(ids)
        dms.dms_append_chunk(cache.ctx, 0, n, to_dev(np.array(ids, np.int32)), to_dev(np.array(cu, np.int32)),
                             cu[-1], max(b - a for a, b in zip(cu, cu[1:])) if n < 2 or cu[1] != 70 else 60, x, x, f)
        rc = dms.dms_status(cache.ctx)
        dms.dms_clear_status(cache.ctx)
        return rc

    assert append([0, 1], [0, 70, 140]) == dms.DMS_ERR_INVALID    # longer than announced; also over capacity
    assert append([0], [0, 65]) == dms.DMS_ERR_CAPACITY
    assert append([0, 1], [0, 40, 80]) == dms.DMS_ERR_OUT_OF_PAGES
    assert cache.export(0).pos.tolist() == [0, 0] and cache.export(0).top == 3
    assert append([0, 1], [0, 40, 60]) == dms.DMS_OK
    assert cache.export(0).pos.tolist() == [40, 20]
    cache.close()
