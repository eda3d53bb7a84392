"""Chunk commits where their passes' rounds end: 16 residue classes per block,
64 members of a class per round, 4096 tokens per scan round; sequence release
with more heads than waves.  Bookkeeping and stored rows are bit-exact."""
import numpy as np
import pytest

from dms_testlib import SeqInputs, compare_pool, compare_state, to_dev
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
