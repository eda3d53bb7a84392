"""Latent decode over units of a few tiles: segments shorter and longer than
the tiles in flight, several heads per unit, the new token in a segment's
first, middle and last tile, stale rows as NaNs; one block of query heads and
a second, partial one."""
import pytest

from dms_testlib import compare_state
from test_mla_parity import MlaInputs, _append_chunks, _decode_steps, _mk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [16, 72])
def test_short_segments(g):
    import torch
    n, P = 300, 32   # ~1000 tiles over 256 units
    lens = {s: 1 + (s * 37) % 190 for s in range(n)}
    dms, cfg, cache, orc = _mk(n, g, 16, P, num_pages=n * 7, maxp=7, max_chunk=n * 32)
    for p in cache.pools:
        p.fill_(0xFF)
    cache.workspace.fill_(0xFF)
    dms.dms_init_state(cache.ctx)
    torch.cuda.synchronize()
    inp = {s: MlaInputs(61, s, lens[s] + 2, g, 0.1) for s in range(n)}
    seqs = sorted(lens)
    _append_chunks(dms, cache, orc, seqs, inp, {s: 0 for s in seqs}, lens, 32)
    compare_state(cache.export(0), orc, seqs)
    _decode_steps(dms, cache, orc, seqs, inp, lens, 2, g)
    cache.close()
