"""Chunked prefill where the attention pass's units end: 32-row tiles and
64-row stages of the cache, the kept keys and the band; one position more than
a workgroup holds; sequences with nothing in the call; more rows than the
ranking pass orders.  Outputs against dense masked attention."""
import pytest

from test_mla_parity import _prefill_run
from test_prefill_parity import _run

pytestmark = pytest.mark.gpu


def _tiles(d, g, w, lens, chunks, H=1, page=32, **kw):
    n, longest = len(lens), max(lens)
    per = -(-longest // page) + 1
    _run(dict(num_layers=1, max_seqs=n, num_kv_heads=H, group_size=g, head_dim=d, window=w, page_size=page,
              num_pages=n * H * per, max_pages_per_head=per, max_chunk_tokens=n * max(chunks)),
         list(range(n)), dict(enumerate(lens)), chunks, 91, 0.5, nan_pools=True, **kw)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g,w,lens,chunks", [
    (1, 1, (1, 31, 33), [1, 32]),                    # one key; a tile and one key
    (4, 64, (64, 97, 161, 130), [64, 33]),           # whole and half stages; finished sequences
    (3, 40, (86, 85, 170), [43, 42, 85]),            # 128 / 3 = 42 positions, 256 / 3 = 85 per workgroup
    (16, 200, (300, 9), [9, 17, 256])])              # window longer than the chunk, straddling stages
def test_edges(fp8, d, g, w, lens, chunks):
    _tiles(d, g, w, lens, chunks, H=2, fp8=fp8)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [5, 33, 70])    # one, two and three tiles
def test_infinite_value_stays_infinite(d, T):
    """Stages hold two tiles; where the second does not exist it adds nothing: an infinite value row seen by
    the last position only makes its output infinite, not NaN, and leaves earlier tiles' positions alone."""
    import torch
    from paper_2506_05345_amd import dms
    H, g, w = 2, 4, 16
    cfg = dms.make_config(1, 1, H, g, d, w, 32, H * 4, 4, T)
    gen = torch.Generator("cuda").manual_seed(5)
    q, k, v = (torch.randn((T, n, d), generator=gen, device="cuda").bfloat16() for n in (H * g, H, H))
    flags = (torch.rand((T, H), generator=gen, device="cuda") < 0.5).to(torch.uint8)
    sid, cu = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.tensor([0, T], dtype=torch.int32, device="cuda")
    outs = []
    for last in (None, float("inf")):
        if last is not None:
            v[T - 1] = last
        cache = dms.DmsCache(cfg)
        out = torch.empty((T, H * g, d), device="cuda")
        dms.dms_prefill_chunk(cache.ctx, 0, 1, sid, cu, T, T, q, k, v, flags, out)
        torch.cuda.synchronize()
        assert dms.dms_status(cache.ctx) == 0
        cache.close()
        outs.append(out)
    assert bool(torch.isposinf(outs[1][T - 1]).all())
    # a workgroup takes 32 positions of 4 heads; the tiles of all but the last end before the row
    before = (T - 1) // 32 * 32
    assert outs[1][:before].equal(outs[0][:before])


@pytest.mark.parametrize("n", [32, 33])   # 512 rows are ranked, 528 are taken in call order
def test_many_rows(n):
    _tiles(64, 2, 8, [5 + (s * 13) % 60 for s in range(n)], [40, 9], H=16)


@pytest.mark.parametrize("g,w,lens,chunks", [
    (1, 1, (1, 31, 33), [1, 32]),            # 128 positions per workgroup
    (16, 64, (64, 97, 130), [64, 33]),
    (43, 40, (66, 33), [32, 33]),            # two positions and 42 unused columns
    (128, 33, (65, 2), [32, 1, 32])])        # a position per workgroup
def test_latent_edges(g, w, lens, chunks):
    _prefill_run(g, list(range(len(lens))), dict(enumerate(lens)), chunks, 93, 0.5, w, 32, nan_fill=True)


def test_latent_many_rows():
    """513 sequences, taken in call order; the last one has nothing in the second call."""
    lens = {s: 6 + s % 4 for s in range(512)}
    lens[512] = 3
    _prefill_run(2, sorted(lens), lens, [5], 95, 0.5, 2, 32, nan_fill=True)
