"""Training attention where its tilings end: query tiles of 32, staged pairs
of 64 keys, key blocks of 128, key-major passes split over several workgroups,
and inputs that are views at odd addresses.  Same oracle and bounds as
tests/test_train_parity.py (bf16 weights and score gradients: 2^-9 each)."""
import numpy as np
import pytest

from test_kernel_asm import test_m0_is_only_the_lds_copy_destination as _m0_check
from test_train_parity import D, GRAD_TOL, _bf16, _dev_bf16, _run


def test_m0_is_only_the_lds_copy_destination_in_training(tmp_path):
    _m0_check(tmp_path, "dms_train.hip")


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,H,g,w,seed", [
    (1, 31, 1, 2, 5, 20), (1, 32, 2, 1, 32, 21), (1, 65, 1, 6, 33, 22), (2, 127, 1, 1, 64, 23),
    (1, 128, 2, 6, 31, 24), (1, 129, 1, 5, 128, 25), (1, 353, 2, 3, 96, 26), (1, 416, 1, 16, 1000, 27)])
def test_tile_edges(B, T, H, g, w, seed):
    r = _run(B, T, H, g, w, seed)
    assert r["out"] <= 1e-2 and r["lse"] <= 5e-3, r
    for name in ("dq", "dk", "dv", "dalpha"):
        assert r[name] <= GRAD_TOL, (name, r)


def _inputs(B, T, H, g, seed):
    import torch
    rng = np.random.default_rng(seed)
    shapes = {"q": (B, T, H * g, D), "k": (B, T, H, D), "v": (B, T, H, D), "dout": (B, T, H * g, D)}
    x = {n: _dev_bf16(_bf16(rng.normal(size=s))) for n, s in shapes.items()}
    x["alpha"] = torch.from_numpy(rng.uniform(0, 1, (B, T, H)).astype(np.float32)).cuda()
    return x


def _fwd_bwd(x, w):
    """(out, lse, dq, dk, dv, dalpha) of one forward and backward call."""
    import torch
    from paper_2506_05345_amd import dms
    B, T, H, _ = x["k"].shape
    cfg = dms.make_train_config(B, T, H, x["q"].shape[2] // H, D, w)
    ws = torch.empty(dms.dms_train_workspace(cfg), dtype=torch.uint8, device="cuda")
    out = torch.empty(x["q"].shape, device="cuda")
    lse = torch.empty((B, x["q"].shape[2], T), device="cuda")
    grads = [torch.empty(x[n].shape, device="cuda") for n in ("q", "k", "v", "alpha")]
    dms.dms_train_attention_fwd(cfg, x["q"], x["k"], x["v"], x["alpha"], out, lse, ws)
    dms.dms_train_attention_bwd(cfg, x["q"], x["k"], x["v"], x["alpha"], out, lse, x["dout"], *grads, ws)
    torch.cuda.synchronize()
    return [out, lse, *grads]


@pytest.mark.gpu
@pytest.mark.parametrize("name,at", [("v", 40), ("k", 40), ("v", 101), ("k", 101)])
def test_later_rows_stay_out_of_earlier_blocks(name, at):
    """Blocks of 32 positions (four query heads) that end on an odd tile: a non-finite row of the tile
    after their last one leaves them as they are, bit for bit."""
    T, first = 128, at // 32 * 32
    x = _inputs(1, T, 2, 4, 31)
    clean = _fwd_bwd(x, 16)
    x[name] = x[name].clone()
    x[name][0, at] = float("inf") if name == "v" else float("nan")
    got = _fwd_bwd(x, 16)
    for i, ax in ((0, 1), (1, 2), (2, 1)):   # out, lse, dq
        assert got[i].narrow(ax, 0, first).equal(clean[i].narrow(ax, 0, first)), i


@pytest.mark.gpu
def test_infinite_last_row_stays_infinite():
    """The rows that fill the last tile add nothing, not a NaN from a repeated infinity."""
    import torch
    T = 50
    x = _inputs(1, T, 1, 4, 32)
    x["v"][0, T - 1] = float("inf")
    assert bool(torch.isposinf(_fwd_bwd(x, 16)[0][0, T - 1]).all())
    x = _inputs(1, T, 1, 4, 32)
    x["dout"][0, T - 1] = float("inf")
    assert bool(torch.isposinf(_fwd_bwd(x, 16)[4][0, T - 1]).all())


@pytest.mark.gpu
def test_evicted_key_takes_nothing_from_old_queries():
    """alpha = 1 on a key whose scores lie about 84 above the log-sum-exp of every query past its window:
    exp(s - lse) is finite in float32, its products with dout (dV) and q (dK) are not.  The key's dK and dV
    are those of the queries in its window alone."""
    import oracle
    T, w, j = 256, 8, 20
    x = _inputs(1, T, 1, 1, 33)
    for n in ("q", "k", "v", "dout"):
        x[n] = x[n].float().mul_(0.01).bfloat16()
    x["alpha"].fill_(0.25)
    x["alpha"][0, j] = 1.0
    x["q"][..., 0] = 32.0
    x["k"][..., 0] = 0.0
    x["k"][0, j, 0, 0] = 31.5      # scaled score 32 * 31.5 / sqrt(128) = 89.1
    x["dout"].fill_(0.0)
    x["dout"][0, :, 0, 1:9] = 16384.0   # into dV only: no value has these dims
    x["dout"][0, :, 0, 10] = 1.0        # sum dout out = 1: dS = -exp(s - lse)
    x["v"][..., 1:9] = 0.0
    x["v"][..., 10] = 1.0
    x["v"][0, j, 0] = 0.0
    got = [t.cpu().numpy() for t in _fwd_bwd(x, w)]
    f = [x[n].float().cpu().numpy() for n in ("q", "k", "v")]
    al, do = x["alpha"].cpu().numpy().astype(np.float64), x["dout"].float().cpu().numpy()
    lse = oracle.train_attention(*f, al, w, 1)[1][0, 0, j + w:]
    p = 32 * 31.5 / np.sqrt(D) - lse
    assert p.min() > 82 and p.max() < 88, (p.min(), p.max())   # exp below 3.4e38, times 16384 above
    gq, gk, gv, _ = oracle.train_attention_grads(*f, al, do, w, 1)
    for name, a, ref in (("dq", got[2], gq), ("dk", got[3], gk), ("dv", got[4], gv)):
        assert np.isfinite(a).all(), name
        assert np.abs(a - ref).max() <= GRAD_TOL * max(1.0, np.abs(ref).max()), name


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,g", [(150, 2, 3), (97, 1, 6), (200, 1, 16), (64, 2, 2)])
def test_unaligned_views_give_the_same_bits(T, H, g):
    """Also where the copies of the inputs leave room for fewer sums than the key-major pass has splits."""
    import torch
    w = 40
    x = _inputs(1, T, H, g, 30)

    def shifted(t):
        buf = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
        v = buf[1:1 + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16
        return v

    y = {n: shifted(t) if n != "alpha" else t for n, t in x.items()}
    for a, b in zip(_fwd_bwd(x, w), _fwd_bwd(y, w)):
        assert torch.equal(a, b)
