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


@pytest.mark.gpu
def test_unaligned_views_give_the_same_bits():
    import torch
    from paper_2506_05345_amd import dms
    B, T, H, g, w = 1, 150, 2, 3, 40
    rng = np.random.default_rng(30)
    shapes = {"q": (B, T, H * g, D), "k": (B, T, H, D), "v": (B, T, H, D), "dout": (B, T, H * g, D)}
    x = {n: _dev_bf16(_bf16(rng.normal(size=s))) for n, s in shapes.items()}
    alpha = torch.from_numpy(rng.uniform(0, 1, (B, T, H)).astype(np.float32)).cuda()
    cfg = dms.make_train_config(B, T, H, g, D, w)
    ws = torch.empty(dms.dms_train_workspace(cfg), dtype=torch.uint8, device="cuda")

    def run(x):
        out = torch.empty(shapes["q"], device="cuda")
        lse = torch.empty((B, H * g, T), device="cuda")
        grads = [torch.empty(shapes[n], device="cuda") for n in ("q", "k", "v")] + [torch.empty_like(alpha)]
        dms.dms_train_attention_fwd(cfg, x["q"], x["k"], x["v"], alpha, out, lse, ws)
        dms.dms_train_attention_bwd(cfg, x["q"], x["k"], x["v"], alpha, out, lse, x["dout"], *grads, ws)
        return [out, lse, *grads]

    def shifted(t):
        buf = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")
        v = buf[1:1 + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16
        return v

    for a, b in zip(run(x), run({n: shifted(t) for n, t in x.items()})):
        # the split of the key-major pass depends on the room that the copies leave
        assert torch.allclose(a, b, rtol=1e-5, atol=1e-5 * float(a.abs().max()))
