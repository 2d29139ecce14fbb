"""GPU parity of the lane-group rounds (csrc/group.hip) where their tiling, class
chunks and splits of the window end: one pixel, one class, a class past a chunk
of three, a pixel past a tile and past a group of four, every window side, both
staging widths, all counts of feature planes.

Bar: that of test_gpu_parity.py, 1e-4 absolute on every probability and rows
summing to 1 within 1e-5 against the double-precision oracle.  The messages are
kept below about 30 (|w| <= 3), where float32 logits are good to 4e-6 and three
rounds multiply that by less than ten.
"""
import numpy as np
import pytest

from oracle import OracleParams
from paper_1805_04777_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def crf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from paper_1805_04777_amd import convcrf as cc
    ctx = cc.ConvCRF(0)
    yield ctx
    ctx.close()


# (B, C, k, H, W, T, compat, D, include_center, offset of the tensors in floats)
CASES = [
    (1, 1, 3, 1, 1, 2, False, 0, False, 0), (2, 2, 3, 9, 65, 3, True, 1, True, 0),
    (1, 24, 3, 17, 68, 2, False, 0, False, 0), (1, 13, 3, 8, 64, 2, True, 0, False, 1),
    (1, 3, 5, 7, 63, 2, False, 2, False, 0), (2, 12, 5, 8, 64, 3, True, 0, True, 0),
    (1, 22, 5, 16, 132, 2, False, 3, False, 0), (1, 4, 5, 5, 2, 2, False, 0, False, 0),
    (1, 21, 7, 9, 67, 2, False, 0, True, 0), (2, 21, 7, 8, 128, 2, True, 4, False, 0),
    (1, 6, 7, 1, 130, 3, False, 0, False, 0), (1, 19, 7, 24, 60, 2, False, 0, False, 3),
    (1, 24, 7, 11, 72, 2, True, 0, False, 0), (1, 21, 9, 4, 64, 2, False, 0, False, 0),
    (2, 7, 9, 5, 65, 2, True, 2, True, 0), (1, 16, 9, 13, 140, 2, False, 4, False, 0),
    (1, 21, 11, 4, 64, 2, False, 0, False, 0), (1, 5, 11, 12, 71, 2, True, 1, True, 0),
    (2, 24, 11, 3, 36, 2, False, 3, False, 2), (1, 21, 13, 5, 68, 2, False, 0, True, 0),
    (1, 10, 13, 17, 33, 2, True, 2, False, 0), (1, 24, 13, 4, 200, 2, False, 4, False, 0),
    (1, 21, 15, 8, 32, 2, False, 0, False, 0), (2, 8, 15, 9, 33, 2, True, 3, True, 0),
    (1, 13, 15, 20, 70, 2, False, 1, False, 1),
]


@pytest.mark.parametrize("B,C,k,H,W,T,compat,D,center,offset", CASES)
def test_lane_group_rounds(crf, oracle_mod, B, C, k, H, W, T, compat, D, center, offset):
    import torch
    from paper_1805_04777_amd import convcrf as cc
    rng = np.random.default_rng(7000 + 100 * k + C + H + W)
    U = rng.normal(0.0, 2.0, (B, C, H, W)).astype(np.float32)
    I = np.clip(np.rint(rng.uniform(0, 200, (B, 3, 1, 1)) + rng.normal(0, 15, (B, 3, H, W))),
                0, 255).astype(np.float32)
    F = None
    if D:
        yy, xx = np.meshgrid(np.arange(H), np.arange(W), indexing="ij")
        F = np.stack([yy, xx, yy, xx][:D])[None] + rng.normal(0.0, 0.5, (B, D, H, W))
        F = np.ascontiguousarray(F, dtype=np.float32)
    mu = synth.random_compat(C, seed=k) if compat else None

    def gpu(a):     # at `offset` floats from an aligned address
        buf = torch.empty(a.size + offset, dtype=torch.float32, device="cuda")
        t = buf[offset:].view(a.shape)
        t.copy_(torch.from_numpy(a))
        return t

    weight = 3.0 if k <= 5 else 30.0 / k ** 2
    p = cc.Params(filter_size=k, compat=mu, include_center=center, w_app=weight,
                  w_smooth=0.3 * weight, features=None if F is None else gpu(F))
    out = gpu(np.full_like(U, np.nan))
    crf.meanfield(gpu(U), gpu(I), p, T, out=out)
    torch.cuda.synchronize()
    Q = out.cpu().numpy().astype(np.float64)
    op = OracleParams(filter_size=k, include_center=center, w_app=p.w_app, w_smooth=p.w_smooth)
    ref = oracle_mod.meanfield(U, I, op, T, compat=mu, features=F)
    assert np.abs(Q - ref).max() <= 1e-4
    assert np.abs(Q.sum(1) - 1.0).max() <= 1e-5
