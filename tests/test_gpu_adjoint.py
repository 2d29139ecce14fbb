"""GPU parity of the reverse rounds on lane groups (csrc/adjoint.hip), which take
grids of at least half as many 64 x 4 tiles as the card has compute units: narrow
and thin images whose tiles are many and mostly empty, a pixel past a tile and past
a group of four, the class counts around each register bound and chunk of two,
every window side, both staging widths, all counts of feature planes.

Bar: that of test_gpu_backward.py, 1e-4 of each tensor's largest magnitude, and
1e-3 of a parameter derivative that does not cancel (at least 1e-2 of the
largest; the others to 1e-4 of it).  The messages are kept below about 30, as in
test_gpu_group.py, which keeps the logits that the derivative starts from good
to 4e-6.
"""
import numpy as np
import pytest

from oracle import OracleParams
from paper_1805_04777_amd import synth

pytestmark = pytest.mark.gpu

TOL_REL = 1e-4
TOL_PARAM = 1e-3


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
    (128, 3, 3, 1, 1, 2, False, 0, True, 0), (1, 2, 3, 512, 1, 3, True, 1, False, 0),
    (2, 21, 3, 256, 5, 2, False, 0, False, 1), (4, 24, 3, 66, 65, 2, True, 3, True, 0),
    (1, 2, 5, 509, 2, 2, False, 2, True, 0), (2, 12, 5, 129, 68, 2, True, 0, False, 0),
    (1, 13, 5, 257, 128, 2, False, 4, False, 0), (3, 22, 5, 171, 3, 3, False, 0, False, 2),
    (1, 21, 7, 512, 4, 2, False, 0, True, 0), (1, 11, 7, 257, 67, 2, True, 0, False, 0),
    (2, 23, 7, 4, 4096, 1, False, 0, False, 0), (128, 5, 7, 3, 7, 2, True, 0, False, 3),
    (1, 21, 7, 255, 132, 2, True, 2, False, 0), (1, 19, 7, 513, 9, 2, False, 3, True, 1),
    (2, 24, 7, 130, 72, 2, True, 4, False, 0), (1, 12, 7, 1, 8200, 2, False, 1, False, 0),
]


@pytest.mark.parametrize("B,C,k,H,W,T,compat,D,center,offset", CASES)
def test_lane_group_adjoint(crf, oracle_mod, B, C, k, H, W, T, compat, D, center, offset):
    import torch
    from paper_1805_04777_amd import convcrf as cc
    rng = np.random.default_rng(9000 + 100 * k + C + H + W)
    U = rng.normal(0.0, 1.5, (B, C, H, W)).astype(np.float32)
    I = np.clip(np.rint(rng.uniform(0, 200, (B, 3, 1, 1)) + rng.normal(0, 15, (B, 3, H, W))),
                0, 255).astype(np.float32)
    G = rng.normal(0.0, 1.0, (B, C, H, W)).astype(np.float32)
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
    args = gpu(U), gpu(I), p, T, gpu(G)
    got = crf.meanfield_backward(*args, grad_compat=True, grad_kernel=True)
    alone = crf.meanfield_backward(*args)
    torch.cuda.synchronize()
    assert torch.equal(alone[0], got[0])    # dL/dU, whatever else is asked for
    got = [x.cpu().numpy().astype(np.float64) for x in got if x is not None]
    op = OracleParams(filter_size=k, include_center=center, w_app=p.w_app, w_smooth=p.w_smooth)
    ref = oracle_mod.meanfield_backward(U, I, op, T, G, compat=mu, features=F)
    assert len(got) == len(ref)
    for name, a, b in zip(("dU", "dmu", None, "dF"), got, ref):
        if name:
            assert np.abs(a - b).max() <= TOL_REL * np.abs(b).max(), name
    dk, rk = got[2], ref[2]
    err, scale = np.abs(dk - rk), np.abs(rk).max()
    assert np.all(err <= np.where(np.abs(rk) >= 1e-2 * scale, TOL_PARAM * np.abs(rk),
                                  TOL_REL * scale)), (dk, rk)


# (B, C, k, H, W, T, blur, compat): one cell, cells past a 32 x 16 tile, a tile exactly,
# class counts at the two register bounds
BLUR_CASES = [
    (1, 1, 3, 2, 2, 2, 2, False), (2, 9, 3, 18, 34, 2, 2, True), (1, 24, 5, 14, 62, 1, 2, False),
    (3, 8, 5, 4, 4, 3, 4, True), (1, 24, 3, 16, 32, 2, 4, True), (2, 21, 7, 20, 68, 2, 4, False),
    (1, 2, 3, 8, 8, 3, 8, True), (1, 24, 3, 24, 40, 2, 8, False), (2, 22, 5, 16, 72, 2, 8, True),
]


@pytest.mark.parametrize("B,C,k,H,W,T,s,compat", BLUR_CASES)
def test_blur_point_and_transpose(crf, oracle_mod, B, C, k, H, W, T, s, compat):
    """The pointwise adjoints with the transpose of the upsampling in the same launch."""
    import torch
    from paper_1805_04777_amd import convcrf as cc
    rng = np.random.default_rng(9500 + 100 * s + C + H + W)
    U = rng.normal(0.0, 1.5, (B, C, H, W)).astype(np.float32)
    I = np.clip(np.rint(rng.uniform(0, 200, (B, 3, 1, 1)) + rng.normal(0, 15, (B, 3, H, W))),
                0, 255).astype(np.float32)
    G = rng.normal(0.0, 1.0, (B, C, H, W)).astype(np.float32)
    mu = synth.random_compat(C, seed=k) if compat else None
    kw = dict(filter_size=k, blur=s, w_app=30.0 / k ** 2, w_smooth=9.0 / k ** 2)
    t = lambda a: torch.from_numpy(a).cuda()
    got = crf.meanfield_backward(t(U), t(I), cc.Params(compat=mu, **kw), T, t(G),
                                 grad_compat=True, grad_kernel=True)
    torch.cuda.synchronize()
    got = [x.cpu().numpy().astype(np.float64) for x in got]
    ref = oracle_mod.meanfield_backward(U, I, OracleParams(**kw), T, G, compat=mu)
    for name, a, b in zip(("dU", "dmu"), got, ref):
        assert np.abs(a - b).max() <= TOL_REL * np.abs(b).max(), name
    scale = np.abs(ref[2]).max()
    big = np.abs(ref[2]) >= 1e-2 * scale
    err = np.abs(got[2] - ref[2])
    assert np.all(err[big] <= TOL_PARAM * np.abs(ref[2])[big]), (got[2], ref[2])
    assert np.all(err[~big] <= TOL_REL * scale), (got[2], ref[2])
