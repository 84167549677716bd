"""The conv grad_X contraction at the edges of its units and panels: sample
counts around 16, 32 and 64 slots per pixel (several pixels per unit below
that), channels around 64-channel panels, output channels that are whole 64s or
not, weights kept whole in LDS, in tap chunks and in channel chunks, more than
64 taps, strides 1 to 3; every group span of the block Householder quantizer
and the general plan.  Within 1e-5 row-normwise of the oracle."""
import numpy as np
import pytest

from oracle import backward as BW
from paper_2010_14298_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def err(got, ref):
    got, ref = got.reshape(got.shape[0], -1).astype(np.float64), ref.reshape(ref.shape[0], -1)
    den = np.abs(ref).max(axis=1)
    num = np.abs(got - ref).max(axis=1)
    return float(np.max(np.where(den > 0, num / np.where(den > 0, den, 1), num)))


def check(seed, n, c, h, w, o, kh, kw, st, pad, qb_x):
    from paper_2010_14298_amd import fqt as f
    rng = np.random.default_rng(seed)
    X = np.maximum(rng.standard_normal((n, h, w, c)), 0).astype(np.float32)
    W = rng.standard_normal((o, kh, kw, c)).astype(np.float32)
    ho, wo = (h + 2 * pad - kh) // st + 1, (w + 2 * pad - kw) // st + 1
    G = synth.lognormal_row_gradient(rng, n, ho * wo * o).reshape(n, ho, wo, o)
    r = BW.conv_backward(X, W, G, st, pad, qb_x=qb_x, seed=6)
    gW, gX, ws = f.fqt_conv_backward_im2col(*(torch.from_numpy(t).cuda() for t in (X, W, G)), st, pad, qb_x=qb_x,
                                            seed=6)
    assert f.fqt_workspace_status(ws) == 0
    assert err(gW.cpu().numpy(), r["grad_W64"]) <= 1e-5
    assert err(gX.cpu().numpy(), r["grad_X64"]) <= 1e-5


@pytest.mark.parametrize("n", [1, 16, 17, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("o", [64, 48])
@pytest.mark.parametrize("qb_x", [("psq", 5, 0), ("bhq", 5, 64), ("bhq", 5, 8), ("bhq", 5, 12)])
def test_samples_per_pixel(n, o, qb_x):
    check(n + o, n, 20, 5, 4, o, 3, 3, 1, 1, qb_x)


@pytest.mark.parametrize("k", [1, 2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("n", [15, 30, 70])
def test_group_spans(k, n):
    check(k * n, n, 65, 3, 3, 64, 3, 3, 2, 1, ("bhq", 5, k))


@pytest.mark.parametrize("geo", [
    # c, h, w, o, kh, kw, stride, pad
    (63, 4, 4, 512, 3, 3, 1, 1),      # 4608 codes per panel row: tap chunks
    (64, 2, 3, 2048, 1, 1, 1, 0),     # channel chunks
    (65, 2, 2, 1040, 1, 1, 1, 0),     # channel chunks, the last one part
    (16, 12, 11, 16, 9, 9, 1, 4),     # 81 taps
    (16, 9, 9, 128, 1, 1, 2, 0),      # pixels without a tap
    (130, 7, 6, 192, 3, 3, 3, 1),     # stride 3, three panels
    (64, 3, 3, 192, 3, 3, 1, 1),      # 112 KB panel
])
@pytest.mark.parametrize("n,qb_x", [(6, ("psq", 8, 0)), (70, ("bhq", 5, 64))])
def test_panels(geo, n, qb_x):
    check(sum(geo), n, *geo, qb_x)


def test_large_general_plan_workspace():
    # the general plan's float64 rows alone take 64 GiB of the workspace; gradient and weights of 0
    # and 1 are whole codes, so grad_X is their product exactly
    from paper_2010_14298_amd import fqt as f
    h, w, c, o = 255, 257, 8208, 16
    assert 8 * 16 * h * w * c > 1 << 36
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    G, W = (torch.rand(s, generator=gen, device="cuda").round() for s in ((1, h, w, o), (o, 1, 1, c)))
    X = torch.zeros((1, h, w, c), device="cuda")
    gW, gX, ws = f.fqt_conv_backward_im2col(X, W, G, 1, 0, qb_x=("bhq", 5, 3), seed=1)
    assert f.fqt_workspace_status(ws) == 0
    del ws
    torch.cuda.empty_cache()
    assert float(gW.abs().max()) == 0.0
    assert float((gX.view(h * w, c) - G.view(h * w, o) @ W.view(o, c)).abs().max()) <= 16 * 2.0 ** -22
