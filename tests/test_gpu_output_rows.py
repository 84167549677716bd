"""Output rows on both sides of the rule that picks nontemporal stores: row
pitches of whole 128-byte lines, of whole 64-byte halves, of whole 16 bytes and
of none, and output buffers on and off those boundaries.  Gradients and activations within
1e-5 row-normwise of the oracle's float64 products, nothing written outside the
buffers."""
import numpy as np
import pytest

from oracle import backward as BW
from oracle import chain as CH
from paper_2010_14298_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
REL_TOL = 1e-5
GUARD = -7.5


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def out(shape, shift):
    """A buffer `shift` floats past a 256-byte boundary, between guard values."""
    n = int(np.prod(shape))
    buf = torch.full((n + 128,), GUARD, device="cuda")
    return buf, buf[shift:shift + n].view(*shape)


def check(buf, t, shift, ref):
    rest = torch.cat([buf[:shift], buf[shift + t.numel():]])
    assert bool((rest == GUARD).all())
    got, ref = t.cpu().numpy().reshape(ref.shape[0], -1).astype(np.float64), ref.reshape(ref.shape[0], -1)
    den = np.abs(ref).max(axis=1)
    num = np.abs(got - ref).max(axis=1)
    assert float(np.max(np.where(den > 0, num / np.where(den > 0, den, 1), num))) <= REL_TOL


SHIFTS = [0, 1, 4, 16]


@pytest.mark.parametrize("width", [32, 48, 33, 36, 160])
@pytest.mark.parametrize("qb_x", [("psq", 8, 0), ("bhq", 5, 64), ("bhq", 5, 12)])
def test_linear(width, qb_x):
    from paper_2010_14298_amd import fqt as f
    X, W, G = synth.linear_small(seed=width, n=70, d_in=width, d_out=64)
    r = BW.linear_backward(X, W, G, qb_x=qb_x, seed=3)
    for shift in SHIFTS:
        bw, gW = out(W.shape, shift)
        bx, gX = out(X.shape, shift)
        f.fqt_linear_backward(dev(X), dev(W), dev(G), qb_x=qb_x, seed=3, grad_W=gW, grad_X=gX)
        check(bw, gW, shift, r["grad_W64"])
        check(bx, gX, shift, r["grad_X64"])


@pytest.mark.parametrize("width", [32, 48, 33])
def test_forward(width):
    from paper_2010_14298_amd import fqt as f
    X, W, _ = synth.linear_small(seed=width, n=70, d_in=64, d_out=width)
    ref = CH.layer_forward(X, W, True)[1]
    for shift in SHIFTS:
        by, Y = out((70, width), shift)
        f.fqt_linear_forward(dev(X), dev(W), relu=True, Y=Y)
        check(by, Y, shift, ref)


@pytest.mark.parametrize("c", [16, 32, 20, 67])
@pytest.mark.parametrize("n,qb_x", [(6, ("psq", 8, 0)), (70, ("bhq", 5, 64))])
def test_conv(c, n, qb_x):
    from paper_2010_14298_amd import fqt as f
    rng = np.random.default_rng(c)
    X = rng.standard_normal((n, 5, 4, c)).astype(np.float32)
    W = rng.standard_normal((64, 3, 3, c)).astype(np.float32)
    G = synth.lognormal_row_gradient(rng, n, 5 * 4 * 64).reshape(n, 5, 4, 64)
    r = BW.conv_backward(X, W, G, 1, 1, qb_x=qb_x, seed=3)
    for shift in SHIFTS:
        bw, gW = out(W.shape, shift)
        bx, gX = out(X.shape, shift)
        f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), 1, 1, qb_x=qb_x, seed=3, grad_W=gW, grad_X=gX)
        check(bw, gW, shift, r["grad_W64"])
        check(bx, gX, shift, r["grad_X64"])
