"""GPU parity of fqt_conv_backward_im2col against the oracle's explicit im2col.

Small shapes cover every element (stride 1 / 2, 1x1, 3x3, 7x7, ragged
sample counts, all three gradient quantizers; rectangular images and
kernels, 25- and 36-tap kernels, part K stages and column tiles); the 3x3
64 -> 64 layer at 56 x 56 with a batch of 128 (the launch configuration of
the conv benchmark) is checked on sampled outputs computed one by one in
float64.
"""
import numpy as np
import pytest

from oracle import backward as BW
from oracle import quantizers as Q
from paper_2010_14298_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
REL_TOL = 1e-5


def fqt():
    from paper_2010_14298_amd import fqt as f
    f.load()
    return f


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def rownorm_err(got, ref):
    got = got.reshape(got.shape[0], -1).astype(np.float64)
    ref = ref.reshape(ref.shape[0], -1).astype(np.float64)
    den = np.abs(ref).max(axis=1)
    num = np.abs(got - ref).max(axis=1)
    return float(np.max(np.where(den > 0, num / np.where(den > 0, den, 1), num)))


def run(X, W, G, stride, pad, qb_x, seed=0):
    f = fqt()
    gW, gX, ws = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=qb_x, seed=seed)
    assert f.fqt_workspace_status(ws) == 0
    return host(gW), host(gX)


SHAPES = [
    # n, c, h, o, k, stride, pad
    (4, 8, 6, 16, 3, 1, 1),
    (3, 5, 7, 16, 3, 2, 1),
    (4, 16, 6, 32, 1, 2, 0),
    (2, 3, 12, 16, 7, 2, 3),
    (5, 8, 5, 16, 1, 1, 0),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("qb_x", [("ptq", 8, 0), ("psq", 5, 0), ("bhq", 5, 2), ("bhq", 4, 4)])
def test_conv_small(shape, qb_x):
    n, c, h, o, k, st, pad = shape
    X, W, G = synth.conv_layer(seed=sum(shape), n=n, c=c, h=h, w=h, o=o, k=k, stride=st, pad=pad, stem=(c == 3))
    r = BW.conv_backward(X, W, G, st, pad, qb_x=qb_x, seed=3)
    gW, gX = run(X, W, G, st, pad, qb_x, seed=3)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


@pytest.mark.parametrize("qb_x", [("bhq", 5, 64), ("psq", 8, 0), ("bhq", 5, 16)])
def test_conv_ragged_batch_groups(qb_x):
    # 130 samples: groups 64 + 64 + 2, slot blocks padded to 192 per pixel
    X, W, G = synth.conv_layer(seed=7, n=130, c=16, h=5, w=5, o=16, k=3, stride=1, pad=1)
    r = BW.conv_backward(X, W, G, 1, 1, qb_x=qb_x, seed=1)
    gW, gX = run(X, W, G, 1, 1, qb_x, seed=1)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


def conv_inputs(seed, n, c, h, w, o, kh, kw, stride, pad):
    """Rectangular images and kernels (the synthetic generator makes square
    ones): X half-normal NHWC, W He-init [o, kh, kw, c], G per-sample
    log-normal scales."""
    rng = np.random.default_rng(seed)
    X = np.maximum(rng.standard_normal((n, h, w, c)), 0.0).astype(np.float32)
    W = (rng.standard_normal((o, kh, kw, c)) * np.sqrt(2.0 / (kh * kw * c))).astype(np.float32)
    ho = (h + 2 * pad - kh) // stride + 1
    wo = (w + 2 * pad - kw) // stride + 1
    G = synth.lognormal_row_gradient(rng, n, ho * wo * o).reshape(n, ho, wo, o)
    return X, W, G


GEOMETRIES = [
    # n, c, h, w, o, kh, kw, stride, pad
    (3, 8, 9, 7, 16, 5, 5, 1, 2),    # 25 taps, rectangular image
    (4, 8, 6, 5, 16, 1, 3, 1, 1),    # 1 x 3 kernel
    (4, 8, 5, 7, 16, 3, 1, 1, 0),    # 3 x 1 kernel, no padding
    (3, 8, 7, 7, 16, 3, 3, 1, 0),    # valid 3 x 3
    (3, 24, 6, 6, 48, 3, 3, 1, 1),   # K = 432: a part K stage; 24 input channels: a part column tile
    (2, 8, 8, 8, 16, 6, 6, 1, 2),    # 36 taps
]


IMPLICIT_GEOMETRIES = [
    # larger images at stride 1: several 128-pixel stages per sample
    (3, 8, 24, 28, 16, 1, 3, 1, 1),   # 1 x 3 kernel, rectangular image
    (3, 8, 28, 30, 16, 3, 1, 1, 1),   # 3 x 1 kernel
    (2, 24, 14, 14, 48, 3, 3, 1, 1),  # part stages, part column tile
    (2, 8, 30, 30, 16, 2, 2, 1, 0),   # even kernel, no padding
]


@pytest.mark.parametrize("geo", GEOMETRIES + IMPLICIT_GEOMETRIES)
@pytest.mark.parametrize("qb_x", [("bhq", 5, 2), ("psq", 6, 0)])
def test_conv_geometries(geo, qb_x):
    n, c, h, w, o, kh, kw, st, pad = geo
    X, W, G = conv_inputs(sum(geo), n, c, h, w, o, kh, kw, st, pad)
    r = BW.conv_backward(X, W, G, st, pad, qb_x=qb_x, seed=5)
    gW, gX = run(X, W, G, st, pad, qb_x, seed=5)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


def test_conv_stage1_mid_size():
    # ResNet-50 stage-1 3x3 64 -> 64 conv at 14 x 14, batch 128, BHQ-5 across samples
    X, W, G = synth.conv_layer(seed=2, n=128, c=64, h=14, w=14, o=64, k=3, stride=1, pad=1)
    r = BW.conv_backward(X, W, G, 1, 1, qb_x=("bhq", 5, 64), seed=0)
    gW, gX = run(X, W, G, 1, 1, ("bhq", 5, 64), seed=0)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


def test_conv_stage1_full_size_sampled():
    """Batch 128, 64 -> 64, 3x3, 56 x 56, BHQ-5: sampled grad_X samples and grad_W entries."""
    X, W, G = synth.conv_layer(seed=0, n=128, c=64, h=56, w=56, o=64, k=3, stride=1, pad=1)
    gW, gX = run(X, W, G, 1, 1, ("bhq", 5, 64), seed=0)
    n, h, w, c = X.shape
    o = W.shape[0]
    qx = Q.quantize_ptq(X.reshape(n, -1), 8, False)
    qw = Q.quantize_ptq(W.reshape(o, -1), 8, False)
    qb2 = Q.quantize_bhq(G.reshape(n, -1), 5, 64, seed=0, stream=1)
    Xr = Q.dequantize(qx).reshape(n, h, w, c)
    Wr = Q.dequantize(qw).reshape(o, 3, 3, c)
    G2r = Q.dequantize(qb2).reshape(n, h, w, o)
    rng = np.random.default_rng(0)
    for i in rng.choice(n, 3, replace=False):
        # input gradient of sample i: sum over taps of shifted G~ times W~
        ref = np.zeros((h, w, c))
        for rr in range(3):
            for ss in range(3):
                gpad = np.zeros((h + 2, w + 2, o))
                gpad[1:-1, 1:-1] = G2r[i]
                # output pixel (y, x) feeds input (y + rr - 1, x + ss - 1)
                sub = gpad[2 - rr: 2 - rr + h, 2 - ss: 2 - ss + w]
                ref += sub @ Wr[:, rr, ss, :]
        assert rownorm_err(gX[i].reshape(1, -1), ref.reshape(1, -1)) <= REL_TOL
    qb1 = Q.quantize_ptq(G.reshape(n, -1), 8, True, seed=0, stream=0)
    G1r = Q.dequantize(qb1).reshape(n, h, w, o)
    xpad = np.zeros((n, h + 2, w + 2, c))
    xpad[:, 1:-1, 1:-1] = Xr
    for oo in rng.choice(o, 4, replace=False):
        ref = np.zeros((3, 3, c))
        for rr in range(3):
            for ss in range(3):
                ref[rr, ss] = np.einsum("nyx,nyxc->c", G1r[..., oo], xpad[:, rr: rr + h, ss: ss + w])
        assert rownorm_err(gW[oo].reshape(1, -1), ref.reshape(1, -1)) <= REL_TOL


def test_conv_unsupported_channels():
    f = fqt()
    X, W, G = synth.conv_layer(seed=0, n=2, c=4, h=5, w=5, o=8, k=3, stride=1, pad=1)
    with pytest.raises(f.FqtError) as e:
        f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), 1, 1, qb_x=("psq", 8, 0))
    assert e.value.code == 2


# ---------------------------------------------------------------------------
# Exact accumulators of the conv contractions.  Inputs on the integer grid
# 0..255 (each tensor, and each gradient sample, holding both 0 and 255) make
# every quantizer exact: Q_f, Q_theta and the per-sample Q_b2 have step 1 and
# zero 0, and the stochastic Q_b1 never rounds (fraction 0).  The float64
# epilogues then evaluate exact integers, so grad_W and grad_X must equal the
# float32 rounding of the exact integer contractions, which sparse inputs
# keep below 2^24: any accumulator off by one (or a zero-point term at a
# padded tap) changes an output.
# ---------------------------------------------------------------------------
def grid_conv_inputs(seed, n, c, h, o, k, stride, pad, dx=0.01, dw=0.1, dg=0.01):
    rng = np.random.default_rng(seed)
    ho = (h + 2 * pad - k) // stride + 1

    def sparse(shape, d):
        v = rng.integers(1, 256, shape)
        return np.where(rng.random(shape) < d, v, 0).astype(np.float32)

    X = sparse((n, h, h, c), dx)
    X.flat[rng.integers(X.size)] = 255.0
    X.flat[rng.integers(X.size)] = 0.0
    W = sparse((o, k, k, c), dw)
    W.flat[rng.integers(W.size)] = 255.0
    W.flat[rng.integers(W.size)] = 0.0
    G = sparse((n, ho, ho, o), dg)
    Gf = G.reshape(n, -1)
    Gf[np.arange(n), rng.integers(0, Gf.shape[1], n)] = 255.0
    Gf[np.arange(n), rng.integers(0, Gf.shape[1], n)] = 0.0
    return X, W, G


def exact_conv_grads(X, W, G, stride, pad):
    """grad_W and grad_X of the conv as float64 tap-by-tap products (exact:
    integer sums below 2^53)."""
    n, h, w, c = X.shape
    o, kh, kw, _ = W.shape
    ho, wo = G.shape[1:3]
    Xp = np.zeros((n, h + 2 * pad, w + 2 * pad, c))
    Xp[:, pad: pad + h, pad: pad + w] = X
    Gf = G.reshape(-1, o).astype(np.float64)
    gW = np.zeros((o, kh, kw, c))
    gXp = np.zeros_like(Xp)
    for r in range(kh):
        for s in range(kw):
            sl = (slice(None), slice(r, r + stride * (ho - 1) + 1, stride), slice(s, s + stride * (wo - 1) + 1, stride))
            gW[:, r, s, :] = Gf.T @ Xp[sl].reshape(-1, c)
            gXp[sl] += (Gf @ W[:, r, s, :].astype(np.float64)).reshape(n, ho, wo, c)
    return gW, gXp[:, pad: pad + h, pad: pad + w]


GRID_GEOMS = [
    (128, 64, 56, 64, 3, 1, 1),     # the 56 x 56 layer at full size
    (150, 16, 9, 32, 3, 2, 1),      # more slots per input pixel than one unit of 64
    (40, 3, 32, 64, 7, 2, 3),       # stem-like: 7 x 7, stride 2, three channels
    (24, 32, 14, 48, 1, 2, 0),      # 1 x 1, stride 2
    (8, 16, 11, 16, 5, 1, 2),       # 5 x 5, odd image
    (6, 8, 14, 16, 3, 1, 1),        # 8 channels, padded to 16
    (4, 16, 28, 32, 3, 1, 1),       # 28 x 28
    (3, 8, 16, 16, 1, 1, 0),        # 1 x 1
    (2, 8, 44, 16, 5, 1, 2),        # 5 x 5 on 44 x 44
    (3, 8, 16, 16, 3, 1, 0),        # valid 3 x 3
]


@pytest.mark.parametrize("geom", GRID_GEOMS, ids=lambda g: "n{}_c{}_h{}_o{}_k{}_s{}_p{}".format(*g))
def test_conv_contractions_exact_on_the_grid(geom):
    n, c, h, o, k, stride, pad = geom
    X, W, G = grid_conv_inputs(n + c + o, n, c, h, o, k, stride, pad)
    refW, refX = exact_conv_grads(X, W, G, stride, pad)
    assert np.abs(refW).max() < 2 ** 24 and np.abs(refX).max() < 2 ** 24
    f = fqt()
    gW, gX, ws = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=("psq", 8, 0),
                                           qb_w=("ptq", 8, 0), seed=1)
    assert f.fqt_workspace_status(ws) == 0
    np.testing.assert_array_equal(host(gW), refW.astype(np.float32))
    np.testing.assert_array_equal(host(gX), refX.astype(np.float32))


def test_conv_contractions_exact_per_sample_scales():
    # per-sample Q_b1 and Q_b2 on the grid with sample i scaled by 2^(i mod 3):
    # each sample's step is 2^(i mod 3), so both quantizers stay exact while a
    # per-tensor one would not, and every sample's int32 block and its scale
    # must be right for grad_W to equal the exact sum
    for geom in GRID_GEOMS:
        n, c, h, o, k, stride, pad = geom
        X, W, G = grid_conv_inputs(n + c + o, n, c, h, o, k, stride, pad)
        G = G * (2.0 ** (np.arange(n) % 3)).reshape(n, 1, 1, 1).astype(np.float32)
        refW, refX = exact_conv_grads(X, W, G, stride, pad)
        assert np.abs(refW).max() < 2 ** 24 and np.abs(refX).max() < 2 ** 24
        f = fqt()
        gW, gX, ws = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=("psq", 8, 0),
                                               qb_w=("psq", 8, 0), seed=2)
        assert f.fqt_workspace_status(ws) == 0
        np.testing.assert_array_equal(host(gW), refW.astype(np.float32), err_msg=str(geom))
        np.testing.assert_array_equal(host(gX), refX.astype(np.float32), err_msg=str(geom))
        # BHQ across samples puts the grad_W operands in slot order: the
        # per-sample scales must follow the permutation
        gW, _, ws = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=("bhq", 5, 4),
                                              qb_w=("psq", 8, 0), seed=2)
        assert f.fqt_workspace_status(ws) == 0
        np.testing.assert_array_equal(host(gW), refW.astype(np.float32), err_msg=str(geom))


# ---------------------------------------------------------------------------
# Per-sample Q_b1: the weight-gradient contraction in one K block per sample
# (the sample's output pixels, padded to whole 128-byte stages), an exact
# int32 sum per block, then the sample's scale in float64.
# ---------------------------------------------------------------------------
def run_w(X, W, G, stride, pad, qb_x, qb_w, seed=0):
    f = fqt()
    gW, gX, ws = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=qb_x, qb_w=qb_w, seed=seed)
    assert f.fqt_workspace_status(ws) == 0
    return host(gW), host(gX)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("qbs", [(("ptq", 8, 0), ("psq", 8, 0)), (("bhq", 5, 2), ("psq", 8, 0)),
                                 (("psq", 5, 0), ("psq", 4, 0))], ids=["ptq8-psq8", "bhq5-psq8", "psq5-psq4"])
def test_conv_per_sample_grad_w(shape, qbs):
    n, c, h, o, k, st, pad = shape
    qb_x, qb_w = qbs
    X, W, G = synth.conv_layer(seed=sum(shape), n=n, c=c, h=h, w=h, o=o, k=k, stride=st, pad=pad, stem=(c == 3))
    r = BW.conv_backward(X, W, G, st, pad, qb_x=qb_x, qb_w=qb_w, seed=4)
    gW, gX = run_w(X, W, G, st, pad, qb_x, qb_w, seed=4)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


@pytest.mark.parametrize("geo", GEOMETRIES[:3] + IMPLICIT_GEOMETRIES)
def test_conv_per_sample_grad_w_geometries(geo):
    n, c, h, w, o, kh, kw, st, pad = geo
    X, W, G = conv_inputs(sum(geo) + 1, n, c, h, w, o, kh, kw, st, pad)
    r = BW.conv_backward(X, W, G, st, pad, qb_x=("bhq", 5, 2), qb_w=("psq", 8, 0), seed=6)
    gW, gX = run_w(X, W, G, st, pad, ("bhq", 5, 2), ("psq", 8, 0), seed=6)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


def test_conv_per_sample_grad_w_ragged_groups():
    # 130 samples in BHQ groups 64 + 64 + 2: 130 K blocks in slot order
    X, W, G = synth.conv_layer(seed=8, n=130, c=16, h=5, w=5, o=16, k=3, stride=1, pad=1)
    r = BW.conv_backward(X, W, G, 1, 1, qb_x=("bhq", 5, 64), qb_w=("psq", 8, 0), seed=1)
    gW, gX = run_w(X, W, G, 1, 1, ("bhq", 5, 64), ("psq", 8, 0), seed=1)
    assert rownorm_err(gW, r["grad_W64"]) <= REL_TOL
    assert rownorm_err(gX, r["grad_X64"]) <= REL_TOL


def test_conv_per_sample_grad_w_full_size_sampled():
    """Batch 128, 64 -> 64, 3x3, 56 x 56 (3136 output pixels: 25 stages per
    sample), BHQ-5 Q_b2 and per-sample 8-bit Q_b1: sampled grad_W rows."""
    X, W, G = synth.conv_layer(seed=0, n=128, c=64, h=56, w=56, o=64, k=3, stride=1, pad=1)
    gW, _ = run_w(X, W, G, 1, 1, ("bhq", 5, 64), ("psq", 8, 0), seed=0)
    n, h, w, c = X.shape
    o = W.shape[0]
    Xr = Q.dequantize(Q.quantize_ptq(X.reshape(n, -1), 8, False)).reshape(n, h, w, c)
    G1r = Q.dequantize(Q.quantize_psq(G.reshape(n, -1), 8, seed=0, stream=0)).reshape(n, h, w, o)
    xpad = np.zeros((n, h + 2, w + 2, c))
    xpad[:, 1:-1, 1:-1] = Xr
    rng = np.random.default_rng(1)
    for oo in rng.choice(o, 4, replace=False):
        ref = np.zeros((3, 3, c))
        for rr in range(3):
            for ss in range(3):
                ref[rr, ss] = np.einsum("nyx,nyxc->c", G1r[..., oo], xpad[:, rr: rr + h, ss: ss + w])
        assert rownorm_err(gW[oo].reshape(1, -1), ref.reshape(1, -1)) <= REL_TOL


@pytest.mark.parametrize("qbs", [(("bhq", 5, 4), ("ptq", 8, 0)), (("psq", 8, 0), ("psq", 8, 0))])
@pytest.mark.parametrize("geom", [(6, 8, 14, 16, 3, 1, 1), (40, 3, 32, 64, 7, 2, 3)])
def test_conv_without_input_gradient(geom, qbs):
    # a NULL grad_X skips Q_b2, Q_theta and the input-gradient contraction;
    # grad_W is unchanged: bit for bit with a per-tensor Q_b1 (exact integer
    # sums), within the float64 order of its per-sample sums otherwise
    n, c, h, o, k, stride, pad = geom
    qb_x, qb_w = qbs
    X, W, G = synth.conv_layer(seed=n + k, n=n, c=c, h=h, w=h, o=o, k=k, stride=stride, pad=pad, stem=(c == 3))
    f = fqt()
    gW, gX, _ = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=qb_x, qb_w=qb_w, seed=3)
    gW1, gX1, ws = f.fqt_conv_backward_im2col(dev(X), dev(W), dev(G), stride, pad, qb_x=qb_x, qb_w=qb_w, seed=3,
                                              input_grad=False)
    assert gX1 is None and f.fqt_workspace_status(ws) == 0
    if qb_w[0] == "ptq":
        np.testing.assert_array_equal(host(gW1), host(gW))
    else:
        assert rownorm_err(host(gW1), host(gW)) <= 1e-6
    r = BW.conv_backward(X, W, G, stride, pad, qb_x=qb_x, qb_w=qb_w, seed=3)
    assert rownorm_err(host(gW1), r["grad_W64"]) <= REL_TOL
