"""General block Householder plans around the sizes where the forward column
term and the inverse change their split: groups of one wave (up to 64 rows),
groups spread over a block, chunks that end inside a group.  Codes bit for bit,
gradients within 1e-5 row-normwise of the oracle's float64 products."""
import numpy as np
import pytest

from oracle import backward as BW
from oracle import quantizers as Q
from paper_2010_14298_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def rownorm_err(got, ref):
    den = np.abs(ref).max(axis=1)
    num = np.abs(got.astype(np.float64) - ref).max(axis=1)
    return float(np.max(np.where(den > 0, num / np.where(den > 0, den, 1), num)))


@pytest.mark.parametrize("block", [3, 63, 65, 128, 130, 701])
def test_group_sizes(block):
    from paper_2010_14298_amd import fqt as f
    N, d_in, d_out = 700, 70, 65
    X, W, G = synth.linear_small(seed=block, n=N, d_in=d_in, d_out=d_out)
    Xd, Wd, Gd = (torch.from_numpy(t).cuda() for t in (X, W, G))
    out = f.fqt_quantize_bhq(Gd, 5, block, seed=2)
    ref = Q.quantize_bhq(G, 5, block, seed=2, stream=0)
    np.testing.assert_array_equal(out["perm"].cpu().numpy(), ref["perm"])
    np.testing.assert_array_equal(out["q"].cpu().numpy(), (ref["code"] - Q.offset(5)).astype(np.int8))
    r = BW.linear_backward(X, W, G, qb_x=("bhq", 5, block), seed=2)
    gW, gX, ws = f.fqt_linear_backward(Xd, Wd, Gd, qb_x=("bhq", 5, block), seed=2)
    assert f.fqt_workspace_status(ws) == 0
    assert rownorm_err(gW.cpu().numpy(), r["grad_W64"]) <= 1e-5
    assert rownorm_err(gX.cpu().numpy(), r["grad_X64"]) <= 1e-5
