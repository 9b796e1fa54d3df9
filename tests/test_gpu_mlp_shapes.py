"""The cost-model network's kernels at the edges of their sizes, against the FP64 oracle: one unit and
one row, the row kernels' largest network and rows that do not fill a workgroup, and networks above
it that take the general kernels."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nin,hid,batch", [(1, 1, 1), (12, 64, 1712), (12, 64, 15), (64, 64, 17), (3, 33, 100),
                                           (65, 64, 33), (5, 80, 100), (70, 130, 40)])
def test_mlp_shapes_match_oracle(nin, hid, batch):
    import torch

    from paper_2608_16940_amd import costmodel as C
    rng = np.random.default_rng([nin, hid, batch])
    p = C.init_params(3, nin, hid)
    p += (0.1 * rng.standard_normal(p.size)).astype(np.float32)
    X = rng.uniform(-1, 1, (batch, nin)).astype(np.float32)
    t = rng.standard_normal(batch).astype(np.float32)
    net = C.DeviceMLP(p, batch, nin=nin, hid=hid)
    Xd, td = torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()
    y = net.forward(Xd).cpu().numpy()
    g = net.backward(Xd, td).cpu().numpy()
    P64 = [a.astype(np.float64) for a in C.split_params(p, nin, hid)]
    yref, _ = oracle.mlp_forward(P64, X.astype(np.float64))
    loss, gref = oracle.mlp_loss_grad(P64, X.astype(np.float64), t.astype(np.float64))
    gref = np.concatenate([np.asarray(a).reshape(-1) for a in gref])
    # FP32 chains of nin, hid and batch / 16 + 80 terms; 64 for what the sums cancel
    tol = 64 * (nin + hid + batch / 16 + 80) * 2.0 ** -24
    say = (nin, hid, batch, np.abs(y - np.ravel(yref)).max(), np.linalg.norm(g - gref) / np.linalg.norm(gref))
    print(say, flush=True)
    assert np.abs(y - np.ravel(yref)).max() <= tol * max(1.0, np.abs(yref).max())
    assert np.linalg.norm(g - gref) <= tol * np.linalg.norm(gref)
    assert abs(net.loss.item() - loss) <= tol * loss
    first = g.copy()
    assert np.array_equal(first, net.backward(Xd, td).cpu().numpy())  # the same bits every time
