"""The whole-network training kernels (rows through all layers; weight gradients of all layers in one
launch) at the edges of their tiles: batches of one row, around a 16-row tile and a 256-row block, and
beyond the 512 work-groups that then walk several tiles; one layer and eight; every padded width,
including 64 x 64 blocks that are half empty; unaligned input rows.  The oracle takes the GPU's own
forward values (forward: each layer's own input), as in the other MLP tests: 1e-6 forward, 1e-3 for
gradients, where a BF16 rounding of a data gradient can still fall the other way."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_common import rel, to_dev, to_np
from oracle.mlp import MLP, pad32
from test_gpu_mlp import _gpu_mlp, _input, _params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,B", [([49, 128, 41], 1), ([49, 128, 41], 15), ([90, 128, 128, 128, 41], 17),
                                      ([90, 128, 128, 128, 41], 255), ([81, 128, 90, 128, 20], 257),
                                      ([30, 60, 20, 128, 128, 100, 128, 64, 30], 100), ([70, 128], 8230),
                                      ([20, 20], 33)])
def test_forward_and_gradients_at_tile_edges(widths, B):
    W, b = _params(widths, 3)
    G, m = _gpu_mlp(widths, W, b)
    nl = len(widths) - 1
    P = [pad32(w) for w in widths]
    x = _input(B, widths[0], 4)
    t = np.zeros((B, P[-1]), dtype=np.float32)
    t[:, :widths[-1]] = np.random.default_rng(5).standard_normal((B, widths[-1]))
    buf = torch.zeros(x.size + 1, dtype=torch.float32, device="cuda")
    xd = buf[1:].view(B, P[0])  # four bytes past an aligned address
    xd.copy_(to_dev(x, torch.float32))
    td = to_dev(t, torch.float32)
    zs, acts, _ = m.forward(xd)
    work = torch.empty(2 * B * 128, dtype=torch.float32, device="cuda")
    m.grad.fill_(7.0)  # overwritten
    loss = C.c_double()
    p = lambda q: C.c_void_p(q.data_ptr())  # noqa: E731
    G._check(G.lib.ilh_mlp_backward(G.ctx, m.nl, m.cw, p(m.WT), p(xd), p(zs), p(acts), p(td), B, p(m.grad),
                                    p(m.grad[m.nW:]), p(work), C.byref(loss)))
    zg, ag, g = to_np(zs), to_np(acts), to_np(m.grad)
    zl, al, o = [], [], 0
    for l in range(nl):
        zl.append(zg[o:o + B * P[l + 1]].reshape(B, P[l + 1]))
        al.append(ag[o:o + B * P[l + 1]].reshape(B, P[l + 1]))
        o += B * P[l + 1]
    for l in range(nl):
        xin = x.astype(np.float64) if l == 0 else al[l - 1]
        z_ref = MLP([widths[l], widths[l + 1]], [W[l]], [b[l]]).forward(xin)[0][0]
        assert rel(zl[l], z_ref) <= 1e-6, l
    dW, db, oloss = MLP(widths, W, b).backward(x, zl, al, t.astype(np.float64))
    assert abs(loss.value - oloss) <= 1e-5 * oloss
    o = 0
    for l in range(nl):
        assert rel(g[o:o + dW[l].size], dW[l].ravel()) <= 1e-3, l
        o += dW[l].size
    for l in range(nl):
        assert rel(g[o:o + db[l].size], db[l]) <= 1e-3, l
        o += db[l].size


def test_unbuilt_layer_shapes_stay_refused():
    import paper_2609_16424_amd as ilh
    for widths in ([90, 90, 41], [30, 90, 41], [49, 64, 90]):
        W, b = _params(widths, 1)
        G, m = _gpu_mlp(widths, W, b)
        with pytest.raises(ilh.IlhError):
            m.forward(to_dev(_input(20, widths[0], 2), torch.float32))
