"""The network's kernels at the edges of their layouts against the oracle: site counts below, at
and past the 64 of a conversion tile with a ragged last one, one to four channels on either side
of a layer (the widths of the weight gradient's wave sum), one field and several.

Bounds: FP32 arithmetic against FP64 with the same weights.  An output takes two layers of at
most 432 products (relative 2^-24 each at worst, far below 2e-5 of the largest output); a weight
gradient sums over every site and field, 1e-4 of the largest."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, say
from oracle import ptnet as onet
from test_gpu_ptnet import bf16c, flat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt,ch,n", [(2, 2, [1, 1], 1), (2, 4, [1, 4, 1], 3), (4, 2, [1, 2, 1], 2),
                                        (6, 2, [1, 4, 4, 1], 1), (2, 8, [1, 1, 2, 1], 5)])
def test_network_edges(ns, nt, ch, n):
    import torch

    import paper_1104_3870_amd as P

    say("ptnet edges", ns, nt, ch, n)
    L = P.Lattice(ns, nt)
    U = synth.gauge_field(ns, nt, 0.4, 5)
    psi, gout = synth.random_spinor(ns, nt, 6, nrhs=n), synth.random_spinor(ns, nt, 7, nrhs=n)
    ws = [bf16c(w) for w in onet.init_weights(ch, seed=3, scale=0.2)]
    net = P.PTNet(L.ctx, ch, seed=1)
    net.set_weights(flat(ws))
    out, gin = (torch.empty(psi.shape, dtype=torch.complex128, device="cuda") for _ in range(2))
    gw = np.zeros(2 * net.n_weights)
    P.laph_ptnet_forward(L.ctx, net.handle, dev(U), -1.0, dev(psi), out, n)
    P.laph_ptnet_backward(L.ctx, net.handle, dev(U), -1.0, dev(psi), dev(gout), gin, gw, n)
    o, gi, gw = host(out), host(gin), gw.view(np.complex128)
    ref_w = [np.zeros_like(w) for w in ws]
    for r in range(n):
        f, acts = onet.forward(U, ws, psi[r], bc_t=-1.0)
        g_in, g_w = onet.backward(U, ws, acts, gout[r])
        assert np.abs(o[r] - f).max() <= 2e-5 * np.abs(f).max()
        assert np.abs(gi[r] - g_in).max() <= 2e-5 * np.abs(g_in).max()
        for l in range(len(ws)):
            ref_w[l] += g_w[l]
    assert np.abs(gw - flat(ref_w)).max() <= 1e-4 * np.abs(flat(ref_w)).max()
    net.close()
    L.close()
