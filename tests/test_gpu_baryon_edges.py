"""The eigenvector tensor at the edges of its kernel: no triple at all (N_v = 1, 2), fewer
pairs than a workgroup's rows, odd N_v (unequal sides), one column tile more than a workgroup
takes, the smallest slice (two stages of four sites), slice counts that are and are not a
multiple of 8, against the definition in numpy.

Bound: every entry is a sum of 3 Ns^3 products of three FP64 numbers, so two orders of
summation differ by at most about 3 Ns^3 2^-52 times the sum of the absolute values."""
import numpy as np
import pytest

from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt,nv,k", [(2, 2, 1, (0, 0, 0)), (2, 8, 2, (1, 0, 0)), (2, 4, 3, (0, 1, 0)),
                                        (2, 8, 17, (0, 0, 0)), (4, 2, 18, (1, 2, 3)), (2, 2, 33, (0, 0, 1)),
                                        (2, 2, 113, (1, 1, 0)), (2, 8, 130, (0, 0, 0))])
def test_tensor_edges(ns, nt, nv, k):
    import torch

    import paper_1104_3870_amd as P

    say("baryon tensor", ns, nt, nv, k)
    rng = np.random.default_rng(ns * 1000 + nv)
    V = rng.standard_normal((nt, nv, ns ** 3, 3)) + 1j * rng.standard_normal((nt, nv, ns ** 3, 3))
    x = np.arange(ns)
    ph = np.exp(-2j * np.pi / ns * (k[2] * x[:, None, None] + k[1] * x[None, :, None] + k[0] * x[None, None, :]))
    ph = ph.reshape(-1, 1)
    T = torch.full((nt, nv, nv, nv), 7.0, dtype=torch.complex128, device="cuda")
    L = P.Lattice(ns, nt)
    P.laph_baryon_tensor(L.ctx, dev(V.reshape(nt, nv, ns, ns, ns, 3)), nv, k, T)
    got = host(T)
    size = np.abs(V).max() ** 3 * 6 * 3 * ns ** 3
    for t in range(nt):
        flat = V[t].reshape(nv, -1)
        for a in range(nv):
            ref = np.cross(ph * V[t, a], V[t]).reshape(nv, -1) @ flat.T
            ref[a] = 0.0  # repeated indices are exact zeros
            ref[:, a] = 0.0
            np.fill_diagonal(ref, 0.0)
            assert np.abs(got[t, a] - ref).max() <= 3 * ns ** 3 * 2.0 ** -52 * size, (t, a)
            assert not got[t, a, a].any() and not got[t, a, :, a].any() and not np.diagonal(got[t, a]).any()
