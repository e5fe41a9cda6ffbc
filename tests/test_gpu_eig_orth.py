"""max_orth of the eigensolver's statistics is the deviation of the returned vectors' Gram matrices
from 1, not the rounding of its own sums: on the free field, whose eigenvectors are plane waves
(terms all of one size, where a long running sum rounds one way), and on a rough field.

Bound: pieces of at most 200 sites add up 600 terms of a unit sum one after the other and their
sums pairwise or by at most 64 more; 600 + 64 half-unit roundings of 1 at worst, 4e-14."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt,nv,m,lamc,eps", [(2, 2, 1, 23, 3.0, 0.5), (10, 2, 20, 60, 1.0, 0.4), (14, 2, 20, 60, 0.5, 0.0),
                                                 (16, 2, 24, 64, 0.5, 0.0), (16, 2, 24, 64, 0.5, 0.4)])
def test_max_orth(ns, nt, nv, m, lamc, eps):
    import torch

    import paper_1104_3870_amd as P

    say("max_orth", ns, nt, nv, eps)
    U = synth.gauge_field(ns, nt, eps, 7) if eps else synth.unit_gauge_field(ns, nt)
    L = P.Lattice(ns, nt)
    evals = np.zeros((nt, nv))
    evecs = torch.empty((nt, nv, ns, ns, ns, 3), dtype=torch.complex128, device="cuda")
    st = P.laph_eigvecs(L.ctx, dev(U), 0.1, 2, nv, evals, evecs, krylov=m, lam_c=lamc, tol=1e-12, max_restarts=200)
    V = host(evecs).reshape(nt, nv, -1)
    want = 0.0
    for v in V:
        # NumPy adds pairwise along the last axis: a few roundings
        G = np.array([np.sum(np.conj(a) * v, axis=-1) for a in v])
        want = max(want, np.abs(G - np.eye(nv)).max())
    say("  reported", st.max_orth, "summed pairwise", want)
    assert abs(st.max_orth - want) <= 600 * 2.0 ** -53 + 64 * 2.0 ** -53
    L.close()
