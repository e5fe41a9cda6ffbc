"""Eigensolver at the edges of its kernels: odd Krylov dimensions (padded Rayleigh-Ritz
blocks), the largest one, slices smaller than one workgroup's rows, a single wanted pair,
against the oracle's dense eigenpairs.

Bounds: a Ritz pair is accepted at a residual of tol |A| on A = T_8(B), whose slope at the
wanted end is above that of -Lap times 8 |A|/12, so tol = 1e-12 leaves residuals on -Lap
below 1e-10; eigenvalues (Rayleigh quotients) then agree to rounding, 1e-11 here, and a
vector's distance from its eigenspace is at most residual / gap, 1e-6 for the gaps above
1e-4 that are compared."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt,nv,m,lamc", [(2, 2, 1, 23, 3.0), (4, 2, 5, 33, 2.5), (4, 4, 9, 64, 2.5),
                                             (4, 2, 60, 160, 4.5), (6, 2, 70, 159, 3.0)])
def test_eigvecs_edges(ns, nt, nv, m, lamc):
    import torch

    import paper_1104_3870_amd as P

    say("eig edges", ns, nt, nv, m)
    U = synth.gauge_field(ns, nt, 0.5, 7)
    S = oracle.stout_spatial(U, 0.1, 2)
    ev_ref, V_ref = oracle.laph_eigpairs(S, nv + 1)
    L = P.Lattice(ns, nt)
    evals = np.zeros((nt, nv))
    evecs = torch.empty((nt, nv, ns, ns, ns, 3), dtype=torch.complex128, device="cuda")
    st = P.laph_eigvecs(L.ctx, dev(U), 0.1, 2, nv, evals, evecs, krylov=m, lam_c=lamc, tol=1e-12, max_restarts=200)
    say("  restarts", st.restarts, "max_res", st.max_residual, "orth", st.max_orth)
    assert st.max_residual < 1e-10 and st.max_orth < 1e-12
    V = host(evecs)
    assert np.abs(evals - ev_ref[:, :nv]).max() < 1e-11
    for t in range(nt):
        gap = np.diff(ev_ref[t])
        for n in range(nv):
            if min(gap[n], gap[n - 1] if n else gap[n]) > 1e-4:
                assert np.linalg.norm(V[t, n] - V_ref[t, n]) < 1e-6, (t, n)
