"""Covariant displacements where a wave's 64 sites straddle time slices or run past the last
site, and where the vector count leaves a remainder of the four in flight, against the oracle.

Bound: a component is three products of a unitary link product with the far site; each
rounding is 2^-53 of a term, some 20 per link and 10 for the last product."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt,n", [(2, 2, 1), (2, 10, 4), (6, 2, 3), (6, 4, 9), (10, 2, 2)])
def test_displace_edges(ns, nt, n):
    import torch

    import paper_1104_3870_amd as P

    rng = np.random.default_rng(100 * ns + n)
    U = synth.gauge_field(ns, nt, 0.6, ns + n)
    v = rng.normal(size=(nt, n, ns, ns, ns, 3)) + 1j * rng.normal(size=(nt, n, ns, ns, ns, 3))
    L = P.Lattice(ns, nt)
    guard = torch.full((v.size + 256,), 7.0, dtype=torch.complex128, device="cuda")
    out = guard[:v.size].view(v.shape)
    for d in range(3):
        for s, ln in ((1, 0), (1, 1), (-1, 2), (-1, 3)):
            say("displace", ns, nt, n, d, s, ln)
            P.laph_displace(L.ctx, dev(U), d, s, ln, dev(v), n, out)
            ref = oracle.displace_evecs(U, v, d, s, ln)
            assert np.abs(host(out) - ref).max() <= (20 * ln + 10) * 2.0 ** -53 * 3 * np.abs(v).max(), (d, s, ln)
    assert (guard[v.size:] == 7.0).all()
    L.close()
