"""Laplacian and Chebyshev step on many small slices, where a workgroup's sites come from several
of them and the last one is ragged, and on either side of the 768 workgroups up to which three
lanes work on a site, against the oracle.

Bound: a component is a sum of 19 products of unit-size links with field values; 64 roundings of
the largest value a step can reach (12 times the field's) covers it."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nt", [(2, 8202), (4, 770), (6, 202), (10, 50), (2, 768),
                                   (2, 770), (12, 28), (16, 12), (14, 18)])
def test_many_slices(ns, nt):
    import torch

    import paper_1104_3870_amd as P

    say("laplacian slices", ns, nt)
    rng = np.random.default_rng(ns + nt)
    U = synth.gauge_field(ns, nt, 0.5, 7)
    v = rng.normal(size=(nt, ns, ns, ns, 3)) + 1j * rng.normal(size=(nt, ns, ns, ns, 3))
    L = P.Lattice(ns, nt)
    out = torch.empty(v.shape, dtype=torch.complex128, device="cuda")
    size = np.abs(v).max()
    P.laph_laplacian_apply(L.ctx, dev(U), dev(v), out)
    assert np.abs(host(out) - oracle.laplacian(U, v)).max() <= 64 * 2.0 ** -53 * 12 * size
    lam_l, lam_c = 15.0, 0.5
    c = 2.0 / (lam_l - lam_c)
    B = lambda a: a + c * (oracle.laplacian(U, a) + lam_c * a)  # noqa: E731
    P.laph_chebyshev_apply(L.ctx, dev(U), lam_l, lam_c, 2, dev(v), out)
    assert np.abs(host(out) - (2 * B(B(v)) - v)).max() <= 64 * 2.0 ** -53 * 2 * (1 + 12 * c) ** 2 * 3 * size
    L.close()
