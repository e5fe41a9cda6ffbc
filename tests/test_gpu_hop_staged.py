"""The FP64 hop of 8, 16 and 32 right-hand sides (links and clover staged per block of sites)
against the same fields applied one at a time by the kernel of small launches: whole and ragged
last blocks of sites, tiles of the site walk of 6, 4 and 2, all epilogues.

Bound: both kernels add the eight directions in the same order and differ at most in how the
compiler contracts products, a few roundings of terms of order one per component."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

BOUND = 64 * 2.0 ** -53


def _setup(ns, nt, R):
    import paper_1104_3870_amd as P

    rng = np.random.default_rng(ns * R)
    f = [dev(rng.standard_normal((R, nt, ns, ns, ns, 4, 3)) + 1j * rng.standard_normal((R, nt, ns, ns, ns, 4, 3)))
         for _ in range(2)]
    return P, P.Lattice(ns, nt), dev(synth.gauge_field(ns, nt, 0.4, 3)), P.laph_dirac(-0.1, 3.5, 1.0, -1.0), f


def _close(a, b):
    scale = max(1.0, float(np.abs(b).max()))
    assert np.abs(a - b).max() <= BOUND * scale


@pytest.mark.parametrize("ns,nt,R", [(6, 38, 8), (6, 22, 16), (6, 10, 32), (8, 18, 8), (10, 4, 32), (2, 260, 32)])
def test_dirac_staged(ns, nt, R):
    import torch

    P, L, U, d, (x, _) = _setup(ns, nt, R)
    say("staged hop", ns, nt, R)
    for op in (P.LAPH_OP_K, P.LAPH_OP_KDAG):
        big, one = torch.empty_like(x), torch.empty_like(x[:1])
        P.laph_dirac_apply(L.ctx, U, d, op, x, big, R)
        for r in (0, 3, R - 1):
            P.laph_dirac_apply(L.ctx, U, d, op, x[r:r + 1].contiguous(), one, 1)
            _close(host(big[r:r + 1]), host(one))
    L.close()


@pytest.mark.parametrize("mode", ["plain", "inv"])
@pytest.mark.parametrize("parity", [0, 1])
@pytest.mark.parametrize("addend", [False, True])
def test_hop_staged(mode, parity, addend):
    import torch

    P, L, U, d, f = _setup(6, 22, 16)
    say("staged hop launch", mode, parity, addend)
    m = P.LAPH_HOP_PLAIN if mode == "plain" else P.LAPH_HOP_INV
    kw = dict(a=0.7, c=-1.3, gamma5=1)
    big, one = torch.empty_like(f[0]), torch.empty_like(f[0][:1])
    P.laph_hop_apply(L.ctx, U, d, "f64", m, parity, f[0], big, x=f[1] if addend else None, **kw)
    for r in (0, 15):
        P.laph_hop_apply(L.ctx, U, d, "f64", m, parity, f[0][r:r + 1].contiguous(), one,
                         x=f[1][r:r + 1].contiguous() if addend else None, **kw)
        _close(host(big[r:r + 1]), host(one))
    L.close()
