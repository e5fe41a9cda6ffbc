"""The FP64 hop of small launches (one wave per direction) against the same hop inside a
batch large enough for the other kernel: same field, all parities, epilogues and operators,
field counts that are no power of two, a ragged last workgroup.

Bound: both kernels add the eight directions in the same order and differ at most in how the
compiler contracts products, a few roundings of terms of order one per component."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

BOUND = 64 * 2.0 ** -53


def _close(a, b):
    scale = max(1.0, float(np.abs(b).max()))
    assert np.abs(a - b).max() <= BOUND * scale


@pytest.mark.parametrize("ns,nt,few,many", [(4, 8, 1, 160), (4, 6, 3, 192), (6, 4, 5, 90), (12, 16, 1, 4),
                                            (12, 16, 2, 3)])
def test_dirac_split_matches_batch(ns, nt, few, many):
    import torch

    import paper_1104_3870_amd as P

    say("split hop", ns, nt, few, many)
    U = dev(synth.gauge_field(ns, nt, 0.4, 3))
    rng = np.random.default_rng(5)
    x = dev(rng.standard_normal((many, nt, ns, ns, ns, 4, 3)) + 1j * rng.standard_normal((many, nt, ns, ns, ns, 4, 3)))
    L = P.Lattice(ns, nt)
    d = P.laph_dirac(-0.1, 3.5, 1.0, -1.0)
    for op in (P.LAPH_OP_K, P.LAPH_OP_OMEGA, P.LAPH_OP_KDAG):
        big, small = torch.empty_like(x), torch.empty_like(x[:few])
        # batches of 32 fields: the last one of `many` is whole
        P.laph_dirac_apply(L.ctx, U, d, op, x, big, many)
        P.laph_dirac_apply(L.ctx, U, d, op, x[:few].contiguous(), small, few)
        _close(host(small), host(big[:few]))


@pytest.mark.parametrize("mode", ["plain", "inv"])
@pytest.mark.parametrize("parity", [0, 1])
@pytest.mark.parametrize("addend", [False, True])
def test_hop_split_matches_batch(mode, parity, addend):
    import torch

    import paper_1104_3870_amd as P

    ns, nt, many = 12, 16, 4
    say("split hop launch", mode, parity, addend)
    U = dev(synth.gauge_field(ns, nt, 0.4, 4))
    rng = np.random.default_rng(6)
    f = [dev(rng.standard_normal((many, nt, ns, ns, ns, 4, 3)) + 1j * rng.standard_normal((many, nt, ns, ns, ns, 4, 3)))
         for _ in range(2)]
    L = P.Lattice(ns, nt)
    d = P.laph_dirac(-0.1, 3.5, 1.0, -1.0)
    m = P.LAPH_HOP_PLAIN if mode == "plain" else P.LAPH_HOP_INV
    big = torch.empty_like(f[0])
    kw = dict(a=0.7, c=-1.3, gamma5=1)
    P.laph_hop_apply(L.ctx, U, d, "f64", m, parity, f[0], big, x=f[1] if addend else None, **kw)
    for n in (1, 2):
        small = torch.empty_like(f[0][:n])
        P.laph_hop_apply(L.ctx, U, d, "f64", m, parity, f[0][:n].contiguous(), small,
                         x=f[1][:n].contiguous() if addend else None, **kw)
        _close(host(small), host(big[:n]))
