"""The batched FP64 products at the edges of their tiles: momentum overlaps of 1 to 129 vectors
(tiles of 16 in workgroup tiles of 64) and baryon functions whose N_v is below, at and past the
staged K tile, with line counts that leave ragged tiles, against numpy.

Bound: an entry is a sum of K products, so two orders of summation differ by at most
about K 2^-52 times the sum of absolute values (three such sums in a row for the baryon
functions)."""
import numpy as np
import pytest

from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

U = 2.0 ** -52


def _c(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


@pytest.mark.parametrize("ns,nt,na,nb", [(2, 2, 1, 1), (2, 8, 17, 64), (2, 3 * 2, 48, 49), (4, 4, 65, 3),
                                         (2, 2, 129, 112), (4, 2, 16, 128)])
def test_overlap_edges(ns, nt, na, nb):
    import torch

    import paper_1104_3870_amd as P

    say("overlap", ns, nt, na, nb)
    rng = np.random.default_rng(na * 1000 + nb)
    a, b = _c(rng, nt, na, ns, ns, ns, 3), _c(rng, nt, nb, ns, ns, ns, 3)
    out = torch.empty((nt, na, nb), dtype=torch.complex128, device="cuda")
    L = P.Lattice(ns, nt)
    k = (1, 0, 1)
    P.laph_mom_overlap(L.ctx, dev(a), na, dev(b), nb, k, out)
    x = np.arange(ns)
    ph = np.exp(-2j * np.pi / ns * (k[2] * x[:, None, None] + k[1] * x[None, :, None] + k[0] * x[None, None, :]))
    ref = np.conj(a.reshape(nt, na, -1)) @ (ph[..., None] * b).reshape(nt, nb, -1).transpose(0, 2, 1)
    size = np.abs(a).reshape(nt, na, -1) @ np.abs(b).reshape(nt, nb, -1).transpose(0, 2, 1)
    assert (np.abs(host(out) - ref) <= 3 * ns ** 3 * U * size).all()


@pytest.mark.parametrize("nt,nv,n1,n2,n3", [(2, 1, 1, 1, 1), (4, 3, 2, 1, 5), (2, 8, 4, 4, 4), (2, 9, 1, 17, 3),
                                            (2, 16, 16, 2, 33), (4, 23, 5, 4, 20)])
def test_baryon_function_edges(nt, nv, n1, n2, n3):
    import torch

    import paper_1104_3870_amd as P

    say("baryon function", nt, nv, n1, n2, n3)
    rng = np.random.default_rng(nv)
    T = _c(rng, nt, nv, nv, nv)
    f = [_c(rng, n, nt, 4, nv) for n in (n1, n2, n3)]
    c = np.zeros((4, 4, 4), dtype=np.complex128)
    c[0, 1, 0], c[1, 0, 0], c[3, 2, 1] = 1.0, -1.0, 0.5j
    out = torch.empty((nt, n1, n2, n3), dtype=torch.complex128, device="cuda")
    L = P.Lattice(2, nt)
    P.laph_baryon_function(L.ctx, dev(T), nv, c, dev(f[0]), n1, dev(f[1]), n2, dev(f[2]), n3, out)

    def full(T, f, c):
        X = np.einsum("tabc,ktgc->tabkg", T, f[2], optimize=True)
        Y = np.einsum("jtbn,tankg->tajbkg", f[1], X, optimize=True)
        return np.einsum("abg,itan,tnjbkg->tijk", c, f[0], Y, optimize=True)

    ref, size = full(T, f, c), full(np.abs(T), [np.abs(v) for v in f], np.abs(c))
    assert (np.abs(host(out) - ref) <= 3 * (nv + 8) * U * size).all()
