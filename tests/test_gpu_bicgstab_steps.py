"""FP64 BiCGStab iteration by iteration against the same iteration in numpy on the oracle's
operator: the target is set between the residuals of iterations k - 1 and k, so that the answer
is the iterate after exactly k steps.  Its alpha, omega and beta are the inner products the
hops sum in their epilogues (split hop up to 32768 pairs, rolled above), so a partial sum lost,
taken twice, conjugated or given to the wrong right-hand side moves the answer at once, where a
solve to convergence would only take more iterations.  Sizes: ragged last blocks, one to 32
right-hand sides, sums at and past the 1280 that the vector passes take themselves.

Bound: with the mass 1 the operator's condition is below 6 and a step a few dozen products and
two inner products, whose rounding (12 Vh terms, summed in a tree on one side) stays below
1e-14 of their size; three steps amplify it by less than 100."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

M0, XI, CSW, BC = 1.0, 3.5, 1.0, -1.0
BOUND = 1e-12


class EvenOdd:
    def __init__(self, ns, nt):
        self.U = synth.gauge_field(ns, nt, 0.4, 100 * ns + nt)
        self.D = oracle.Dirac(self.U, M0, XI, CSW, BC)
        self.Ainv = np.linalg.inv(self.D.A)
        t, z, y, x = np.meshgrid(*(np.arange(n) for n in (nt, ns, ns, ns)), indexing="ij")
        self.even = ((x + y + z + t) % 2 == 0)[..., None, None]

    def ainv(self, v):
        return (self.Ainv @ v.reshape(v.shape[:-2] + (12, 1))).reshape(v.shape)

    def hop(self, v, even):
        """H v on the even (odd) sites, v living on the other ones."""
        return np.where(self.even == even, self.D.K(v), 0)

    def mhat(self, v):
        return v - self.ainv(self.hop(self.ainv(self.hop(v, True)), False))

    def rhs(self, eta):
        b = np.einsum("ab,...bc->...ac", oracle.gamma(3), eta)
        be, bo = np.where(self.even, b, 0), np.where(self.even, 0, b)
        return be, self.ainv(bo - self.hop(self.ainv(be), False))

    def full(self, be, xo):
        return xo + self.ainv(be - self.hop(xo, True))


def _iterates(E, eta, steps):
    """[x after k steps of BiCGStab] and [|r| / |bhat|], k = 0 .. steps."""
    be, bhat = E.rhs(eta)
    x, r = np.zeros_like(bhat), bhat.copy()
    r0, p, rho = r.copy(), r.copy(), np.vdot(r, r)
    xs, res = [x], [1.0]
    for _ in range(steps):
        v = E.mhat(p)
        alpha = rho / np.vdot(r0, v)
        s = r - alpha * v
        t = E.mhat(s)
        omega = np.vdot(t, s) / np.vdot(t, t)
        x = x + alpha * p + omega * s
        r = s - omega * t
        new = np.vdot(r0, r)
        p = r + (new / rho) * (alpha / omega) * (p - omega * v)
        rho = new
        xs.append(E.full(be, x))
        res.append(np.linalg.norm(r) / np.linalg.norm(bhat))
    return xs, res


# (ns, nt, R): pairs 48 (one ragged block), 64, 2048 (1280 sums), 4096 (2048 sums: taken by
# kernels of their own), 4320 (ragged, R = 4); above 32768 pairs 32928 and 33696 (ragged), 34560
@pytest.mark.parametrize("ns,nt,R", [(2, 12, 1), (2, 6, 2), (4, 2, 1), (4, 2, 32), (4, 4, 32), (6, 10, 4), (14, 24, 1),
                                     (6, 78, 4), (12, 20, 2)])
def test_iterates(ns, nt, R):
    import torch

    import paper_1104_3870_amd as P

    say("bicgstab steps", ns, nt, R)
    E = EvenOdd(ns, nt)
    etas = synth.random_spinor(ns, nt, 7 + R, nrhs=R)
    steps = 3
    ref = [_iterates(E, e, steps) for e in etas]
    L = P.Lattice(ns, nt)
    U, D = dev(E.U), P.laph_dirac(M0, XI, CSW, BC)
    x = torch.empty(etas.shape, dtype=torch.complex128, device="cuda")
    for k in range(1, steps + 1):
        above, below = min(r[1][k - 1] for r in ref), max(r[1][k] for r in ref)
        assert below < 0.9 * above, (above, below)
        # the even-odd target is half of tol
        st = P.dirac_solve(L.ctx, U, D, dev(etas), x, R, P.solver_params(tol=2 * np.sqrt(above * below), block_rhs=R))
        got = host(x)
        for r in range(R):
            assert (st[r].status, st[r].fallback_used, st[r].iters) == (0, 0, k), (r, k, st[r].iters)
            want = ref[r][0][k]
            err = np.linalg.norm(got[r] - want) / np.linalg.norm(want)
            assert err <= BOUND, (r, k, err)
    L.close()


@pytest.mark.parametrize("solver", ["bicgstab", "cgnr"])
@pytest.mark.parametrize("ns,nt,R,prec", [(4, 4, 1, "f16"), (4, 2, 32, "f32"), (6, 4, 4, "bf16"), (16, 4, 32, "f16"),
                                          (16, 6, 32, "f16")])
def test_low_precision_counts(ns, nt, R, prec, solver):
    """The low-precision sums, from one block to past 1024 (one and two stages), judged by what a
    wrong scalar costs: no fallback and no more iterations than FP64 takes on the same sources,
    plus half of them (BF16 drifts) and eight (updates wait for the block and lag by one)."""
    import torch

    import paper_1104_3870_amd as P

    say("counts", ns, nt, R, prec, solver)
    kind = P.LAPH_SOLVER_BICGSTAB if solver == "bicgstab" else P.LAPH_SOLVER_CGNR
    L = P.Lattice(ns, nt)
    U, D = dev(synth.gauge_field(ns, nt, 0.3, ns + nt)), P.laph_dirac(0.2, XI, CSW, BC)
    eta = dev(synth.random_spinor(ns, nt, R, nrhs=R))
    x, its = torch.empty_like(eta), {}
    for p in ("f64", prec):
        st = P.dirac_solve(L.ctx, U, D, eta, x, R, P.solver_params(tol=1e-10, maxiter=2000, precision=p, solver=kind,
                                                                  block_rhs=R))
        assert all((q.status, q.fallback_used) == (0, 0) for q in st), p
        its[p] = [q.iters for q in st]
    say("  iters", its["f64"][:4], its[prec][:4])
    assert all(a <= 1.5 * b + 8 for a, b in zip(its[prec], its["f64"])), its
    L.close()
