"""Solves at the edges of their reductions, judged by the true residual of the FP64 operator.
Low precision: from less than one block of partial sums to 1024 blocks (taken in one stage) and
past them (two stages).  FP64 BiCGStab: partial sums taken by the vector passes themselves, from
the split and from the rolled hop, with ragged last blocks, up to and past their largest number.

Bound: the solver stops on its own FP64 residual of 1e-10, so an independent evaluation can
exceed it by that evaluation's rounding only; twice the target covers it."""
import pytest

import synth
from gpu_util import dev, say

pytestmark = pytest.mark.gpu


LOW = [(4, 4, 1, "f16"), (4, 2, 32, "f32"), (6, 4, 4, "bf16"), (16, 4, 32, "f16"), (16, 6, 32, "f16")]
FP64 = [(4, 2, 1, "f64"), (4, 2, 16, "f64"), (4, 2, 32, "f64"), (6, 10, 1, "f64"), (6, 10, 4, "f64"),
        (16, 16, 1, "f64"), (16, 18, 1, "f64"), (12, 20, 2, "f64")]


@pytest.mark.parametrize("ns,nt,R,prec,solver", [(*c, "bicgstab") for c in LOW + FP64] + [(*c, "cgnr") for c in LOW])
def test_solve_reduction_edges(ns, nt, R, prec, solver):
    import torch

    import paper_1104_3870_amd as P

    say("solve", ns, nt, R, prec, solver)
    kind = P.LAPH_SOLVER_BICGSTAB if solver == "bicgstab" else P.LAPH_SOLVER_CGNR
    L = P.Lattice(ns, nt)
    U = dev(synth.gauge_field(ns, nt, 0.3, ns + nt))
    D = P.laph_dirac(0.2, 3.5, 1.0, -1.0)
    g = torch.Generator(device="cuda").manual_seed(R)
    shape = (R, nt, ns, ns, ns, 4, 3)
    eta = torch.view_as_complex(torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=g))
    x, back = torch.empty_like(eta), torch.empty_like(eta)
    P.dirac_solve(L.ctx, U, D, eta, x, R, P.solver_params(tol=1e-10, maxiter=2000, precision=prec, solver=kind,
                                                         block_rhs=R))
    P.laph_dirac_apply(L.ctx, U, D, P.LAPH_OP_OMEGA, x, back, R)
    rel = (back - eta).reshape(R, -1).norm(dim=1) / eta.reshape(R, -1).norm(dim=1)
    assert (rel <= 2e-10).all(), rel
    L.close()
