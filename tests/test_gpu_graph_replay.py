"""use_graph replays an iteration's launches from HIP graphs: counted by the library's own
report (LAPH_VERBOSE, read once per process, hence a process of its own) for BiCGStab and CG
in low precision and CG in FP64, and none without use_graph or with timing on.  The solutions
and iteration counts are the same bits either way."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

PROGRAM = """
import sys
import torch
import paper_1104_3870_amd as P
import synth

L = P.Lattice(4, 8)
U = torch.from_numpy(synth.gauge_field(4, 8, 0.3, 3)).cuda()
D = P.laph_dirac(0.1, 3.5, 1.0, -1.0)
eta = torch.from_numpy(synth.random_spinor(4, 8, 5, nrhs=3)).cuda()
for prec, solver in (("f16", 0), ("f32", 1), ("f64", 1)):
    got = []
    for graph, timing in ((0, 0), (1, 0), (1, 1), (1, 0)):
        print("run", prec, solver, graph, timing, file=sys.stderr, flush=True)
        x = torch.zeros_like(eta)
        P.laph_set_timing(L.ctx, bool(timing))
        st = P.dirac_solve(L.ctx, U, D, eta, x, 3, P.solver_params(precision=prec, solver=solver, block_rhs=4,
                                                                   use_graph=graph))
        torch.cuda.synchronize()
        assert all(q.status == 0 and q.fallback_used == 0 for q in st)
        got.append((x, [q.iters for q in st]))
    assert all(torch.equal(got[0][0], g[0]) and got[0][1] == g[1] for g in got), (prec, solver)
L.close()
"""


def test_graph_replays():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, LAPH_VERBOSE="1", PYTHONPATH=root)
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=root, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-4000:]
    runs = re.split(r"^run (\w+ \d \d \d)$", r.stderr, flags=re.M)[1:]
    assert len(runs) == 24
    for what, log in zip(runs[::2], runs[1::2]):
        prec, solver, graph, timing = what.split()
        n = sum(int(q) for q in re.findall(r"graph replays (\d+)", log))
        print(what, "replays", n, flush=True)
        assert (n > 8) if graph == "1" and timing == "0" else n == 0, (what, log)
