"""Lengths whose tiles fill a workgroup's LDS to the last bytes: they are launched, with the results
of any other length (operator: numpy's FFT, 1e-12 relative; solves: the oracle's iterate, 1e-9)."""
import numpy as np
import pytest
import torch

from paper_1508_02045_amd import fgh, inputs
from test_gpu_lengths import reference

pytestmark = pytest.mark.gpu


def _grid(N):
    rng = np.random.default_rng(sum(N))
    phase = (rng.random(N) < 0.3).astype(np.uint8)
    return phase, inputs.iso_tables(len(N), [1.0, 10.0]), rng.standard_normal((len(N),) + N)


# rows of 3381 = 7 x 483 and 1449 = 3 x 483 points (dense step); a strided pass of 3413 points (prime, mixed radix)
@pytest.mark.parametrize("N", [(3, 3381), (45, 45, 1449), (3, 3413, 3)])
def test_apply_full_tile(N):
    phase, tables, x = _grid(N)
    plan = fgh.Plan(N, phase=torch.from_numpy(phase).cuda(), phase_table=inputs.sym_pack(tables).T)
    print(N, "apply", flush=True)
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.close()
    ref = reference(inputs.phase_to_full(phase, tables), x, N, N)
    assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("solver,N,bodies", [("cg", (3, 3381), 5), ("richardson", (3, 3381), 5), ("cg", (3, 3413, 3), 1)])
def test_loop_full_tile(solver, N, bodies):
    from oracle import orc

    d = len(N)
    phase, tables, _ = _grid(N)
    plan = fgh.Plan(N, phase=torch.from_numpy(phase).cuda(), phase_table=inputs.sym_pack(tables).T, c_A=1.0, C_A=10.0)
    E = np.eye(d)[0]
    print(N, solver, flush=True)
    e, st, stats = plan.solve_fixed(solver, E, bodies)
    assert st == fgh.FGH_OK and stats[0]["iters"] == bodies
    ref = orc.solve(N, orc.GANI, inputs.phase_to_full(phase, tables), E, solver, 1.0, 10.0, 1e-8, fixed_iters=bodies)
    full = np.linalg.norm(ref.e + E.reshape((d,) + (1,) * d))
    assert np.linalg.norm(e.cpu().numpy() - ref.e) <= 1e-9 * full
    plan.close()
