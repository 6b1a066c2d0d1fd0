"""Operator applications at lengths without a specialised kernel: products of two register radices,
dense steps (prime and composite), lengths around the edges of their tiles, in every pass position.

Reference: G A x by numpy's FFT in double precision.  Tolerances: the operator parity tolerances of
test_gpu_parity.py (1e-12 in FP64 and 2e-6 in FP32, relative L2); a dense step of p points sums
(p + 1) / 2 products, whose rounding stays below p / 2 ulps (1e-13 at p = 1021, FP64; 6e-5 at worst
and about sqrt(p / 2) ulps = 1.4e-6 in practice in FP32)."""
import numpy as np
import pytest
import torch

from paper_1508_02045_amd import fgh, inputs

pytestmark = pytest.mark.gpu


def reference(A, x, N, grid):
    """G A x on `grid` with the band N: A [*grid, d, d], x [d, *grid]."""
    d = len(grid)
    z = np.einsum("...ij,j...->i...", A, x)
    k = []
    for a in range(d):
        f = np.round(np.fft.fftfreq(grid[a]) * grid[a])
        shape = [1] * d
        shape[a] = grid[a]
        k.append(f.reshape(shape))
    kk = sum(f * f for f in k)
    w = np.where(kk > 0, 1.0 / np.where(kk > 0, kk, 1.0), 0.0)
    for f, n in zip(k, N):
        w = w * (2 * np.abs(f) < n)
    axes = tuple(range(1, d + 1))
    Z = np.fft.fftn(z, axes=axes)
    t = sum(k[c] * Z[c] for c in range(d)) * w
    return np.real(np.fft.ifftn(np.stack([k[c] * t for c in range(d)]), axes=axes))


def spd(N, rng):
    d = len(N)
    v = rng.standard_normal(tuple(N) + (d,))
    return np.einsum("...i,...j->...ij", v, v) + (1.0 + rng.random(N))[..., None, None] * np.eye(d)


# register pairs (3 .. 17 x 17), dense primes around multiples of 16 rows and of 4 terms, dense
# composites, 1 to 32 dense products per workgroup
GRIDS_2D = [(3, 3), (5, 17), (15, 27), (17, 9), (19, 21), (23, 29), (31, 33), (35, 37), (61, 67), (85, 169), (99, 101),
            (127, 129), (255, 289), (343, 51), (511, 509), (767, 221), (729, 25), (1023, 13), (13, 1023), (1021, 19),
            (19, 1021), (1033, 7), (7, 1369)]
GRIDS_3D = [(3, 5, 7), (17, 19, 21), (23, 15, 13), (33, 31, 29), (51, 85, 35), (67, 65, 9), (9, 101, 55), (89, 45, 17),
            (17, 201, 15), (15, 11, 255), (255, 7, 9), (45, 77, 63), (25, 27, 23), (5, 1021, 3), (289, 3, 5)]


@pytest.mark.parametrize("N", GRIDS_2D + GRIDS_3D)
@pytest.mark.parametrize("kind", ["sym", "iso", "phase"])
def test_apply_any_length(N, kind):
    rng = np.random.default_rng(sum(N))
    d = len(N)
    if kind == "phase":
        phase = rng.integers(0, 3, size=N).astype(np.uint8)
        tables = [spd((1,) * d, rng).reshape(d, d) for _ in range(3)]
        A = inputs.phase_to_full(phase, tables)
        tab = np.stack([inputs.sym_pack(t[None])[:, 0] for t in tables])
        kw = dict(phase=torch.from_numpy(phase).cuda(), phase_table=tab)
    elif kind == "iso":
        a = 1.0 + rng.random(N)
        A = a[..., None, None] * np.eye(d)
        kw = dict(A=torch.from_numpy(a).cuda())
    else:
        A = spd(N, rng)
        kw = dict(A=torch.from_numpy(inputs.sym_pack(A)).cuda())
    x = rng.standard_normal((d,) + N)
    ref = reference(A, x, N, N)
    plan = fgh.Plan(N, precision=fgh.FGH_FP32_REFINED, **kw)
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    y32 = plan.apply(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy()
    ref32 = reference(A, x.astype(np.float32).astype(np.float64), N, N)
    err32 = np.linalg.norm(y32 - ref32) / np.linalg.norm(ref32)
    print(N, kind, f"fp64 {err:.2e} fp32 {err32:.2e}", flush=True)
    plan.close()
    assert err <= 1e-12 and err32 <= 2e-6


@pytest.mark.parametrize("N", [(9, 11), (27, 45), (51, 61), (85, 85), (255, 21), (9, 11, 13), (17, 21, 45), (41, 23, 33)])
def test_apply_double_grid_any_length(N):
    """Band-limited passes (exact integration, grid 2N - 1) against the same reference."""
    rng = np.random.default_rng(sum(N))
    d = len(N)
    a = 1.0 + rng.random(N)
    plan = fgh.Plan(N, rule=fgh.FGH_GA, precision=fgh.FGH_FP32_REFINED, A=torch.from_numpy(a).cuda())
    A = plan.ga_coefficients().cpu().numpy()[0][..., None, None] * np.eye(d)
    x = rng.standard_normal((d,) + plan.grid)
    ref = reference(A, x, N, plan.grid)
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    y32 = plan.apply(torch.from_numpy(x.astype(np.float32)).cuda()).cpu().numpy()
    err32 = np.linalg.norm(y32 - ref) / np.linalg.norm(ref)
    print(N, f"fp64 {err:.2e} fp32 {err32:.2e}", flush=True)
    plan.close()
    assert err <= 1e-12 and err32 <= 2e-6


@pytest.mark.parametrize("N", [(51, 85), (61, 45), (33, 97), (17, 15, 19), (27, 35, 23), (37, 9, 21)])
@pytest.mark.parametrize("solver", ["richardson", "cg", "chebyshev", "eyre_milton"])
def test_solvers_any_length(N, solver):
    """Every solver's epilogue and multiplier at such lengths: iterates after a fixed count against
    the oracle's (the tolerance of the iterate-matched parity tests)."""
    from oracle import orc

    d = len(N)
    phase = inputs.paper_square(N)
    tab = inputs.sym_pack(inputs.iso_tables(d, [1.0, 10.0])).T
    plan = fgh.Plan(N, phase=torch.from_numpy(phase).cuda(), phase_table=tab, c_A=1.0, C_A=10.0)
    E = np.eye(d)[0]
    e, st, stats = plan.solve_fixed(solver, E, 7)
    A = inputs.phase_to_full(phase, inputs.iso_tables(d, [1.0, 10.0]))
    ref = orc.solve(N, orc.GANI, A, E, solver, 1.0, 10.0, 1e-8, fixed_iters=7)
    diff = np.linalg.norm(e.cpu().numpy() - ref.e) / np.linalg.norm(ref.e + E.reshape((d,) + (1,) * d))
    plan.close()
    assert diff <= 1e-9


@pytest.mark.parametrize("N,rule", [((85, 33), 0), ((81, 169), 0), ((35, 105), 0), ((61, 13), 0), ((2187, 3), 0), ((2401, 3), 0),
                                    ((27, 11), 1), ((21, 15, 27), 0), ((17, 49, 11), 0),
                                    ((9, 75, 25), 0), ((11, 9, 13), 1)])
@pytest.mark.parametrize("solver", ["cg", "eyre_milton", "chebyshev"])
def test_refined_solves_any_length(N, rule, solver):
    """Refined solves (mixed-radix passes: paired radices, direct sums spread over a workgroup, all
    components in one transform or one after the other) against the FP64 solve of the same problem
    (run-time-length passes).  Both stop on a residual (step) of 1e-9 relative; the solutions then
    differ by at most that times the condition number 10, with a factor 10 in hand: 1e-7."""
    if solver == "eyre_milton" and rule == 1:
        pytest.skip("Eyre-Milton has no exact-integration form")
    d = len(N)
    phase = torch.from_numpy(inputs.paper_square(N)).cuda()
    tab = inputs.sym_pack(inputs.iso_tables(d, [1.0, 10.0])).T
    E = np.eye(d)[d - 1]
    e = []
    for prec in (fgh.FGH_FP64, fgh.FGH_FP32_REFINED):
        plan = fgh.Plan(N, rule=rule, precision=prec, phase=phase, phase_table=tab)
        x, st, stats = plan.solve(solver, E, 1e-9)
        assert st == fgh.FGH_OK
        e.append(x.cpu().numpy())
        plan.close()
    full = np.linalg.norm(e[0] + E.reshape((d,) + (1,) * d))
    assert np.linalg.norm(e[0] - e[1]) <= 1e-7 * full


@pytest.mark.parametrize("N,rule", [((51, 85), 0), ((33, 97), 0), ((85, 85), 1), ((17, 15, 19), 0), ((37, 9, 21), 0),
                                    ((9, 11, 13), 1)])
@pytest.mark.parametrize("solver", ["richardson", "chebyshev", "eyre_milton"])
def test_fused_bodies_any_length(N, rule, solver, monkeypatch):
    """The last pass fused with the next body's first (run-time lengths) against the separate passes
    (FGH_FUSE=0): the same operations on the same values, so a product contracted differently by
    the compiler is all that may differ -- 7 bodies of a contraction, 1e-13 of the field."""
    if solver == "eyre_milton" and rule == 1:
        pytest.skip("Eyre-Milton has no exact-integration form")
    d = len(N)
    rng = np.random.default_rng(sum(N))
    A = torch.from_numpy(1.0 + 9.0 * rng.random(N)).cuda()
    plan = fgh.Plan(N, rule=rule, A=A)
    e = []
    for on in ("0", "1"):
        monkeypatch.setenv("FGH_FUSE", on)
        x, st, stats = plan.solve_fixed(solver, np.eye(d)[0], 7)
        assert st == fgh.FGH_OK and stats[0]["iters"] == 7
        e.append(x.cpu().numpy())
    plan.close()
    assert np.linalg.norm(e[0] - e[1]) <= 1e-13 * np.sqrt(e[0][0].size)


@pytest.mark.parametrize("N", [(93, 3), (999, 257), (1023, 1021), (1023, 1023)])
def test_apply_few_columns(N):
    """The dense middle pass where its columns cannot give each unit two workgroups (fewer than 512),
    from two columns to the first count above that."""
    test_apply_any_length(N, "phase")
