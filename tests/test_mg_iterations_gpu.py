"""Iterations of the multigrid-preconditioned solves (velocity, energy) at two
step sizes: those of a V-cycle run launch by launch on every level, within one (a
fiftieth of the long ones).  A wrong weight, level or sweep of the coarse levels
shows here before it shows in the converged solution."""
import pytest

from paper_2106_02159_amd import abi, workloads as W

pytestmark = pytest.mark.gpu

# nodes, periodic, iterations at dt = 5e-3 (velocity, energy) and at dt = 1
CASES = [((33, 33), (0, 0), (7, 7, 16, 18)), ((64, 64), (0, 0), (8, 7, 16, 17)),
         ((64, 64), (1, 0), (8, 7, 18, 17)), ((65, 64), (0, 1), (8, 7, 18, 17)),
         ((90, 77), (1, 1), (9, 8, 28, 18)), ((200, 150), (0, 0), (9, 8, 13, 15)),
         ((501, 400), (0, 0), (9, 9, 15, 18)), ((1365, 3), (0, 0), (9, 99, 10, 218)),
         ((1366, 3), (0, 0), (9, 101, 10, 216)), ((500, 9), (1, 0), (9, 22, 11, 42)),
         ((12, 12, 12), (0, 0, 0), (6, 6, 8, 10)), ((16, 8, 16), (1, 0, 1), (7, 7, 9, 11)),
         ((25, 5, 16), (0, 0, 0), (7, 7, 9, 14)), ((26, 5, 16), (0, 0, 0), (7, 7, 9, 14)),
         ((16, 8, 8), (0, 0, 0), (7, 6, 8, 10)), ((15, 9, 8), (0, 0, 0), (7, 6, 8, 11)),
         ((8, 16, 8), (1, 0, 1), (7, 7, 12, 11)), ((10, 11, 10), (0, 1, 0), (6, 6, 9, 9)),
         ((24, 24, 24), (0, 0, 0), (7, 7, 9, 9)), ((24, 24, 24), (1, 1, 1), (7, 7, 12, 11)),
         ((31, 17, 45), (0, 1, 0), (8, 7, 12, 13)), ((48, 48, 48), (0, 0, 0), (8, 7, 10, 11))]


@pytest.mark.parametrize("n,per,its", CASES, ids=lambda v: "x".join(map(str, v)))
def test_iterations(n, per, its):
    dim = len(n)
    mesh = W.Mesh(dim, n, (0.0,) * dim, tuple(k / max(n) for k in n), tuple(map(bool, per)))
    U = W.random_rough_state(mesh, seed=sum(n))
    found = []
    for dt in (5e-3, 1.0):
        s = abi.Solver(abi.Graph(mesh))
        s.set_state(U)
        s.set_viscous(mu=1.0, lam=0.5, kappa=1.4, cv=2.5, cg_rtol=1e-10, cg_maxit=3000,
                      precond=abi.PC_GMG)
        s.step_parabolic(dt)
        info = s.parabolic_info()
        found += [info.it_v, info.it_e]
    print("mg iterations", n, per, found, flush=True)
    assert all(a <= b + max(1, b // 50) for a, b in zip(found, its))
