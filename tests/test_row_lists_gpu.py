"""2D limiter lists on meshes of many blocks (several rounds of the waves, a
ragged end, more blocks than lists): fronts along x and y, few rows and all rows
limited, one mesh and a pack; two steps against the persistent kernel, which
takes every row by itself, bit for bit."""
import time

import numpy as np
import pytest

from paper_2106_02159_amd import abi, workloads as W

pytestmark = pytest.mark.gpu


def box(n, per=(0, 0)):
    return W.Mesh(2, n, (0.0, 0.0), tuple(0.01 * k for k in n), tuple(map(bool, per)))


def state(mesh, kind):
    x, y = mesh.coords()
    rough = W.random_rough_state(mesh, seed=mesh.n[0])
    if kind == "rough":
        return rough
    if kind == "waves":  # all rows limited, alike along x
        w = [0.3 * np.sin(2.0 * np.pi * y / (6.0 * mesh.spacing()[1]) + k) for k in range(3)]
        return W.conserved(1.0 + w[0], (0.5 * w[1], 0.5 * w[2]), 1.0 + w[0], 1.4)
    U = W.constant_state(mesh, rho=1.0, vel=(0.3, -0.2))
    where = np.abs((x if kind == "along y" else y) - 0.5 * mesh.hi[0 if kind == "along y" else 1])
    hit = where < 0.03
    U[:, hit] = rough[:, hit]
    return U


@pytest.mark.parametrize("precision", [abi.PREC_FP64, abi.PREC_MIXED])
@pytest.mark.parametrize("kind", ["along x", "along y", "rough"])
@pytest.mark.parametrize("n,per", [((301, 257), (0, 0)), ((640, 419), (1, 0))],
                         ids=lambda v: "x".join(map(str, v)))
def test_one_mesh(n, per, kind, precision):
    mesh = box(n, per)
    U, g, out = state(mesh, kind), abi.Graph(mesh), []
    for persistent in (False, True):
        print("row lists", n, kind, precision, persistent, flush=True)
        s = abi.Solver(g, cfl=0.5, precision=precision)
        s.set_state(U)
        (s.step_cfl_persistent if persistent else s.step_cfl_async)(2)
        while not s.query():
            time.sleep(1e-3)
        rc, t = s.async_finish()
        assert rc == abi.NS_OK
        out.append((t, s.get_state()))
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("precision", [abi.PREC_FP64, abi.PREC_MIXED])
@pytest.mark.parametrize("kind", ["waves", "rough"])
def test_many_rows(kind, precision):
    """More limited rows than a round of 512 workgroups with 512 rows each."""
    test_one_mesh((701, 613), (0, 0), kind, precision)


def test_pack():
    meshes = [box((131, 97)), box((64, 64), (1, 1)), box((200, 150), (0, 1)), box((33, 57))]
    U = [state(m, k) for m, k in zip(meshes, ("along x", "rough", "rough", "along y"))]
    graphs, out = [abi.Graph(m) for m in meshes], []
    for persistent in (False, True):
        print("row lists pack", persistent, flush=True)
        p = abi.Pack(graphs, cfl=0.5)
        for k, u in enumerate(U):
            p.set_state(k, u)
        (p.step_cfl_persistent if persistent else p.step_cfl_async)(2)
        status, t = p.finish()
        assert all(s == abi.NS_OK for s in status)
        out.append((t, [p.get_state(k) for k in range(len(U))]))
    assert np.array_equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1], out[1][1]):
        assert np.array_equal(a, b)
