"""Meshes of which most rows are at an end of the mesh (two to four nodes
thick, 25000 such rows or more): the sweeps that take every row by itself,
against the oracle with the bars of the parity tests and, for two passes, against
the persistent kernel bit for bit; and a mesh just below that count."""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2106_02159_amd import abi, workloads as W
from tests.helpers import state_rel_err

pytestmark = pytest.mark.gpu

MESHES = [((15000, 2), (0, 0)), ((12499, 2), (0, 0)), ((3, 20011), (1, 0)),
          ((16600, 4), (0, 1)), ((131, 120, 2), (0, 0, 0)),
          ((4000, 3, 3), (0, 1, 1)), ((2, 127, 131), (0, 1, 0))]


def setup(n, per, seed=0):
    dim = len(n)
    mesh = W.Mesh(dim, n, (0.0,) * dim, tuple(0.01 * k for k in n), tuple(map(bool, per)))
    U = W.random_rough_state(mesh, seed=seed)
    calm = np.arange(mesh.N) % 1000 < 400  # rows without a limited pair too
    U[:, calm] = U[:, :1]
    return mesh, U


@pytest.mark.parametrize("n,per", MESHES, ids=lambda v: "x".join(map(str, v)))
def test_stage(n, per):
    mesh, U = setup(n, per)
    og = O.Graph(mesh.dim, mesh.n, mesh.lo, mesh.hi, mesh.periodic)
    U = og.slip_bc(U)
    g = abi.Graph(mesh)
    for kw in ({}, dict(passes=1), dict(indicator=1), dict(indicator=2)):
        print("thin mesh", n, per, kw, flush=True)
        prm = O.params(cfl=0.9, **kw)
        tau = og.compute_dt(prm, U)
        ref, _, dbg = og.fe_stage(prm, U, tau, debug=True)
        s = abi.Solver(g, cfl=0.9, **kw)
        s.set_state(U, project=False)
        assert s.compute_dt() == pytest.approx(tau, rel=1e-14, abs=0)
        assert s.fe_stage(tau) == abi.NS_OK
        assert np.all(state_rel_err(s.debug("stage_out"), ref) <= 1e-12)
        assert np.abs(s.debug("alpha") - dbg["alpha"]).max() <= 1e-10
        assert np.all(state_rel_err(s.debug("UL"), dbg["UL"]) <= 1e-13)
        if "passes" not in kw:
            assert np.all(state_rel_err(s.debug("U1"), dbg["U1"]) <= 1e-12)


@pytest.mark.parametrize("precision", [abi.PREC_FP64, abi.PREC_MIXED])
@pytest.mark.parametrize("n,per", MESHES, ids=lambda v: "x".join(map(str, v)))
def test_same_bits_as_persistent(n, per, precision):
    mesh, U = setup(n, per, seed=1)
    g, out = abi.Graph(mesh), []
    for persistent in (False, True):
        print("thin mesh bits", n, per, precision, persistent, flush=True)
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


def test_pack():
    meshes = [setup(n, per)[0] for n, per in (((9001, 2), (0, 0)), ((2, 7777), (0, 0)),
                                              ((40, 33), (0, 0)), ((700, 3), (1, 0)))]
    U = [W.random_rough_state(m, seed=k) for k, m in enumerate(meshes)]
    graphs, out = [abi.Graph(m) for m in meshes], []
    for persistent in (False, True):
        print("thin pack", persistent, flush=True)
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
