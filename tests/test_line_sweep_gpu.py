"""The sweeps along stencil lines (interior rows) and the listed rows beside
them: mesh widths around the wavefront and workgroup sizes, so that lines,
wavefronts and workgroups end at different places, against the oracle with
the bars of the parity tests; and two steps against the persistent kernel,
which runs every row by the general path, bit for bit."""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2106_02159_amd import abi, workloads as W
from tests.helpers import ell_to_csr_index, rel_err, state_rel_err

pytestmark = pytest.mark.gpu

MESHES = [((62, 5), (0, 0)), ((63, 9), (0, 1)), ((64, 7), (1, 0)), ((65, 6), (1, 1)),
          ((66, 4), (0, 0)), ((127, 5), (0, 0)), ((129, 4), (1, 0)), ((256, 3), (0, 0)),
          ((257, 3), (1, 1)), ((3, 90), (0, 0)), ((4, 65), (1, 0)), ((2, 70), (0, 0)),
          ((64, 4, 3), (0, 0, 0)), ((65, 3, 4), (1, 0, 1)), ((5, 3, 23), (0, 0, 0)),
          ((3, 43, 3), (0, 1, 0)), ((63, 3, 3), (0, 0, 1))]


@pytest.mark.parametrize("n,per", MESHES, ids=lambda v: "x".join(map(str, v)))
def test_line_sweeps(n, per):
    dim = len(n)
    mesh = W.Mesh(dim, n, (0.0,) * dim, tuple(0.01 * k for k in n), tuple(map(bool, per)))
    og = O.Graph(dim, mesh.n, mesh.lo, mesh.hi, mesh.periodic)
    U = og.slip_bc(W.random_rough_state(mesh, seed=sum(n)))
    print("line sweeps", n, per, flush=True)
    prm = O.params(cfl=0.9)
    tau = og.compute_dt(prm, U)
    ref, st, dbg = og.fe_stage(prm, U, tau, debug=True)
    g = abi.Graph(mesh)
    s = abi.Solver(g, cfl=0.9)
    s.set_state(U, project=False)
    assert s.compute_dt() == pytest.approx(tau, rel=1e-14, abs=0)
    assert s.fe_stage(tau) == abi.NS_OK
    assert np.all(state_rel_err(s.debug("stage_out"), ref) <= 1e-12)
    ex = g.export()
    mask, idx = ell_to_csr_index(ex["col"], og.row_ptr, og.col)
    off = og.col[idx] != np.broadcast_to(np.arange(og.N), mask.shape)[mask]
    assert rel_err(s.debug("d")[mask][off], dbg["d"][idx][off]) <= 1e-13
    assert np.abs(s.debug("alpha") - dbg["alpha"]).max() <= 1e-10
    assert np.all(state_rel_err(s.debug("UL"), dbg["UL"]) <= 1e-13)
    assert np.all(state_rel_err(s.debug("FH") * og.mi, dbg["FH"]) <= 1e-12)
    # the same two steps by the launches and by the persistent kernel
    out = []
    for persistent in (False, True):
        s = abi.Solver(g, cfl=0.5)
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
@pytest.mark.parametrize("n", [(9, 9, 9), (66, 5, 5), (130, 4, 6), (34, 21, 4)],
                         ids=lambda v: "x".join(map(str, v)))
def test_limited_entries(n, precision):
    """3D limiter by entries: interior slices with none, few and more than a
    wavefront of limited entries (smooth on one side, rough on the other),
    the same two steps as the general path row by row, bit for bit."""
    mesh = W.Mesh(3, n, (0.0,) * 3, tuple(0.01 * k for k in n), (False,) * 3)
    U = W.random_rough_state(mesh, seed=sum(n))
    smooth = np.arange(mesh.N) % n[0] < n[0] // 2
    U[:, smooth] = U[:, :1]
    g = abi.Graph(mesh)
    out = []
    for persistent in (False, True):
        print("limited entries", n, precision, persistent, flush=True)
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
