"""2-D launches at the edges of their row segments and chunks: rows of one wave's
62 output columns and one more, the 248- and 496-column backwards and the 256-node
forward segments and one more, 1024-node forward segments with a ragged last one, two
and three interior rows, chunk ends.  (tests/test_launch_rule.py holds the launches to
that.)  Every entry point against the oracle, node by node, in both boundary modes; the
one-pass gradient bitwise bwd + bc on the rows both march."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2607_18020_amd import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

SHAPES = [(3, 3), (4, 62), (5, 64), (3, 248), (9, 249), (40, 256), (33, 257), (130, 65), (12, 497),
          (21, 1025), (600, 6)]
# grids whose forward takes the 1024-node segments
WIDE = [(W.BURGERS_1DT, (200, 2047)), (W.HELMHOLTZ_2D, (500, 1010)), (W.BURGERS_1DT, (700, 2050)),
        (W.NS_2D_STEADY, (500, 1950))]


@pytest.mark.parametrize("bc_mode", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("op", [W.BURGERS_1DT, W.HELMHOLTZ_2D, W.NS_2D_STEADY])
def test_row_edges(op, shape, bc_mode, oracle_mod):
    _check_rows(op, shape, bc_mode, oracle_mod)


@pytest.mark.parametrize("bc_mode", [0, 1])
@pytest.mark.parametrize("op,shape", WIDE,
                         ids=[f"{W.OP_NAMES[o]}-{'x'.join(map(str, s))}" for o, s in WIDE])
def test_wide_segments(op, shape, bc_mode, oracle_mod):
    _check_rows(op, shape, bc_mode, oracle_mod)


def _check_rows(op, shape, bc_mode, oracle_mod):
    import torch  # noqa: PLC0415
    from paper_2607_18020_amd import binding as B  # noqa: PLC0415
    wl = W.normal_fields(op, shape, 46)
    print(f"case rows {W.OP_NAMES[op]} {shape} bc_mode={bc_mode}", flush=True)
    R_ref, L_ref, g_ref = oracle_mod.on_workload(wl, bc_mode=bc_mode)
    R, L, g = H.run_gpu(wl, bc_mode=bc_mode)
    for r, ref in zip(R, R_ref):
        assert H.max_rel_err(r, ref) <= H.TOL_RES
    assert abs(L - L_ref) <= H.TOL_RES * abs(L_ref)
    f = [torch.from_numpy(x).cuda() for x in wl.fields]
    c = [torch.from_numpy(x).cuda() for x in wl.consts]
    Lv, gv = B.fpde_residual_value_and_grad(op, f, c, wl.h, wl.coeffs, bc_mode=bc_mode)
    bound = B.bind("value_and_grad", op, f, c, wl.h, wl.coeffs, bc_mode=bc_mode)
    Lb, gb = bound()
    # float64 sums of the same squares in another order
    assert abs(Lv.item() - L) <= 1e-12 * L and abs(Lb.item() - L) <= 1e-12 * L
    rows = slice(None) if bc_mode else slice(1, shape[0] - 1)
    for x, v, b, ref in zip(g, gv, gb, g_ref):
        assert np.isfinite(x).all() and H.max_rel_err(x, ref) <= H.TOL_GRAD
        v, b = v.cpu().numpy(), b.cpu().numpy()
        assert H.max_rel_err(v, ref) <= H.TOL_GRAD
        assert np.array_equal(v[rows], x[rows]) and np.array_equal(v, b)
