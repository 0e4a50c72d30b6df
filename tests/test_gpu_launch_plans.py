"""3-D launches at the sizes where the launch rule changes its mind: one-plane chunks,
a last chunk of one plane, a single chunk, more tiles than a round of workgroups holds,
and the wide and narrow tiles of each kernel, ragged against both.
(tests/test_launch_rule.py holds the launches to that.)
Every entry point against the oracle, node by node, in both boundary modes."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2607_18020_amd import workloads as W
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

CASES = [
    (W.NS_3D_BE, (3, 40, 130)),      # one interior plane; one-plane chunks with the loss
    (W.NS_3D_BE, (67, 64, 66)),      # five-plane chunks, two tiles per row
    (W.NS_3D_STEADY, (62, 9, 129)),  # two- and three-plane chunks, a last tile of one column
    (W.NS_2DT, (5, 290, 520)),       # single chunks
    (W.NS_3D_BE, (17, 33, 193)),     # narrow backward tiles, a last one of one column
    (W.NS_2DT, (17, 33, 193)),
    (W.HEAT_3D_BE, (37, 33, 65)),    # narrow tiles; a last chunk of one plane
    (W.HEAT_3D_BE, (20, 41, 255)),   # wide forward tiles
    (W.POISSON_3D, (70, 12, 257)),
    (W.NS_3D_BE, (5, 290, 1200)),    # more tiles than a round holds, of every kernel
    (W.NS_2DT, (4, 400, 1000)),      # the same, wide backward tiles
    (W.HEAT_3D_BE, (3, 500, 1030)),  # and one field's
    (W.HEAT_3D_BE, (5, 300, 520)),   # wide explicit-sensitivity tiles
    (W.NS_3DT, (4, 19, 13, 131)),
    # the time-marching backward's blocks: 4x8x32 (one chunk of levels per level, two
    # chunks, one), 8x8x32 and 8x6x32, ragged against each
    (W.NS_3DT, (5, 9, 21, 33)),
    (W.NS_3DT, (12, 21, 47, 90)),
    (W.NS_3DT, (5, 17, 41, 65)),
    (W.NS_3DT, (5, 64, 57, 123)),
    (W.NS_3DT, (9, 33, 34, 34)),
]


@pytest.mark.parametrize("bc_mode", [0, 1])
@pytest.mark.parametrize("op,shape", CASES,
                         ids=[f"{W.OP_NAMES[o]}-{'x'.join(map(str, s))}" for o, s in CASES])
def test_launch_plans(op, shape, bc_mode, oracle_mod):
    import torch  # noqa: PLC0415
    from paper_2607_18020_amd import binding as B  # noqa: PLC0415
    wl = W.normal_fields(op, shape, 45)
    print(f"case launch plan {W.OP_NAMES[op]} {shape} bc_mode={bc_mode}", flush=True)
    a = (op, shape, wl.h, wl.coeffs, wl.fields)
    R_ref = oracle_mod.residual(*a, wl.consts, bc_mode=bc_mode)
    L_ref = oracle_mod.loss(*a, wl.consts, bc_mode=bc_mode)
    g_ref = oracle_mod.grad(*a, wl.consts, bc_mode=bc_mode)
    R, L, g = H.run_gpu(wl, bc_mode=bc_mode)
    for r, ref in zip(R, R_ref):
        inner = (lambda x: x) if bc_mode else H.interior
        assert H.max_rel_err(inner(r), inner(ref)) <= H.TOL_RES
    assert abs(L - L_ref) <= H.TOL_RES * abs(L_ref)
    for x, ref in zip(g, g_ref):
        assert np.isfinite(x).all() and H.max_rel_err(x, ref) <= H.TOL_GRAD
    f = [torch.from_numpy(x).cuda() for x in wl.fields]
    c = [torch.from_numpy(x).cuda() for x in wl.consts]
    Lv, gv = B.fpde_residual_value_and_grad(op, f, c, wl.h, wl.coeffs, bc_mode=bc_mode)
    assert abs(Lv.item() - L_ref) <= H.TOL_RES * abs(L_ref)
    sens = W.sensitivities(op, shape, 8)
    gj = B.fpde_residual_vjp(op, f, wl.h, wl.coeffs, [torch.from_numpy(s).cuda() for s in sens],
                             bc_mode=bc_mode)
    gj_ref = oracle_mod.vjp(*a, wl.consts, sens, bc_mode=bc_mode)
    for x, ref in zip(gv, g_ref):
        assert H.max_rel_err(x.cpu().numpy(), ref) <= H.TOL_GRAD
    for x, ref in zip(gj, gj_ref):
        assert H.max_rel_err(x.cpu().numpy(), ref) <= H.TOL_GRAD
