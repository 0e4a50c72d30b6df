"""The launch rule on the host (no GPU): what each call would queue, read from the
library's own host source (tests/c/launch_rule.cpp)."""
from __future__ import annotations

import os

import numpy as np
import pytest

from paper_2607_18020_amd import workloads as W
from paper_2607_18020_amd.csrc import build as B
from tests import launch_rule as L

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    return L.compile_rule(tmp_path_factory.mktemp("rule"))


# long thin space-time levels: few nodes per block of the time march
@pytest.mark.parametrize("call", ["bwd", "vg"])
@pytest.mark.parametrize("shape", [(3, 50_000_000, 3, 3), (3, 25_000_000, 7, 3),
                                   (4, 19_000_000, 9, 3), (3, 3, 3, 50_000_000)],
                         ids=lambda s: "x".join(map(str, s)))
def test_time_march_stays_launchable(rule, call, shape):
    """A launch holds fewer than 2^32 threads (the runtime refuses more), for every
    level that the size limits admit."""
    for ls in L.launches(rule, [(call, W.NS_3DT, shape, bc) for bc in (0, 1)]):
        assert "bwdt_kernel" in [x.name for x in ls]
        for x in ls:
            assert x.blocks * x.threads < 1 << 32, x


CALLS = ("fwd", "fwdR", "fwd_ws", "bwd", "vg", "vg_ws", "bc", "vjp", "vjp_acc")
# grids of a few nodes to a few times 10^7, narrow and wide rows
GRIDS = {2: [(9, 50), (128, 256), (700, 900), (3000, 3000)],
         3: [(9, 10, 40), (64, 64, 64), (150, 131, 257), (256, 256, 256), (40, 4, 128),
             (66, 64, 512), (300, 300, 300)],
         4: [(5, 9, 10, 40), (10, 32, 32, 32), (22, 29, 32, 28), (14, 56, 55, 83),
             (20, 128, 128, 128)]}


def test_every_kernel_is_reached(rule):
    """The library holds no kernel that the rule never launches."""
    req = [(call, op, shape, bc) for op, spec in W.OPS.items() for shape in GRIDS[spec.ndim]
           for bc in (0, 1) for call in CALLS]
    seen = {x.kernel for ls in L.launches(rule, req) for x in ls}
    assert L.kernels(rule) == seen


@pytest.mark.parametrize("op,shape", [(W.POISSON_2D, (5, 4_500_000)),
                                      (W.HELMHOLTZ_2D, (40, 5_000_000)),
                                      (W.NS_2D_STEADY, (6, 4_300_000)),
                                      (W.HEAT_3D_BE, (9, 1100, 8000)),
                                      (W.NS_3D_BE, (9, 600, 8100))],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_more_workgroups_than_the_workspace_holds(rule, op, shape):
    """Such a launch sums its loss by atomics and is planned so: what the call with a
    workspace queues is what the call without one queues."""
    for call in ("fwd", "vg"):
        plain, ws = L.launches(rule, [(call, op, shape, 0), (call + "_ws", op, shape, 0)])
        assert ws[-1].blocks > 4096 and plain == ws, (plain, ws)


@pytest.mark.parametrize("op,shape", [(W.NS_3DT, (14, 40, 60, 64)), (W.NS_3DT, (20, 60, 60, 40)),
                                      (W.HEAT_3D_BE, (440, 300, 64)),
                                      (W.NS_3D_BE, (200, 200, 60))],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_stored_residuals_on_short_rows(rule, op, shape):
    """More residuals than the L2s hold, on rows that a 64-node tile covers: the forward
    takes it, and leaves no half of a wide tile idle."""
    assert 4 * len(W.OPS[op].residuals) * float(np.prod(shape)) > 2 ** 25
    for bc in (0, 1):
        (ls,) = L.launches(rule, [("fwdR", op, shape, bc)])
        march = [x for x in ls if x.name == "fwd_kernel"]
        assert [x.args[:2] for x in march] == [("64", "8")], march


@pytest.mark.parametrize("shape", [(305, 495, 196), (237, 186, 637), (343, 278, 307)],
                         ids=lambda s: "x".join(map(str, s)))
def test_large_2dt_forward_fills_its_round(rule, shape):
    """On grids whose fields do not fit the caches, two of the three workgroups that a CU
    holds are 1.2 times slower than three: the forward takes a full round, or nearly."""
    (ls,) = L.launches(rule, [("fwd", W.NS_2DT, shape, 0)])
    x = ls[-1]
    per_round = 256 * (3 if x.args[0] == "128" else 4)
    rounds = x.blocks / per_round
    assert x.name == "fwd_kernel" and rounds > 0.6 and abs(rounds - round(rounds)) < 0.33, x
    assert x.blocks > 512, x


@pytest.fixture(scope="module")
def check_rule(tmp_path_factory):
    return L.compile_rule(tmp_path_factory.mktemp("check_rule"), B.CHECK_FLAGS)


def test_checking_build_runs_other_tiles(rule, check_rule):
    """The GPU test that compares the two builds bit for bit needs a different tile (or
    algorithm) in each: every marching launch of every one of its cases."""
    from tests.test_gpu_check_build import CASES  # noqa: PLC0415
    req = [(call, W.CONFIGS[cfg].op, shape, bc) for cfg, shape in CASES for bc in (0, 1)
           for call in ("fwdR", "bwd", "vg", "vjp")]
    for what, a, b in zip(req, L.launches(rule, req), L.launches(check_rule, req)):
        a, b = ([x for x in ls if x.tiles] for ls in (a, b))
        a, b = ([x for x in ls if not x.name.startswith(("bc", "zero"))] for ls in (a, b))
        assert len(a) == len(b) == 1
        tile = lambda x: (x.name, *x.args[:4 if x.name == "bwdt_kernel" else 2])  # noqa: E731
        assert tile(a[0]) != tile(b[0]), (what, a, b)


def _march(ls):
    (x,) = [x for x in ls if x.tiles and not x.name.startswith(("bc", "zero"))]
    return x


def test_edge_cases_of_the_3d_launches(rule):
    """The grids of tests/test_gpu_launch_plans.py reach the edges that they are there for."""
    from tests.test_gpu_launch_plans import CASES  # noqa: PLC0415
    calls = ("fwd", "fwdR", "bwd", "vg", "vjp")
    req = [(call, op, s, bc) for op, s in CASES for bc in (0, 1) for call in calls]
    got = {q: _march(ls) for q, ls in zip(req, L.launches(rule, req))}
    res = {(k, op, tx, ty): (a, b) for k, op, tx, ty, a, b in L.residency(rule)}
    for call in calls:
        space = {q: x for q, x in got.items() if q[0] == call and x.name != "bwdt_kernel"}
        one = last_one = single = rounds = ragged = False
        for (_, op, s, bc), x in space.items():
            inner = 0 if bc or call in ("vg", "vjp") else 2
            planes = (s[1] if len(s) == 4 else s[0]) - inner
            chunks = -(-planes // x.chunk)
            one |= x.chunk == 1 and chunks > 1
            last_one |= x.chunk > 1 and planes % x.chunk == 1
            single |= chunks == 1
            tx, ty = int(x.args[0]), int(x.args[1])
            per_cu = res[("fwd" if call == "fwdR" else call, op, tx, ty)][bc]
            rounds |= chunks == 1 and x.tiles[0] * x.tiles[1] > 256 * per_cu
            ragged |= s[-1] % tx == 1
        assert (one or call == "vjp") and last_one and single and rounds and ragged, \
            (call, one, last_one, single, rounds, ragged)
    tiles = {(x.name, W.OP_NAMES[q[1]], *x.args[:2]) for q, x in got.items()}
    for name, op, wide, narrow in [("fwd_kernel", W.NS_3D_BE, ("128", "4"), ("64", "8")),
                                   ("fwd_kernel", W.HEAT_3D_BE, ("256", "4"), ("64", "8")),
                                   ("bwd_kernel", W.NS_2DT, ("128", "8"), ("64", "8")),
                                   ("vjp_kernel", W.HEAT_3D_BE, ("128", "8"), ("64", "8"))]:
        for tile in (wide, narrow):
            assert (name, W.OP_NAMES[op], *tile) in tiles, (name, op, tile)
    blocks = {x.args[:3] for x in got.values() if x.name == "bwdt_kernel"}
    assert blocks == {("4", "8", "32"), ("8", "6", "32"), ("8", "8", "32")}


def test_edge_cases_of_the_2d_launches(rule):
    """The grids of tests/test_gpu_rows.py: each segment width with a ragged last one."""
    from tests.test_gpu_rows import SHAPES, WIDE  # noqa: PLC0415
    ops = (W.BURGERS_1DT, W.HELMHOLTZ_2D, W.NS_2D_STEADY)
    width = {"fwdq_kernel": lambda x: int(x.args[0]), "bwdq_kernel": lambda x: 62 * int(x.args[0])}
    over = set()  # (operator, kernel, width) with one node in the last segment
    req = [(call, op, s, bc) for op in ops for s in SHAPES for bc in (0, 1)
           for call in ("fwd", "fwdR", "bwd", "vg", "vg_ws")]
    for (call, op, s, bc), ls in zip(req, L.launches(rule, req)):
        x = _march(ls)
        w = width[x.name](x)
        if s[1] % w == 1:
            over.add((op, x.name, w))
    for op in ops:
        assert {(op, "fwdq_kernel", 256), (op, "bwdq_kernel", 248)} <= over
        if op != W.NS_2D_STEADY:
            assert (op, "bwdq_kernel", 496) in over
    req = [(call, op, s, bc) for op, s in WIDE for bc in (0, 1) for call in ("fwd", "fwdR")]
    for q, ls in zip(req, L.launches(rule, req)):
        x = _march(ls)
        assert x.args[0] == "1024" and q[2][1] % 1024 != 0, (q, x)
