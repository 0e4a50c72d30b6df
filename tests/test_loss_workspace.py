"""The loss calls with a workspace (what ``binding.bind`` queues): argument rules
on the host, and on the GPU the loss at the workgroup counts where the sum over
slots changes shape, against the call without a workspace."""
from __future__ import annotations

import ctypes
import os

import pytest

from paper_2607_18020_amd import workloads as W

BASE = 0x7F0000000000  # fake device addresses, never dereferenced (every call is refused)


def _refused(ws, loss=BASE + (9 << 32)):
    from paper_2607_18020_amd import binding as B  # noqa: PLC0415
    g = B.make_grid((8, 8), (0.1, 0.1), four=True)
    c = B.make_coeffs(W.Coeffs(nu=0.01))
    f = (ctypes.c_void_p * 1)(BASE)
    out = (ctypes.c_void_p * 1)(BASE + (1 << 32))
    lib = B.lib()
    dloss = BASE + (8 << 32)
    a = lib.fpde_residual_fwd_ws4(W.BURGERS_1DT, ctypes.byref(g), ctypes.byref(c), f, None, out,
                                  loss, ws, None)
    b = lib.fpde_residual_value_and_grad_ws4(W.BURGERS_1DT, ctypes.byref(g), ctypes.byref(c), f,
                                             None, dloss, loss, out, ws, None)
    return a, b


@pytest.mark.parametrize("ws,status", [
    (None, -1), (BASE + (2 << 32) + 4, -5),
    (BASE, -1), (BASE + 8 * 8 * 4 - 8, -1),      # the field
    (BASE + (1 << 32) - 65536 + 8, -1),          # the output
    (BASE + (9 << 32) - 65536 + 8, -1),          # the loss
])
def test_workspace_arguments(ws, status):
    assert _refused(ws) == (status, status)


def test_workspace_size():
    from paper_2607_18020_amd import binding as B  # noqa: PLC0415
    import re  # noqa: PLC0415
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = open(os.path.join(root, "include", "fpde.h")).read()
    assert int(re.search(r"#define FPDE_WORKSPACE_BYTES (\d+)", src).group(1)) == B.WORKSPACE_BYTES


# (operator, grid): what the calls with a workspace launch, (workgroups of the forward, of
# the value and gradient).  One workgroup; a full group of 64 and one more, as one row of
# workgroups or several; a last group of one behind two full ones and a ragged one; the 64
# full groups of the slots, and one workgroup more, which adds by atomics (the value and
# gradient of one field takes half as many wider ones then, which the slots hold again)
COUNTS = {
    (W.BURGERS_1DT, (3, 50)): (1, 3),
    (W.BURGERS_1DT, (66, 70)): (64, 33),
    (W.BURGERS_1DT, (67, 70)): (33, 34),
    (W.BURGERS_1DT, (3, 16385)): (65, 67),
    (W.BURGERS_1DT, (3, 15873)): (63, 65),
    (W.HELMHOLTZ_2D, (3, 32769)): (129, 133),
    (W.HELMHOLTZ_2D, (195, 1500)): (234, 231),
    (W.NS_2D_STEADY, (3, 1015808)): (3968, 4096),
    (W.BURGERS_1DT, (3, 1015809)): (993, 2049),
    (W.BURGERS_1DT, (3, 1024 * 4096)): (4096, 8457),
    (W.BURGERS_1DT, (3, 1024 * 4096 + 1)): (4097, 8457),
    (W.NS_3D_STEADY, (30, 40, 70)): (140, 150),
    (W.HEAT_3D_BE, (64, 65, 66)): (234, 396),
    (W.NS_3DT, (5, 12, 20, 40)): (150, 54),
}
SHAPES = list(COUNTS)


def test_workgroup_counts(tmp_path):
    """The grids below launch the workgroup counts that they stand for, and up to 4096 of
    them without the fill that the sum by atomics needs (so they go through the slots)."""
    from paper_2607_18020_amd.csrc import build as build_mod  # noqa: PLC0415
    from tests import launch_rule as L  # noqa: PLC0415
    if not os.path.exists(build_mod.HIPCC):
        pytest.skip("hipcc not available")
    exe = L.compile_rule(tmp_path)
    for (op, shape), want in COUNTS.items():
        for call, n in zip(("fwd_ws", "vg_ws"), want):
            (ls,) = L.launches(exe, [(call, op, shape, 0)])
            march = [x for x in ls if x.tiles and not x.name.startswith("bc")]
            assert [x.blocks for x in march] == [n], (shape, call, ls)
            assert ("fill_f64_kernel" in [x.name for x in ls]) == (n > 4096), (shape, call, ls)


@pytest.mark.gpu
@pytest.mark.parametrize("op,shape", SHAPES,
                         ids=[f"{W.OP_NAMES[o]}-{'x'.join(map(str, s))}" for o, s in SHAPES])
def test_bound_losses(op, shape):
    import torch  # noqa: PLC0415
    from paper_2607_18020_amd import binding as B  # noqa: PLC0415
    print(f"case workspace {W.OP_NAMES[op]} {shape}", flush=True)
    spec = W.OPS[op]
    gen = torch.Generator(device="cuda").manual_seed(3)
    f = [torch.randn(shape, generator=gen, device="cuda") for _ in spec.fields]
    c = [torch.randn(shape, generator=gen, device="cuda") for _ in spec.consts]
    h = [0.1] * len(shape)
    co = W.Coeffs(nu=0.01, k=1.0, dt=0.1, alpha=0.1)
    fwd = B.bind("fwd", op, f, c, h, co)
    vg = B.bind("value_and_grad", op, f, c, h, co)
    first = None
    for k in range(4):  # the counters are zero again after every call
        ref = B.fpde_residual_fwd(op, f, c, h, co).item()
        fwd.result.fill_(float("nan"))
        vg.result[0].fill_(float("nan"))
        a, b = fwd().item(), vg()[0].item()
        # float64 sums of at most 2^23 float32 squares in another order
        assert abs(a - ref) <= 1e-12 * ref and abs(b - ref) <= 1e-12 * ref, (k, a, b, ref)
        if len(spec.fields) > 1:  # (no more workgroups than slots: a fixed order)
            first = first or (a, b)
            assert a == first[0]
            # (the checking build's narrow tiles make 7936 workgroups of the widest grid)
            if os.environ.get("FPDE_TEST_LIBRARY") != "check" or shape[-1] < 1015808:
                assert b == first[1]


@pytest.mark.gpu
def test_bound_calls_on_two_streams_and_captured():
    import torch  # noqa: PLC0415
    from paper_2607_18020_amd import binding as B  # noqa: PLC0415
    op, shape, h, co = W.NS_2D_STEADY, (300, 700), (0.1, 0.1), W.Coeffs(nu=0.01)
    calls, refs = [], []
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in streams:
        f = [torch.randn(shape, device="cuda") for _ in range(3)]
        refs.append(B.fpde_residual_fwd(op, f, [], h, co).item())
        torch.cuda.synchronize()
        calls.append(B.bind("fwd", op, f, [], h, co, stream=s))
    for _ in range(20):
        for call in calls:
            call()
    torch.cuda.synchronize()
    for call, ref in zip(calls, refs):
        assert abs(call.result.item() - ref) <= 1e-12 * ref
    # captured: no reference to the workspace, and every replay starts from zero;
    # a call bound while capturing works outside the graph too
    g = torch.cuda.CUDAGraph()
    loss = torch.empty((), dtype=torch.float64, device="cuda")
    loss2 = torch.empty((), dtype=torch.float64, device="cuda")
    before = B.bind("fwd", op, f, [], h, co, loss=loss2, stream=streams[0])
    with torch.cuda.graph(g, stream=streams[0]):
        inside = B.bind("fwd", op, f, [], h, co, loss=loss)
        inside()
        before()
    for _ in range(3):
        loss.fill_(float("nan"))
        loss2.fill_(float("nan"))
        g.replay()
        calls[1]()
        torch.cuda.synchronize()
        assert abs(loss.item() - refs[1]) <= 1e-12 * refs[1]
        assert abs(loss2.item() - refs[1]) <= 1e-12 * refs[1]
    for call in (inside, before):
        call.result.fill_(float("nan"))
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        assert abs(call.result.item() - refs[1]) <= 1e-12 * refs[1]
