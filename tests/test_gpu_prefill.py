"""GPU parity of the tiled kernel.  Calls of more than 2048 tokens always run on it, so the shapes
here stay small; every test asks the library which kernel and tile its call takes."""
import numpy as np
import pytest
import torch

import paper_2603_25385_amd as G
from glowq_inputs import UnitShape
from oracle import glowq_oracle as O
from gpu_util import DeviceUnit, Workspace, stream
from util import recipe_unit, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-3                     # the forward's bar: fp32 accumulation, R rounded once
ULP = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}
LARGE, HALF = 0, 1


def route_of(du, slabs=True):
    r = G.glowq_debug_route([du.desc], slabs)[0]
    assert r.kernel == G.GLOWQ_ROUTE_TILED
    return r


def make(T, d_in, d_outs, act, Gs=128, r=24, seed=None):
    return recipe_unit(O, 1, 0, T, r=r, shape=UnitShape("g", d_in, d_outs), act=act, G=Gs, method="alg1", qr="none", seed=seed)


def check(ys, refs, tol):
    for y, ref in zip(ys, refs):
        assert y.shape == ref.shape and np.isfinite(y).all()
        e = rel_err(y, ref)
        assert e <= tol, e


def test_one_workspace_for_calls_of_different_sizes():
    # a long prompt whose projection runs in K parts (their arrival counters lie past the first 256
    # bytes of the workspace), and short calls that leave partial sums there, in turn through one
    # buffer that was cleared once: the same bits every time, no wait expired
    units = [make(T, 4352, (64, 40), "f16", seed=60 + T) for T in (2056, 1, 40, 130)]
    dus = [DeviceUnit(u) for u in units]
    route_of(dus[0])
    nbytes = max(G.glowq_workspace_bytes([d.desc]) for d in dus)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    G.glowq_workspace_init(ws.data_ptr(), nbytes, stream())
    failed = torch.zeros(1, dtype=torch.int32, device="cuda")
    first = {}
    for k in (0, 1, 0, 2, 0, 3, 0, 1, 2, 3, 0) * 3:
        dus[k].clear()
        G.glowq_group_forward(dus[k].desc, True, ws.data_ptr(), nbytes, stream())
        G.glowq_workspace_status([dus[k].desc], ws.data_ptr(), nbytes, failed.data_ptr(), stream())
        ys = dus[k].outputs()
        assert int(failed.item()) == 0
        if k not in first:
            check(ys, O.group_forward(units[k], True), TOL)
            first[k] = ys
        assert all(np.array_equal(a, b) for a, b in zip(first[k], ys)), k
