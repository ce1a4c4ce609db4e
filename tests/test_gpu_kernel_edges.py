"""Kernel branches at the sizes where they can go wrong, against the FP64 oracle
at the suite's parity bar (relative L2 1e-5, no element off by 1e-4 of the
largest)."""
import numpy as np
import pytest
import torch

from oracle import bst as obst
from oracle.geometry import Geometry
from test_gpu_parity import DEV, P, _sinos, assert_parity  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,V,P_r,P_c,interp", [
    (64, 2, 2, 2, "linear"),      # fewer angles than the arcsine series takes
    (64, 15, 2, 2, "linear"),
    (64, 16, 2, 2, "linear"),     # the first count it takes
    (64, 17, 4, 1, "keys"),
    (256, 40, 1, 4, "linear"),    # radii in quarter steps: integers, halves, quarters exact
    (256, 41, 4, 1, "linear"),
    (64, 16384, 2, 2, "linear"),  # the finest angle grid
    (1024, 90, 1, 4, "keys"),     # radii up to the largest n, keys reach past M/2
])
def test_point_coordinates(P, N, V, P_r, P_c, interp):
    print(f"[coordinates] N={N} V={V} Pr={P_r} Pc={P_c} {interp}", flush=True)
    kw = {"interp": "keys", "taper": "keys"} if interp == "keys" else {}
    plan = P.Plan(N, V, pad_radial=P_r, pad_cart=P_c, max_batch=2, **kw)
    sino = _sinos(2, V, N, 31 + N + V)
    img = plan.backproject(sino)
    torch.cuda.synchronize()
    for b in range(2):
        ref = obst.backproject(sino[b].double().cpu().numpy(), Geometry(N, V, N), obst.Params(P_r, P_c, **kw))
        assert_parity(img[b].cpu().numpy(), ref)
