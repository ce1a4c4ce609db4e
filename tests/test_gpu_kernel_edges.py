"""Kernel branches at the sizes where they can go wrong, against the FP64 oracle
at the suite's parity bar (relative L2 1e-5, no element off by 1e-4 of the
largest)."""
import numpy as np
import pytest
import torch

from oracle import bst as obst
from oracle import ramp as oramp
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


@pytest.mark.parametrize("N,V,P_c,interp,B", [
    (16, 9, 1, "linear", 5),       # one block holds every column
    (512, 90, 2, "linear", 3),     # G = 1024: 8 points per thread
    (512, 90, 4, "keys", 9),       # G = 2048: 16 points, single slices
    (1024, 91, 2, "linear", 7),    # G = 2048, an odd last pair
    (1024, 64, 4, "linear", 5),    # G = 4096, a quarter of the rows kept
    (2048, 65, 1, "keys", 8),      # every row kept
    (2048, 64, 4, "linear", 3),    # G = 8192
])
def test_gather_chunking_is_bitwise(P, N, V, P_c, interp, B):
    """Blocks of one group, of several with the overlapped gather, ragged last
    blocks and the default choice give the same bits, and the oracle's values."""
    print(f"[chunking] N={N} V={V} Pc={P_c} {interp} B={B}", flush=True)
    kw = {"interp": "keys", "taper": "keys"} if interp == "keys" else {}
    sino = _sinos(B, V, N, 57 + N + V)
    ref = P.Plan(N, V, pad_cart=P_c, max_batch=B, **kw).backproject(sino)
    for gs in (2, 4, 1024):
        got = P.Plan(N, V, pad_cart=P_c, max_batch=B, gather_slices=gs, **kw).backproject(sino)
        assert torch.equal(got, ref), gs
    alone = P.Plan(N, V, pad_cart=P_c, max_batch=1, **kw).backproject(sino[B - 1:])
    assert torch.equal(alone[0], ref[B - 1])
    o = obst.backproject(sino[B - 1].double().cpu().numpy(), Geometry(N, V, N), obst.Params(2, P_c, **kw))
    assert_parity(ref[B - 1].cpu().numpy(), o)


@pytest.mark.parametrize("kind,N,V,P_c,B", [
    ("golden", 1024, 70, 2, 5),       # flipped samples below theta_0, pairs, an odd last one
    ("golden keys", 512, 90, 4, 5),   # single slices
    ("golden", 2048, 40, 2, 4),       # G = 4096: 512 threads a block
    ("tent", 1024, 64, 2, 5),         # wide points from each slice's patch
    ("tent", 2048, 48, 2, 4),
])
def test_overlapped_gather_variants(P, kind, N, V, P_c, B):
    """Blocks that walk several groups with non-uniform angles and with the tent
    rule: the bits of blocks of one group, and the oracle's values."""
    print(f"[overlapped] {kind} N={N} V={V} Pc={P_c} B={B}", flush=True)
    th = np.sort(np.mod(0.05 + np.arange(V) * (np.pi * (np.sqrt(5.0) - 1.0) / 2.0), np.pi)) if "golden" in kind else None
    kw = {"interp": "keys", "taper": "keys"} if "keys" in kind else {}
    if kind == "tent":
        kw["angular"] = "tent"
    sino = _sinos(B, V, N, 13 + N + V)
    ref = P.Plan(N, V, angles=th, pad_cart=P_c, max_batch=B, gather_slices=1024, **kw).backproject(sino)
    one = P.Plan(N, V, angles=th, pad_cart=P_c, max_batch=1, **kw)
    for b in range(B):
        assert torch.equal(one.backproject(sino[b:b + 1])[0], ref[b]), b
    assert torch.equal(P.Plan(N, V, angles=th, pad_cart=P_c, max_batch=B, **kw).backproject(sino), ref)
    for b in (B - 2, B - 1):
        o = obst.backproject(sino[b].double().cpu().numpy(), Geometry(N, V, N, angles=th), obst.Params(2, P_c, **kw))
        assert_parity(ref[b].cpu().numpy(), o)


@pytest.mark.parametrize("V,interp", [(5000, "linear"), (3700, "keys")])
def test_gather_of_large_spectra_is_bitwise(P, V, interp):
    """G = 4096 with more projections than the caches hold: one group alone takes
    the overlapped form's blocks; the bits do not depend on it."""
    print(f"[large spectra] V={V} {interp}", flush=True)
    kw = {"interp": "keys", "taper": "keys"} if interp == "keys" else {}
    N, B = 2048, 3
    sino = torch.randn(B, V, N, generator=torch.Generator().manual_seed(V)).to(DEV)
    ref = P.Plan(N, V, max_batch=B, gather_slices=1024, **kw).backproject(sino)
    one = P.Plan(N, V, max_batch=1, **kw)
    for b in range(B):
        assert torch.equal(one.backproject(sino[b:b + 1])[0], ref[b]), b
    assert torch.equal(P.Plan(N, V, max_batch=B, gather_slices=2, **kw).backproject(sino), ref)


@pytest.mark.parametrize("N,V,P_r,P_c", [(16, 16, 1, 1), (16, 33, 2, 1), (16, 40, 4, 2), (32, 17, 1, 4)])
def test_point_coordinates_on_small_grids(P, N, V, P_r, P_c):
    """The half-plane's mirrored coordinates where two to eight threads share a column."""
    print(f"[small grids] N={N} V={V} Pr={P_r} Pc={P_c}", flush=True)
    sino = _sinos(2, V, N, 3 + N + V)
    img = P.Plan(N, V, pad_radial=P_r, pad_cart=P_c, max_batch=2).backproject(sino)
    for b in range(2):
        ref = obst.backproject(sino[b].double().cpu().numpy(), Geometry(N, V, N), obst.Params(P_r, P_c))
        assert_parity(img[b].cpu().numpy(), ref)


@pytest.mark.parametrize("N,V,filt,mono,B", [
    (16, 9, "ramp", 0.0, 3),       # one group a block, several slices in flight
    (2048, 33, "ramp", 0.0, 7),    # blocks of seven groups, across slices
    (2048, 33, "none", 0.4, 7),    # the monopole of each slice a block walks
    (4096, 17, "ramp", 0.0, 3),    # groups of four rows, twelve a block
    (512, 50, "none", 0.4, 33),
])
def test_row_blocks_across_slices(P, N, V, filt, mono, B):
    """Row blocks that walk several slices: every slice as when it runs alone,
    and the oracle's values."""
    print(f"[row blocks] N={N} V={V} {filt} B={B}", flush=True)
    plan = P.Plan(N, V, filter=filt, monopole_width=mono, max_batch=B)
    sino = _sinos(B, V, N, 91 + N + B)
    img = plan.backproject(sino)
    for b in range(B):
        assert torch.equal(plan.backproject(sino[b:b + 1])[0], img[b]), b
    ref = obst.backproject(sino[B - 1].double().cpu().numpy(), Geometry(N, V, N),
                           obst.Params(filter=filt, monopole=mono))
    assert_parity(img[B - 1].cpu().numpy(), ref)


@pytest.mark.parametrize("N,V,B,check", [
    (512, 9, 35, (0, 17, 34)),        # one group a block
    (512, 9, 130, (0, 65, 129)),      # 8320 groups in threes: a short last block
    (128, 4, 4100, (0, 2047, 4099)),  # more than a block's most groups: two rounds of shares of three
    (2048, 4, 65, (0, 31, 64)),       # the same where a unit holds one block: two rounds of 33
])
def test_row_block_shares(P, N, V, B, check):
    """Shares that do not divide the batch's groups: every slice as when it runs
    alone, and nothing written past the last image."""
    print(f"[row shares] N={N} V={V} B={B}", flush=True)
    plan = P.Plan(N, V, max_batch=B)
    sino = torch.randn(B, V, N, generator=torch.Generator().manual_seed(N + B)).to(DEV)
    buf = torch.full((B * N * N + 16 * N,), 7.0, device=DEV)
    img = plan.backproject(sino, out=buf[:B * N * N].view(B, N, N))
    for b in check:
        assert torch.equal(plan.backproject(sino[b:b + 1])[0], img[b]), b
    assert bool((buf[B * N * N:] == 7.0).all())
    ref = obst.backproject(sino[check[-1]].double().cpu().numpy(), Geometry(N, V, N), obst.Params())
    assert_parity(img[check[-1]].cpu().numpy(), ref)


@pytest.mark.parametrize("n,V,B,offset", [
    (16, 1 + 1, 1, 0),    # fewer outputs and projections than a tile
    (32, 17, 2, 1),       # one projection past a tile; rows at odd floats
    (256, 16, 1, 0),      # exactly one tile of projections, two blocks of outputs
    (512, 31, 3, 1),
    (4096, 18, 1, 0),     # the longest row
])
def test_ramp_filter_tiles(P, n, V, B, offset):
    """The FP64 matrix-unit ramp at the edges of its tiles: within float
    rounding (2^-24 of the output's own scale) of the FP64 convolution."""
    print(f"[ramp] n={n} V={V} B={B} offset={offset}", flush=True)
    plan = P.Plan(n, V, max_batch=B)
    buf = torch.randn(B * V * n + 2, generator=torch.Generator().manual_seed(n + V)).to(DEV)
    sino = buf[offset:offset + B * V * n].view(B, V, n)
    out = torch.full((B * V * n + 2,), 7.0, device=DEV)
    plan.ramp_filter(sino, out=out[offset:offset + B * V * n].view(B, V, n))
    torch.cuda.synchronize()
    got = out.cpu().double().numpy()
    assert np.all(got[:offset] == 7.0) and np.all(got[offset + B * V * n:] == 7.0)
    y = sino.cpu().double().numpy()
    ref = np.stack([oramp.filter_fft(v, 2.0 / n) for v in y])
    err = np.abs(got[offset:offset + B * V * n].reshape(ref.shape) - ref)
    assert np.all(err <= 2.0 ** -23 * np.abs(ref) + 1e-12 * np.abs(ref).max())


@pytest.mark.parametrize("N,angles", [
    (64, [0.0, 3.1415926]),                       # two angles at the ends
    (64, [1.5707963267948966 - 1e-9, 1.5707963267948966]),   # a gap below the search table's step
    (128, list(np.arange(128) * 1e-6 + 1.0) + [3.0]),        # a whole cluster in one bucket
    (128, list(np.sort(np.mod(np.arange(90) * 1.9416135460476904, np.pi)))),
    (64, list(np.arange(40) * (np.pi / 40))),                # directions exactly on angles
])
def test_angle_search(P, N, angles):
    """The bracketing angle of every direction, from the search table: two
    angles, clusters inside a bucket, directions on an angle."""
    print(f"[angle search] N={N} V={len(angles)}", flush=True)
    V = len(angles)
    th = np.asarray(angles)
    plan = P.Plan(N, V, angles=th, max_batch=2)
    sino = _sinos(2, V, N, 7 + N + V)
    img = plan.backproject(sino)
    torch.cuda.synchronize()
    for b in range(2):
        ref = obst.backproject(sino[b].double().cpu().numpy(), Geometry(N, V, N, angles=th), obst.Params())
        assert_parity(img[b].cpu().numpy(), ref)


@pytest.mark.parametrize("N,V,P_r,P_c,B,check", [
    (16, 3, 1, 1, 17, (16,)),        # M = G = 16: one thread per transform, half a projection pair
    (512, 9, 1, 2, 33, (0, 15, 32)), # G = 1024: three slice groups, the last ragged
    (256, 8, 4, 4, 33, (17, 32)),    # the same grid, a quarter of the rows kept
    (1024, 7, 4, 1, 18, (17,)),      # every row kept
    (2048, 4, 4, 4, 2, (1,)),        # G = M = 8192: one slice per pass
])
def test_projector_column_walk(P, N, V, P_r, P_c, B, check):
    print(f"[projector] N={N} V={V} Pr={P_r} Pc={P_c} B={B}", flush=True)
    plan = P.Plan(N, V, pad_radial=P_r, pad_cart=P_c, max_batch=B, adjoint=True)
    img = _sinos(B, N, N, 77 + N + V)
    out = plan.project(img)
    for b in check:
        assert torch.equal(plan.project(img[b:b + 1].contiguous())[0], out[b])
        ref = obst.project(img[b].double().cpu().numpy(), Geometry(N, V, N), obst.Params(P_r, P_c))
        assert_parity(out[b].cpu().numpy(), ref)
