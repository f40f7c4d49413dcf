"""GPU parity of the volumetric (3-D convolution) entry points against the CPU oracle:
stored probe output element by element, weight-gradient estimate to the tolerances of the
2-D parity tests (fp32 1e-4, 16-bit storage 2e-2 of the largest magnitude)."""
import numpy as np
import pytest
import torch

from oracle import xconv_oracle as xo
from paper_2106_06998_amd import binding as xb
from paper_2106_06998_amd import synth
from test_gpu_parity import DEV, GRAD_TOL, ODT, OPROBE, ULP, rel_max, say

pytestmark = pytest.mark.gpu

# name, dtype, B, C_in, C_out, (D,H,W), (kD,kH,kW), stride (depth, in-plane), (pd,ph,pw), r, probe, keep_q15, Z from the seed
VOL = [
    ("f32-3x3x3", "f32", 2, 16, 32, (6, 16, 16), (3, 3, 3), (1, 1), (1, 1, 1), 16, "gaussian", 0, False),
    ("f32-seed", "f32", 2, 16, 32, (6, 16, 16), (3, 3, 3), (1, 1), (1, 1, 1), 16, "gaussian", 0, True),
    ("bf16-ragged-groups", "bf16", 3, 32, 64, (5, 12, 12), (3, 3, 3), (1, 1), (1, 1, 1), 32, "rademacher", 0, False),
    ("f16-odd-planes", "f16", 2, 24, 40, (4, 7, 7), (3, 3, 3), (1, 1), (1, 1, 1), 12, "rademacher", 0, True),
    ("f32-stack-of-2d", "f32", 2, 8, 16, (5, 12, 12), (1, 3, 3), (1, 1), (0, 1, 1), 8, "rademacher", 0, False),
    ("f32-deep-kernel-stride2", "f32", 1, 16, 16, (7, 17, 16), (5, 3, 3), (1, 2), (2, 1, 1), 16, "gaussian", 0, False),
    ("bf16-depth-only-kernel", "bf16", 2, 32, 32, (9, 8, 8), (3, 1, 1), (1, 1), (1, 0, 0), 32, "rademacher", 0, True),
    ("f16-sparse", "f16", 2, 32, 64, (4, 12, 12), (3, 3, 3), (1, 1), (1, 1, 1), 32, "gaussian", 16384, True),
    ("f32-single-slice", "f32", 1, 8, 8, (1, 8, 8), (1, 3, 3), (1, 1), (0, 1, 1), 8, "rademacher", 0, False),
    ("f32-no-depth-padding", "f32", 2, 16, 16, (6, 8, 8), (3, 3, 3), (1, 1), (0, 1, 1), 16, "rademacher", 0, False),
    ("bf16-wide-depth-padding", "bf16", 2, 32, 32, (4, 8, 8), (3, 3, 3), (1, 1), (2, 1, 1), 32, "rademacher", 0, True),
    ("f16-even-depth-kernel", "f16", 3, 16, 24, (5, 6, 8), (2, 3, 3), (1, 1), (1, 1, 1), 16, "gaussian", 0, False),
    ("f32-deep-kernel-no-padding", "f32", 1, 8, 8, (9, 8, 8), (4, 1, 3), (1, 1), (0, 0, 1), 8, "gaussian", 0, True),
    ("f32-depth-stride2", "f32", 2, 16, 16, (8, 8, 8), (3, 3, 3), (2, 2), (1, 1, 1), 16, "gaussian", 0, False),
    ("bf16-depth-stride2-odd-depth", "bf16", 3, 32, 32, (7, 8, 8), (3, 3, 3), (2, 1), (1, 1, 1), 32, "rademacher", 0, True),
    ("f16-depth-stride3-deep-kernel", "f16", 2, 16, 32, (11, 6, 8), (5, 3, 3), (3, 1), (2, 1, 1), 16, "rademacher", 0, False),
    ("f32-depth-stride2-no-padding", "f32", 2, 8, 8, (9, 8, 8), (2, 3, 3), (2, 1), (0, 1, 1), 8, "rademacher", 0, True),
    ("f32-depth-stride-beyond-kernel", "f32", 1, 8, 8, (10, 8, 8), (2, 1, 1), (4, 1), (1, 0, 0), 8, "gaussian", 0, False),
    ("f32-odd-volume", "f32", 2, 6, 10, (3, 5, 5), (3, 3, 3), (1, 1), (1, 1, 1), 5, "gaussian", 0, False),
    ("f16-one-voxel-row", "f16", 5, 16, 16, (3, 4, 8), (3, 3, 3), (1, 1), (1, 1, 1), 16, "rademacher", 0, False),
    ("f16-67200-slices", "f16", 4200, 8, 8, (16, 4, 4), (3, 3, 3), (1, 1), (1, 1, 1), 4, "rademacher", 0, False),  # beyond one grid extent
]


def run_volume(e, nhwc=False):
    name, dtype, B, C_in, C_out, dims, k, st, pad, r, probe, keep, seed_path = e
    say("volumetric %s" % (e,))
    D, H, W = dims
    stride3 = (st[0], st[1], st[1])
    out = tuple(xo.out_extent(n, kk, s, p) for n, kk, s, p in zip(dims, k, stride3, pad))
    seeds = (7101 + len(name), 7202 + len(name), 7303 + len(name))
    X, dY = synth.make_volume(B, C_in, C_out, dims, out, seeds, dtype)
    Z = xo.probe_matrix(OPROBE[probe], seeds[2], C_in, r, keep)
    v = xb.make_desc3d(B, C_in, C_out, D, H, W, k, stride3, pad, r, dtype, probe, seeds[2], keep,
                       xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    assert xb.xconv3d_check_desc(v) == xb.XCONV_OK
    # channels-last: the same values handed over as [B, D, H, W, C]
    Xd = xb.to_device(np.ascontiguousarray(X.transpose(0, 2, 3, 4, 1)) if nhwc else X, dtype, DEV)
    Xt = xb.alloc_bytes(xb.xconv3d_xt_bytes(v), DEV)
    Xt.fill_(0x7f)                                   # poison: data and the zero slices must all be written
    Zd = None if seed_path else torch.from_numpy(Z).to(DEV)
    xb.xconv3d_probe_fwd(v, Xd, Xt, Zd, xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_PROBE), DEV))
    got_xt = torch.empty((B, r, D, H, W), dtype=torch.float32, device=DEV)
    xb.xconv3d_xt_unpack(v, Xt, got_xt)
    torch.cuda.synchronize()
    got_xt = got_xt.cpu().numpy()
    want_xt = xo.probe_fwd3d(X, Z, ODT[dtype])
    scale = np.max(np.abs(want_xt))
    if dtype == "f32":
        assert np.max(np.abs(got_xt - want_xt)) <= 2e-6 * scale
    else:
        floor = 1e-6 if (probe == "rademacher" or dtype == "f16") else 1e-4
        tol = 2.0 * ULP[dtype] * np.maximum(np.abs(want_xt), 2.0 ** -14) + floor * scale
        assert not (np.abs(got_xt - want_xt) > tol).any(), rel_max(got_xt, want_xt)
    dYd = xb.to_device(np.ascontiguousarray(dY.transpose(0, 2, 3, 4, 1)) if nhwc else dY, dtype, DEV)
    dW = torch.full((C_out, C_in) + tuple(k), float("nan"), dtype=torch.float32, device=DEV)
    ws = xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_ESTIMATE), DEV)
    ws.fill_(0x7f)
    xb.xconv3d_dw_estimate(v, dYd, Xt, Zd, dW, ws)
    torch.cuda.synchronize()
    got = dW.cpu().numpy().astype(np.float64)
    want = xo.dw_from_xt3d(dY, want_xt, Z, k, stride3, pad, nnz_norm=keep != 0)
    assert np.all(np.isfinite(got))
    err = rel_max(got, want)
    assert err <= GRAD_TOL[dtype], err
    # exact gradient of the same layer
    dWx = torch.full_like(dW, float("nan"))
    wsx = xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_EXACT), DEV)
    wsx.fill_(0x7f)
    xb.xconv3d_dw_exact(v, dYd, Xd, dWx, wsx)
    torch.cuda.synchronize()
    errx = rel_max(dWx.cpu().numpy().astype(np.float64), xo.dw_exact3d(dY, X, k, stride3, pad))
    assert errx <= GRAD_TOL[dtype], errx
    return v, got


@pytest.mark.parametrize("e", VOL, ids=[e[0] for e in VOL])
def test_volumetric_layers(e):
    run_volume(e)


NDHWC = [VOL[0], VOL[1], VOL[2], VOL[3], VOL[5], VOL[7], VOL[13], VOL[15], VOL[20],
         ("f32-ndhwc-odd-channels", "f32", 2, 6, 10, (3, 5, 5), (3, 3, 3), (1, 1), (1, 1, 1), 5, "gaussian", 0, False),
         ("bf16-ndhwc-channel-tail", "bf16", 2, 24, 40, (4, 6, 8), (3, 3, 3), (2, 1), (1, 1, 1), 16, "rademacher", 0, True)]


@pytest.mark.parametrize("e", NDHWC, ids=[e[0] for e in NDHWC])
def test_channels_last_volumes(e):
    run_volume(e, nhwc=True)


@pytest.mark.parametrize("e", [VOL[0], VOL[2], VOL[5]], ids=[VOL[0][0], VOL[2][0], VOL[5][0]])
def test_volumetric_layers_through_the_dy_copy(e, monkeypatch):
    # layers whose dY the correlation kernel reads in place by default: the slice-major copy gives the same
    monkeypatch.setenv("XCONV_VOL_COPY", "1")
    _, a = run_volume(e)
    monkeypatch.delenv("XCONV_VOL_COPY")
    _, b = run_volume(e)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("nhwc", [False, True], ids=["planes", "channels-last"])
@pytest.mark.parametrize("e", [VOL[0], VOL[2], VOL[7], VOL[14], VOL[16]], ids=[VOL[i][0] for i in (0, 2, 7, 14, 16)])
def test_volumes_beyond_the_offset_table(e, nhwc, monkeypatch):
    # a launch per kernel-depth offset, as volumes with more than 1 GiB of dY take
    monkeypatch.setenv("XCONV_VOL_TABLE_BYTES", "1")
    run_volume(e, nhwc)


@pytest.mark.parametrize("fused", ["0", "1"], ids=["two-launches", "one-launch"])
def test_volumetric_second_pass_routes(fused, monkeypatch):
    monkeypatch.setenv("XCONV_FUSED_PASS2", fused)
    for e in VOL[:4]:
        run_volume(e)


def test_volumetric_estimate_is_deterministic():
    _, a = run_volume(VOL[2])
    _, b = run_volume(VOL[2])
    assert np.array_equal(a, b)


def test_volumetric_full_rank_probe_gives_the_exact_gradient():
    # Z = Hadamard rows (Z Z^T = r I): the estimate equals Eq. (2)/(5) with kD*kH*kW offsets
    B, C, C_out, dims, k, pad = 2, 4, 8, (4, 8, 8), (3, 3, 3), (1, 1, 1)
    say("volumetric hadamard")
    X, dY = synth.make_volume(B, C, C_out, dims, dims, (7401, 7402, 0), "f32")
    Zh = np.array([[1, 1, 1, 1], [1, -1, 1, -1], [1, 1, -1, -1], [1, -1, -1, 1]], dtype=np.float32)
    v = xb.make_desc3d(B, C, C_out, dims[0], dims[1], dims[2], k, 1, pad, 4, "f32", "user", 0)
    Xd, dYd, Zd = xb.to_device(X, "f32", DEV), xb.to_device(dY, "f32", DEV), torch.from_numpy(Zh).to(DEV)
    Xt = xb.alloc_bytes(xb.xconv3d_xt_bytes(v), DEV)
    xb.xconv3d_probe_fwd(v, Xd, Xt, Zd, None)
    dW = torch.empty((C_out, C) + k, dtype=torch.float32, device=DEV)
    xb.xconv3d_dw_estimate(v, dYd, Xt, Zd, dW, xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_ESTIMATE), DEV))
    torch.cuda.synchronize()
    want = xo.dw_exact3d(dY, X, k, (1, 1, 1), pad)
    assert rel_max(dW.cpu().numpy().astype(np.float64), want) <= 1e-4


# ---------------------------------------------------------------------------
# seeded random volumes: every kernel depth, depth stride and depth padding the entry points
# accept, with the in-plane shapes that select each of the correlation kernels
# ---------------------------------------------------------------------------
def _random_volumes(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        dtype = ["f32", "bf16", "f16"][rng.integers(3)]
        kD = int([1, 2, 3, 3, 4, 5, 7][rng.integers(7)])
        k = int([1, 3, 3, 5][rng.integers(4)])
        sd = int([1, 1, 2, 3][rng.integers(4)])
        s = int([1, 1, 2][rng.integers(3)])
        pd = int(rng.integers(0, kD))
        p = int(rng.integers(0, k // 2 + 2))
        D = int(rng.integers(max(kD - 2 * pd, 1), 12))
        H, W = int(rng.integers(k + 1, 14)), int(rng.integers(k + 1, 22))
        if rng.random() < 0.6:
            W = (W + 3) // 4 * 4
        if (H + 2 * p - k) // s + 1 < 1 or (W + 2 * p - k) // s + 1 < 1:
            continue
        B = int(rng.integers(1, 6))
        C_in = int([4, 8, 16, 32, 40][rng.integers(5)])
        C_out = int([8, 16, 32, 48, 72][rng.integers(5)])
        r = int([1, 4, 8, 16, 32][rng.integers(5)])
        probe = ["rademacher", "gaussian"][rng.integers(2)]
        keep = int([0, 0, 0, 16000][rng.integers(4)])
        if B * D * C_out * H * W * C_in * kD > 4e7:      # keep the oracle quick
            continue
        out.append(("rnd%02d" % len(out), dtype, B, C_in, C_out, (D, H, W), (kD, k, k), (sd, s), (pd, p, p), r, probe, keep,
                    bool(rng.random() < 0.5)))
    return out


RANDOM_VOLUMES = _random_volumes(32, 20240611)


@pytest.mark.parametrize("e", RANDOM_VOLUMES, ids=["%s-%s" % (e[0], e[1]) for e in RANDOM_VOLUMES])
def test_random_volumes(e):
    run_volume(e)


# ---------------------------------------------------------------------------
# the volumetric benchmark layers at full size, in the launch configuration bench.py times
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("name", ["V1", "V2"])
def test_volumetric_full_size_sampled(name):
    import bench
    c = bench.VOLUMES[name]
    B, C_in, C_out, dims, k, r, dtype = c["B"], c["C_in"], c["C_out"], c["dims"], c["k"], c["r"], c["dtype"]
    D, H, W = dims
    k3, one, pad = (k, k, k), (1, 1, 1), (c["pad"],) * 3
    say("%s full size, sampled entries" % name)
    X, dY = synth.make_volume(B, C_in, C_out, dims, dims, c["seeds"], dtype)
    Z = xo.probe_matrix(OPROBE[c["probe"]], c["seeds"][2], C_in, r)
    v = xb.make_desc3d(B, C_in, C_out, D, H, W, k, 1, c["pad"], r, dtype, c["probe"], c["seeds"][2])
    Xd, dYd = xb.to_device(X, dtype, DEV), xb.to_device(dY, dtype, DEV)
    Xt = xb.alloc_bytes(xb.xconv3d_xt_bytes(v), DEV)
    ws = xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_ESTIMATE), DEV)
    xb.xconv3d_probe_fwd(v, Xd, Xt, None, ws)                       # Z from the seed, as the bench does
    dW = torch.full((C_out, C_in) + k3, float("nan"), dtype=torch.float32, device=DEV)
    xb.xconv3d_dw_estimate(v, dYd, Xt, None, dW, ws)
    dWx = torch.full_like(dW, float("nan"))
    xb.xconv3d_dw_exact(v, dYd, Xd, dWx, xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_EXACT), DEV))
    xt_g = torch.empty((B, r, D, H, W), dtype=torch.float32, device=DEV)
    xb.xconv3d_xt_unpack(v, Xt, xt_g)
    torch.cuda.synchronize()
    got, got_x, xt_g = dW.cpu().numpy().astype(np.float64), dWx.cpu().numpy().astype(np.float64), xt_g.cpu().numpy()
    assert np.all(np.isfinite(got)) and np.all(np.isfinite(got_x))
    say("%s oracle probe" % name)
    xt_o = xo.probe_fwd3d(X, Z, ODT[dtype])
    scale = np.max(np.abs(xt_o))
    if dtype == "f32":
        assert np.max(np.abs(xt_g - xt_o)) <= 2e-6 * scale
    else:
        tol = 2.0 * ULP[dtype] * np.maximum(np.abs(xt_o), 2.0 ** -14) + 1e-6 * scale
        assert not (np.abs(xt_g - xt_o) > tol).any()
    rng = np.random.default_rng(6)
    n = 32
    idx = np.stack([rng.integers(0, C_out, n), rng.integers(0, C_in, n), rng.integers(0, k, n), rng.integers(0, k, n),
                    rng.integers(0, k, n)], axis=1).astype(np.int32)
    idx[0] = (0, 0, 0, 0, 0)
    idx[1] = (C_out - 1, C_in - 1, k - 1, k - 1, k - 1)
    say("%s oracle samples" % name)
    want = xo.dw_from_xt3d_at(dY, xt_o, Z, idx, k3, one, pad)
    g = np.array([got[tuple(i)] for i in idx])
    assert np.max(np.abs(want)) <= 1.05 * np.max(np.abs(got))
    assert np.max(np.abs(g - want)) <= GRAD_TOL[dtype] * np.max(np.abs(want)), (np.max(np.abs(g - want)), np.max(np.abs(want)))
    wx = xo.dw_exact3d_at(dY, X, idx, k3, one, pad)
    gx = np.array([got_x[tuple(i)] for i in idx])
    assert np.max(np.abs(gx - wx)) <= GRAD_TOL[dtype] * np.max(np.abs(wx))
    # property that holds at any size: the estimate is the exact gradient mixed by Z Z^T / r
    G = Z.astype(np.float64) @ Z.astype(np.float64).T / r
    mixed = np.einsum("nq,mqzyx->mnzyx", G, got_x)
    assert rel_max(got, mixed) <= 2 * GRAD_TOL[dtype]
