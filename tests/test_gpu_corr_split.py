"""Correlations of fp32 layers on the 16-bit matrix cores, every float as the sum of three bf16 numbers: strips with a narrow last one,
runs across strips and groups of images, waves without k-steps, strides, 3x3 to 5x5 kernels, both column widths of a tile (estimate and exact
gradient); infinities and NaN; volumes read in place.  Host: the loads written as opaque instructions are waited for, and read no
scalar register that a vector instruction wrote within five wait states."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest
import torch

import test_isa_waits as waits
from paper_2106_06998_amd import binding as xb

DEV = "cuda:0"


def split_taken(d, op):
    plan = xb.xconv_plan_info(d, op)
    return plan["ws"] == 2 and plan["M_WG"] == 32 * plan["WM"]       # (the kernel on fp32 instructions: 16 channels a wave)


def gradients(d, X, dY, k):
    Xd, dYd = X.to(DEV), dY.to(DEV)
    xt, dw = xb.alloc_xt(d, DEV), torch.full((dY.shape[1], X.shape[1], *k), float("nan"), device=DEV)
    dwx, xtu = torch.full_like(dw, float("nan")), torch.empty((X.shape[0], d.r, *X.shape[2:]), device=DEV)
    xb.xconv_probe_fwd(d, Xd, xt, None, xb.alloc_ws(d, xb.XCONV_OP_PROBE, DEV))
    xb.xconv_dw_estimate(d, dYd, xt, None, dw, xb.alloc_ws(d, xb.XCONV_OP_ESTIMATE, DEV))
    xb.xconv_dw_exact(d, dYd, Xd, dwx, xb.alloc_ws(d, xb.XCONV_OP_EXACT, DEV))
    xb.xconv_xt_unpack(d, xt, xtu)
    torch.cuda.synchronize()
    return dw.cpu(), dwx.cpu(), xtu.cpu()


def weight_gradient(A, dY, k, s, p):
    return torch.nn.grad.conv2d_weight(A.double(), (dY.shape[1], A.shape[1], *k), dY.double(), s, p)


# B, C_in, C_out, H, W, k, stride, pad, r
CASES = [
    (9, 48, 72, 10, 28, (3, 3), 1, 1, 40),       # one column width of 16, last strip narrow, a group of one image
    (8, 40, 30, 24, 20, (5, 5), 1, 2, 20),       # three groups of offsets, four waves along the reduction
    (5, 64, 200, 28, 28, (3, 3), 1, 1, 32),
    (17, 24, 33, 20, 36, (2, 5), 1, (0, 2), 12),
    (6, 32, 24, 33, 15, (3, 3), 2, 1, 16),       # a strip of four columns for four waves
    (16, 96, 64, 7, 8, (3, 3), 3, 0, 32),
]


@pytest.mark.gpu
@pytest.mark.parametrize("splits", ["1", "3"])
@pytest.mark.parametrize("case", CASES, ids=["b%d-c%d-%d-%dx%d-k%dx%d-s%d" % (*c[:5], *c[5], c[6]) for c in CASES])
def test_split_correlation_against_64_bits(case, splits, monkeypatch):
    B, C_in, C_out, H, W, k, s, pad, r = case
    ph, pw = (pad, pad) if isinstance(pad, int) else pad
    monkeypatch.setenv("XCONV_WS32_SPLITS", splits)
    d = xb.make_desc(B, C_in, C_out, H, W, k, (s, s), (ph, pw), r, "f32", "rademacher", 7)
    g = torch.Generator().manual_seed(B + C_in)
    X = torch.randn((B, C_in, H, W), generator=g)
    dY = torch.randn((B, C_out, (H + 2 * ph - k[0]) // s + 1, (W + 2 * pw - k[1]) // s + 1), generator=g)
    if splits == "1" and dY.shape[3] % 4 == 0:
        assert split_taken(d, xb.XCONV_OP_EXACT)
    dw, dwx, xt = gradients(d, X, dY, k)
    Z = torch.from_numpy(xb.xconv_probe_matrix(d)).double()
    # a product of h + m + l less 3 * 2^-25 of it, K = B * H' * W' of them in sums of 16 that round once or twice, one sum of the splits;
    # a tenth of the worst case, which no sum of random terms comes near
    K = B * dY.shape[2] * dY.shape[3]
    bound = 0.1 * (K / 8 + 16) * 2.0 ** -24
    G, size = weight_gradient(xt, dY, k, s, (ph, pw)), weight_gradient(xt.abs(), dY.abs(), k, s, (ph, pw))
    for got, want, scale in ((dw, torch.einsum("nj,mjyx->mnyx", Z, G) / r, torch.einsum("nj,mjyx->mnyx", Z.abs(), size) / r),
                             (dwx, weight_gradient(X, dY, k, s, (ph, pw)), weight_gradient(X.abs(), dY.abs(), k, s, (ph, pw)))):
        assert bool(((got.double() - want).abs() <= bound * scale).all()), float(((got.double() - want).abs() / scale).max() / 2.0 ** -24)


@pytest.mark.gpu
def test_split_correlation_keeps_infinities_and_nan(monkeypatch):
    monkeypatch.setenv("XCONV_WS32_SPLITS", "2")
    d = xb.make_desc(9, 24, 40, 12, 12, 3, 1, 1, 8, "f32", "rademacher", 7)
    assert split_taken(d, xb.XCONV_OP_EXACT)
    g = torch.Generator().manual_seed(3)
    X, dY = torch.randn((9, 24, 12, 12), generator=g), torch.randn((9, 40, 12, 12), generator=g) * 0.1
    inf, top = float("inf"), torch.finfo(torch.float32).max
    dY[:, 5] = dY[:, 5].bfloat16().float()         # one piece each: m and l are zero beside the infinities
    X[8, 3, 5, 6], X[2, 7, 6, 6], X[1, 11, 4, 4], X[0, 2, 5, 5] = inf, -inf, float("nan"), top
    dY[3, 9, 6, 5], dY[4, 10, 6, 6] = inf, float("nan")
    dwx = gradients(d, X, dY, (3, 3))[1]
    want = weight_gradient(X, dY, (3, 3), 1, 1).float()
    assert torch.equal(torch.isnan(dwx), torch.isnan(want)) and torch.equal(torch.isinf(dwx), torch.isinf(want))
    assert torch.equal(dwx[torch.isinf(want)], want[torch.isinf(want)])
    ok = torch.isfinite(want)
    assert bool(((dwx - want)[ok].abs() <= 1e-5 * (want[ok].abs() + 1)).all())


@pytest.mark.gpu
def test_split_correlation_of_volumes(monkeypatch):
    monkeypatch.setenv("XCONV_WS32_SPLITS", "2")
    g = torch.Generator().manual_seed(4)
    X, dY = torch.randn((2, 20, 6, 9, 12), generator=g), torch.randn((2, 24, 6, 9, 12), generator=g)
    X[1, 3, 4, 5, 6] = 3.3e38                       # bf16 rounds it to nearly its largest number; read once more out of the volume
    dY[:, :, :, 4:7, 5:8] *= 1e-3
    v = xb.make_desc3d(2, 20, 24, 6, 9, 12, 3, 1, 1, 8, "f32", "rademacher", 7)
    dw = torch.full((24, 20, 3, 3, 3), float("nan"), device=DEV)
    Xd, dYd = X.to(DEV), dY.to(DEV)
    xb.xconv3d_dw_exact(v, dYd, Xd, dw, xb.alloc_bytes(xb.xconv3d_workspace_bytes(v, xb.XCONV_OP_EXACT), DEV))
    torch.cuda.synchronize()
    want = torch.nn.grad.conv3d_weight(X.double(), (24, 20, 3, 3, 3), dY.double(), 1, 1)
    ok = want.abs() < 3e38
    size = torch.nn.grad.conv3d_weight(X.double().abs(), (24, 20, 3, 3, 3), dY.double().abs(), 1, 1)
    assert bool(((dw.cpu().double() - want).abs() <= 1e-5 * size)[ok].all())


def scalar_hazards(text, states=5):
    """(function, line number, load) of every memory instruction of hand-written code whose scalar operands a vector instruction wrote fewer
    wait states before: the compiler, which inserts them for its own instructions, does not look into opaque ones."""
    found, name, last = [], "", []
    for i, line in enumerate(text.split("\n")):
        t = line.strip()
        m = re.match(r"(_ZN2xc\w+):", t)
        if m:
            name, last = m.group(1), []
        if not t or t[0] in ";.":
            continue

        def scalars(operands):
            out = set()
            for a, b, one in re.findall(r"s\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
                out |= {int(one)} if one else set(range(int(a), int(b) + 1))
            return out

        if t.startswith("buffer_load"):
            used, distance = scalars(t.split(None, 1)[1]), 0
            for n, written in reversed(last):
                if distance >= states:
                    break
                if written & used:
                    found.append((name, i, t))
                    break
                distance += n
        m = re.match(r"(?:v_readfirstlane_b32|v_readlane_b32|v_cmp\w*) (s\[\d+:\d+\]|s\d+)", t)
        nop = re.match(r"s_nop (\d+)", t)
        last = (last + [(1 + int(nop.group(1)) if nop else 1, scalars(m.group(1)) if m else set())])[-8:]
    return found


def test_the_scan_for_scalar_hazards_finds_one():
    code = "_ZN2xc1kE:\n\tv_readfirstlane_b32 s18, v3\n\ts_mov_b32 s19, 0\n%s\tbuffer_load_dwordx4 v[0:3], v4, s[16:19], 0 offen\n"
    assert len(scalar_hazards(code % "")) == 1 and not scalar_hazards(code % "\ts_nop 3\n") and len(scalar_hazards(code % "\ts_nop 2\n")) == 1


@pytest.mark.skipif(not os.path.exists(waits.HIPCC), reason="hipcc not installed")
def test_opaque_loads_are_waited_for_and_read_settled_registers(tmp_path):
    def assembly(src):
        out = str(tmp_path / (src + ".s"))
        subprocess.run([waits.HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "--cuda-device-only", "-S", os.path.join(waits.CSRC, src), "-o", out], check=True, stderr=subprocess.DEVNULL)
        return open(out).read()

    sources = ["corr_split_kernels.hip", "corr_ws32_kernels.hip", "corr_ws_kernels.hip", "corr_row_kernels.hip"]
    with ThreadPoolExecutor(4) as ex:
        for src, text in zip(sources, ex.map(assembly, sources)):
            assert "buffer_load_dwordx4" in text
            assert not waits.early_copies(text), src
            assert not scalar_hazards(text), (src, scalar_hazards(text)[:5])


def test_the_call_without_a_workspace_keeps_the_smaller_scratch():
    # 5 groups of 10 kernel offsets instead of 6 of 9: more splits, and more partial tiles, than the kernel on fp32 instructions has
    L, limit = xb.lib(), xb.lib().xconv_static_scratch_bytes()
    for C_out in range(32, 160, 8):
        d = xb.make_desc(16, 128, C_out, 64, 64, 7, 1, 3, 64, "f32", "rademacher", 7)
        assert split_taken(d, xb.XCONV_OP_ESTIMATE)
        one = xb.ctypes.c_void_p(16)
        # (null dW: refused behind the check of the scratch, on any machine)
        status = L.xconv_dw_estimate_static(xb.ctypes.byref(d), one, one, None, None, None)
        tile, splits = 49 * 64 * -(-C_out // 64) * 64 * 4, 256 // (6 * -(-C_out // 64))
        if tile * splits + 128 * 64 * 4 + 4096 < limit:
            assert status != xb.XCONV_EWORKSPACE, (C_out, status)
