"""Launch plans of the forward convolution and the input gradient on the host (no GPU): the byte offsets of a tile, which count
from its first image, fit the descriptor (or, with 64-bit addresses, the 32-bit element tables) of the kernel that the plan takes,
whatever the layer.  A tile of a strip of SW columns takes SW positions of every row, so it crosses TU / (Ho * SW) images."""
import os
import random
import subprocess
import sys
import time

import numpy as np
import pytest

from paper_2106_06998_amd import binding as xb

# B, C_in, C_out, H, W, k, stride, pad, dtype, channels-last
LARGE = [
    (8, 256, 1024, 500, 500, 1, 1, 0, "bf16", True),       # one row of 250000 positions per image, 512 MB of output each
    (8, 384, 192, 500, 500, 1, 1, 0, "f32", True),
    (8, 16, 1024, 512, 512, 1, 1, 0, "bf16", True),
    (64, 8, 512, 512, 512, 1, 1, 0, "f16", False),
    (16, 192, 192, 4, 50000, 3, 1, 1, "f32", False),       # few long rows
    (40, 512, 512, 28, 602, 4, 5, 0, "f32", False),        # few output rows and large images
    (3, 64, 8, 4000, 4000, 3, 1, 1, "f16", False),         # one image is past the descriptor
    (300, 2000, 2000, 1, 5000, 1, 1, 0, "f32", True),
    (1, 1, 2, 11000, 11000, 3, 1, 1, "f32", False),        # few channels on large planes
    (2, 3, 1, 12000, 12000, 3, 1, 1, "f16", False),
]


def offsets_fit(case):
    B, C_in, C_out, H, W, k, s, p, dtype, nhwc = case
    Ho, Wo, es = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1, 4 if dtype == "f32" else 2
    d = xb.make_desc(B, C_in, C_out, H, W, k, s, p, 1, dtype, layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    assert xb.xconv_check_desc(d) == xb.XCONV_OK
    image = max(C_in * H * W, C_out * Ho * Wo)
    for transposed in (0, 1):
        for ws in (0, 1):
            v = xb.xconv_conv_plan_info(d, transposed, ws)
            rows = v["B"] * v["Ho"]
            first = np.arange(min(-(-rows * v["SW"] // v["TU"]), 1 << 18), dtype=np.int64) * v["TU"]
            last = np.minimum((first + v["TU"] - 1) // v["SW"], rows - 1)
            images = int(np.max(last // v["Ho"] - first // v["SW"] // v["Ho"])) + 1
            assert images <= v["images"], (case, transposed, ws, v)
            reach = images * image
            assert reach < 2 ** 32 - 1 if v["big"] else reach * es < 2 ** 31, (case, transposed, ws, reach, v)
            assert v["lds_bytes"] <= 160 * 1024
            assert v["big"] or image * es < 2 ** 31
            # scalar offsets of whole units of input channels and blocks of 32 output channels
            if not v["big"] and not nhwc:
                cin, cout, ue = (C_out, C_in, 16 // es) if transposed else (C_in, C_out, 16 // es)
                unit = 2 * ue if cin <= 8 * ue else 8 * ue
                planes = (Ho * Wo, H * W) if transposed else (H * W, Ho * Wo)
                assert -(-cin // unit) * unit * planes[0] * es < 2 ** 31 and -(-cout // 32) * 32 * planes[1] * es < 2 ** 31


@pytest.mark.parametrize("case", LARGE, ids=["-".join(str(v) for v in c) for c in LARGE])
def test_offsets_of_a_tile_fit_large_layers(case):
    offsets_fit(case)


def test_offsets_of_a_tile_fit_drawn_layers():
    rng = random.Random(5)
    n = 0
    while n < 150:
        k = rng.choice([1, 1, 1, 2, 3, 4, 5, 7])
        s = rng.choice([1, 1, 1, 2, 3, 5])
        H, W = int(2 ** rng.uniform(0, 12)), int(2 ** rng.uniform(3, 16))
        C_in, C_out = int(2 ** rng.uniform(0, 11)), int(2 ** rng.uniform(0, 11))
        p = rng.choice([0, k // 2])
        Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
        if H + 2 * p < k or W + 2 * p < k or max(C_in * H * W, C_out * Ho * Wo) >= 2 ** 31 or max(C_in * H * W, C_out * Ho * Wo) < 2 ** 22:
            continue
        n += 1
        offsets_fit((rng.choice([2, 5, 16, 64, 300]), C_in, C_out, H, W, k, s, p, rng.choice(["f32", "bf16", "f16"]), rng.random() < 0.5))


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_few_channels_stage_few_units_without_a_workspace(dtype):
    # a chunk of 8 units for 3 channels leaves no room in LDS for the patch of a whole tile of a strided layer
    for B, C_in, C_out, n, k, s, p in ((16, 3, 64, 224, 7, 4, 3), (36, 6, 283, 149, 4, 2, 2), (53, 8, 8, 254, 5, 2, 2)):
        d = xb.make_desc(B, C_in, C_out, n, n, k, s, p, 1, dtype)
        v = xb.xconv_conv_plan_info(d, 0, False)
        assert 4 * v["TU"] >= 3 * 32 * (v["shape"] % 10) * (4 // v["WM"]), v


def test_strided_input_gradients_take_few_launches():
    # one launch for the positions that kernel offsets reach, up to 16 remainders of the stride, whatever the stride
    for k, s, launches in ((3, 1, 1), (3, 2, 1), (3, 3, 1), (4, 4, 1), (1, 8, 1), (3, 5, 1), (2, 64, 1), (5, 7, 2), (7, 16, 4), (7, 64, 4)):
        for ws in (0, 1):
            v = xb.xconv_conv_plan_info(xb.make_desc(2, 16, 24, 224, 224, k, s, 0, 1, "f16"), 1, ws)
            assert (v["launches"], v["pack_launches"]) == (launches, launches * ws), (k, s, v)
    v = xb.xconv_conv_plan_info(xb.make_desc(2, 4, 6, 1, 1, 1, 5, 2, 1, "f16"), 1, 1)
    assert v["launches"] == 0


def test_the_search_does_not_grow_with_the_image():
    xb.xconv_conv_plan_info(xb.make_desc(1, 8, 8, 64, 64, 3, 1, 1, 1, "f16"), 0, 1)
    for n in (3000, 10000):
        d = xb.make_desc(1, 8, 8, n, n, 1, 1, 0, 1, "f16")
        t = time.perf_counter()
        xb.xconv_conv_plan_info(d, 0, 1)
        assert time.perf_counter() - t < 0.03           # 0.3 ms; 70 and 490 ms when every number of strips was tried


def test_running_out_of_host_memory_is_a_status(tmp_path):
    # operator new of a process of its own fails on request; an exception would end it at the C boundary
    src = tmp_path / "new.cpp"
    src.write_text("""#include <cstdlib>
#include <new>
static int fail = 0;
extern "C" void set_fail(int on) { fail = on; }
void *operator new(std::size_t n) { void *p = fail ? nullptr : std::malloc(n ? n : 1); if (!p) throw std::bad_alloc(); return p; }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
""")
    so = str(tmp_path / "new.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(src), "-o", so], check=True)
    code = """
import ctypes, sys
new = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
from paper_2106_06998_amd import binding as xb
L, out = xb.lib(), (ctypes.c_int32 * 16)()
warm, d = (xb.make_desc(2, 64, 64, n, n, 3, 2, 1, 8, "f16") for n in (28, 30))
assert L.xconv_conv_plan_info(ctypes.byref(warm), 1, 1, out) == 0
one = ctypes.c_void_p(4096)
new.set_fail(1)
status = [L.xconv_conv_plan_info(ctypes.byref(d), t, 1, out) for t in (0, 1)]
status.append(L.xconv_conv_fwd(ctypes.byref(d), one, one, one, None))
size = L.xconv_conv_workspace_bytes(ctypes.byref(d), 1)
new.set_fail(0)
assert size == L.xconv_conv_workspace_bytes(ctypes.byref(d), 1) > 0
assert all(s != 0 for s in status), status
assert L.xconv_conv_plan_info(ctypes.byref(d), 1, 1, out) == 0
print("statuses", status)
"""
    p = subprocess.run([sys.executable, "-c", code, so], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=120)
    assert p.returncode == 0 and "statuses" in p.stdout, (p.returncode, p.stdout)


def test_many_positions_take_runs_of_images_on_one_kernel():
    d = xb.make_desc(300, 2, 3, 2048, 2048, 3, 1, 1, 1, "f16")
    for transposed in (0, 1):
        for ws in (0, 1):
            v = xb.xconv_conv_plan_info(d, transposed, ws)
            assert (v["launches"], v["pack_launches"], v["big"]) == (2, ws, 0)
