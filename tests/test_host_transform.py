"""The A route's transform against the layout of the products it reads, in the
library's host sources built without a GPU (see test_host_build.py)."""
import os
import shutil
import subprocess

import pytest

from test_host_build import CSRC, HOST_SOURCES, ROOT, STUB, _launcher_stubs

DRIVER = r'''
#include "gw.h"
#include "gw_plan.h"
#include <cstdio>
#include <cstdlib>
int g_by = 0;  // 1: the product, 2: the FFT, by the stubs

// driver PLANNED NOW N: GW_A_TRANSFORM while the workspace is laid out and while
// the transform is enqueued
int main(int, char **argv) {
    gw_ctx *c = nullptr;
    if (gw_create(0, 1ull << 30, &c) != GW_OK) return 1;
    const int n = std::atoi(argv[3]), N = 256, nhb = 5;
    gwp::ARouteWs w;
    setenv("GW_A_TRANSFORM", argv[1], 1);
    if (gwp::a_route_ws(c, "", n, nhb, N, &w) != GW_OK) return 1;
    setenv("GW_A_TRANSFORM", argv[2], 1);
    if (gwp::a_transform_enqueue(c, nullptr, n, N, nhb, w, nullptr, nullptr, 0, 0.125, 0.1, nullptr) != GW_OK) return 1;
    std::printf("%d %lld\n", g_by, (long long)w.xs);
    return gw_destroy(c) == GW_OK ? 0 : 1;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("hosttransform")
    stubs = _launcher_stubs()
    for name, by in (("launch_cauchy_A(", 1), ("launch_fftconv_A(", 2)):
        i = stubs.index("return hipSuccess;", stubs.index(name))
        stubs = stubs[:i] + "g_by = %d; " % by + stubs[i:]
    (d / "stubs.cpp").write_text("extern int g_by;\n" + stubs)
    (d / "driver.cpp").write_text(DRIVER)
    exe = d / "driver"
    srcs = [os.path.join(CSRC, f) for f in HOST_SOURCES] + [str(d / "stubs.cpp"), str(d / "driver.cpp")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", STUB, "-I", CSRC, "-I",
                        os.path.join(ROOT, "include")] + srcs + ["-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return str(exe)


@pytest.mark.parametrize("n", [6, 7])
@pytest.mark.parametrize("planned", ["product", "fft"])
@pytest.mark.parametrize("now", ["product", "fft"])
def test_the_transform_is_the_one_the_bins_were_laid_out_for(driver, planned, now, n):
    """The FFT reads bins n^2 values apart, the product an even number of them:
    the switch is read once, when the workspace is laid out."""
    r = subprocess.run([driver, planned, now, str(n)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    by, stride = map(int, r.stdout.split())
    assert by == (2 if planned == "fft" else 1)
    assert stride == (n * n if planned == "fft" else n * n + (n & 1))
