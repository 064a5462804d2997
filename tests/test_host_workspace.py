"""The solve's workspace against what its kernels write, in the library's host
sources built without a GPU under the address sanitizer (see
test_host_build.py): the stubs of the factorisations fill their outputs, so a
batch larger than its workspace is found as a heap overflow."""
import os
import re
import shutil
import subprocess

import pytest

from test_host_build import CSRC, HOST_SOURCES, ROOT, STUB, _launcher_stubs

FILL = ("const size_t b = batch, k = (n + 63) / 64; std::memset(A, 0, b * n * n * sizeof(*A)); "
        "std::memset(ipiv, 0, b * n * 4); std::memset(Linv, 0, b * k * 4096 * sizeof(*A)); "
        "std::memset(Uinv, 0, b * k * 4096 * sizeof(*A)); std::memset(info, 0, b * 4); "
        "std::memset(scratch, 0, b * (64 * n * sizeof(*A) + 4 * 257)); g_solved += batch; return hipSuccess;")

DRIVER = r'''
#include "gw.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
int g_solved = 0;  // frequencies factorised, by the stubs

// driver BUDGET N N_OMEGA PREC FROM_A: one solve on a context of its own
int main(int, char **argv) {
    gw_ctx *c = nullptr;
    if (gw_create(0, std::strtoull(argv[1], nullptr, 10), &c) != GW_OK) return 1;
    const int n = std::atoi(argv[2]), N = std::atoi(argv[3]);
    const gw_precision prec = (gw_precision)std::atoi(argv[4]);
    std::vector<double> v((size_t)n * n, 0.0), X(2 * (size_t)N * n * n), W(2 * (size_t)N * n * n);
    gw_report rep{};
    const gw_status s = std::atoi(argv[5])
                            ? gw_solve_W_A(c, v.data(), 0, n, X.data(), N, prec, 1e-7, nullptr, W.data(), &rep)
                            : gw_solve_W(c, v.data(), 0, n, X.data(), N, prec, 1e-7, nullptr, W.data(), &rep);
    std::printf("%d %d %d\n", (int)s, rep.n_solved, g_solved);
    return gw_destroy(c) == GW_OK ? 0 : 1;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("hostworkspace")
    stubs, count = re.subn(r"(getrf_batched<z\w+>\([^)]*\) \{) return hipSuccess;", r"\1 " + FILL, _launcher_stubs())
    assert count == 2
    (d / "stubs.cpp").write_text("#include <cstring>\nextern int g_solved;\n" + stubs)
    (d / "driver.cpp").write_text(DRIVER)
    exe = d / "driver"
    srcs = [os.path.join(CSRC, f) for f in HOST_SOURCES] + [str(d / "stubs.cpp"), str(d / "driver.cpp")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-pthread", "-I", STUB, "-I", CSRC, "-I", os.path.join(ROOT, "include")] + srcs +
                       ["-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return str(exe)


FP64, FP32_IR, BF16X_IR = 0, 1, 2


@pytest.mark.parametrize("from_a", [0, 1])
@pytest.mark.parametrize("prec", [FP64, FP32_IR, BF16X_IR])
@pytest.mark.parametrize("n_omega", [2, 4, 6, 16])
@pytest.mark.parametrize("streams", ["1", "2"])
def test_a_batch_fits_its_workspace(driver, n_omega, prec, from_a, streams):
    """A context's first solve, so that nothing larger is there from another;
    a roomy budget and one of a single frequency per batch."""
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1", GW_SOLVE_STREAMS=streams)
    env.pop("GW_FAULT", None)
    want = 2 if n_omega == 2 else n_omega // 2 + 1
    for n, budget in ((5, 1 << 30), (70, 1 << 30), (70, 1 << 19)):
        r = subprocess.run([driver, str(budget), str(n), str(n_omega), str(prec), str(from_a)], capture_output=True,
                           text=True, env=env, timeout=60)
        assert r.returncode == 0, r.stderr[-3000:]
        assert list(map(int, r.stdout.split())) == [0, want, want]
