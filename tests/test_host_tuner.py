"""The batched driver's autotuner, in the library's host sources built without a
GPU (see test_host_build.py): what it allocates, and which table entries it
reads."""
import json
import os
import shutil
import subprocess

import pytest

from test_host_build import CSRC, HOST_SOURCES, ROOT, STUB, _launcher_stubs

DRIVER = r'''
#include "gw.h"
#include "gw_ctx.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
size_t g_test_bytes = 0;  // operands filled for timing, by the stub of launch_fill_test

// driver BUDGET N PREC: records one molecule of N products; prints the operands'
// bytes and what the context keeps of them
int main(int, char **argv) {
    const size_t budget = std::strtoull(argv[1], nullptr, 10);
    const int n = std::atoi(argv[2]);
    gw_ctx *c = nullptr;
    if (gw_create(0, budget, &c) != GW_OK) return 1;
    std::vector<double> eig{-0.5, 0.7}, X{1, 0, 0, 1}, vals(4 * (size_t)n, 0.5), v((size_t)n * n, 0.0);
    std::vector<int32_t> blk_prod{0, n}, blk_orb{0, 2}, orb_idx{0, 1};
    std::vector<int64_t> blk_val{0, 4 * (int64_t)n};
    gw_molecule m{};
    m.n_orb = 2; m.n_occ = 1; m.n_prod = n; m.eig = eig.data(); m.X = X.data(); m.n_blk = 1;
    m.blk_prod = blk_prod.data(); m.blk_orb = blk_orb.data(); m.orb_idx = orb_idx.data();
    m.blk_val = blk_val.data(); m.vals = vals.data();
    const gw_grid g{64, -2.0, 2.0, 0.1, -1};
    std::vector<double> chi(2 * 64 * (size_t)n * n);
    const double *vs[1] = {v.data()};
    void *cs[1] = {chi.data()};
    gw_batch *b = nullptr;
    const gw_status s = gw_batch_create(c, 1, &m, vs, &g, (gw_precision)std::atoi(argv[3]), 1e-7, 2, nullptr, cs, cs, &b);
    std::printf("%d %zu %zu\n", (int)s, g_test_bytes, c->bufs.count("tune") ? c->bufs["tune"].bytes : (size_t)0);
    if (b) gw_batch_destroy(b);
    return gw_destroy(c) == GW_OK ? 0 : 1;
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("hosttuner")
    stubs = _launcher_stubs()
    head = "launch_fill_test(hipStream_t st, uint32_t *p, int64_t n, bool dbl) { "
    assert head in stubs
    stubs = "#include <cstddef>\nextern size_t g_test_bytes;\n" + stubs.replace(head, head + "g_test_bytes = 4 * (size_t)n; ")
    (d / "stubs.cpp").write_text(stubs)
    (d / "driver.cpp").write_text(DRIVER)
    exe = d / "driver"
    srcs = [os.path.join(CSRC, f) for f in HOST_SOURCES] + [str(d / "stubs.cpp"), str(d / "driver.cpp")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", STUB, "-I", CSRC, "-I",
                        os.path.join(ROOT, "include")] + srcs + ["-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return str(exe)


FP64, FP32_IR = 0, 1


def _run(exe, budget, n, prec, table):
    env = dict(os.environ, GW_TUNE_FILE=str(table))
    env.pop("GW_FAULT", None)
    env.pop("GW_BATCH_MODE", None)
    r = subprocess.run([exe, str(budget), str(n), str(prec)], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    status, filled, kept = map(int, r.stdout.split())
    assert status == 0
    return filled, kept


@pytest.mark.parametrize("prec", [FP64, FP32_IR])
@pytest.mark.parametrize("n", [257, 600])
@pytest.mark.parametrize("budget", [1 << 24, 1 << 26, 1 << 33])
def test_operands_stay_within_the_budget_and_are_given_back(driver, tmp_path, budget, n, prec):
    """(A solve whose one frequency needs more than half the budget is planned
    all the same; its operands are one frequency's.)"""
    filled, kept = _run(driver, budget, n, prec, tmp_path / "t.json")
    one = ((n - 256) ** 2 + 2 * (n - 256) * 256) * (16 if prec == FP64 else 8)
    assert one <= filled <= max(one, budget // 2)
    assert kept == 0


def test_float_entries_measured_otherwise_are_not_read(driver, tmp_path):
    """The first table written by measurements on zeros is measured again, its
    entry left alone; a second run reads the new one."""
    table = tmp_path / "t.json"
    table.write_text('{"cgemm_fp32_n768": 1}')
    assert _run(driver, 1 << 30, 600, FP32_IR, table)[0] > 0
    entries = json.loads(table.read_text())
    assert entries.pop("cgemm_fp32_n768") == 1 and len(entries) == 1
    assert _run(driver, 1 << 30, 600, FP32_IR, table)[0] == 0
