"""The kernel symbol that the benchmark line names for a profile entry, against the kernels that the library
launches for those solves."""
import importlib.util
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_line", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("args,symbol", [
    (("spmm", 7, True, "cocg", 64), "chaff::kr7::k_cocg_mfma"),
    (("nbhd_apply", 7, True, "cocg", 64), "chaff::kr7::k_cocg_mfma"),
    (("spmm_narrow", 7, True, "cocg", 8), "chaff::kr7::k_cocg_mfma"),
    (("spmm_narrow", 7, True, "cocg_rr", 4), "chaff::kr7::k_cocg_stream"),
    (("spmm_narrow", 7, False, "cocg", 3), "chaff::kr7::k_cocg_stream"),
    (("spmm", 7, False, "cocg", 64), "chaff::kr7::k_cocg_spmm"),
    (("spmm", 19, True, "cocg", 64), "chaff::kr19::k_cocg_spmm"),
    (("spmm_narrow", 19, True, "cocg", 1), "chaff::kr19::k_cocg_spmm"),
    (("spmm", 7, True, "gmres", 8), "chaff::kr7::k_spmm_"),
    (("solve_small", 7, True, "gmres", 1), "chaff::kr7::small::k_solve_small"),
    (("lone_solve", 19, True, "cocg", 64), "chaff::kr19::k_lone_apply"),
    (("lone_solve", 7, True, "cocg", 8), "chaff::kr7::k_lone_solve"),
    (("k_cg_update", 19, True, "cocg", 64), "chaff::kr19::k_cg_update"),
    (("k_cg_update", 7, True, "cocg", 64, True), "chaff::kr7::k_cg_update_cl"),
    (("k_cg_p", 7, True, "cocg", 64, True), "chaff::kr7::k_cg_pdir_z"),
    (("fill_mutual", 7, True, "cocg", 64), "chaff::k_mutual"),
    (("precond", 7, True, "gmres", 1), "precond"),
])
def test_symbol(bench, args, symbol):
    assert bench.kernel_symbol(*args) == symbol
    if "::" in symbol:   # a kernel of that name (prefix) is in the sources
        src = "".join(open(os.path.join(ROOT, "paper_2410_03060_amd", "csrc", f)).read()
                      for f in os.listdir(os.path.join(ROOT, "paper_2410_03060_amd", "csrc")) if f.endswith((".hip", ".hpp")))
        assert re.search(r"__global__[^;{]*\b" + symbol.rsplit("::", 1)[1], src)


def test_roofline_of_fp64_work(bench):
    k = dict(total_ms=2.0, launches=2, bytes=2e6, flops=2 * 39.3e9)
    assert abs(bench.roofline_of(k, False, True)["frac"] - 0.5) < 1e-12
    r = bench.roofline_of(k, True)
    assert abs(r["frac"] - 39.3 / 157.3) < 1e-12 and r["bound"] == "mfma"
