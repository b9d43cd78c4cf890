"""The bench prices a matrix-core read against the matrix cores or the memory,
never against the VALU, and names the kernel that a plan launches."""
import importlib.util
import os

import pytest

import paper_2001_08250_amd as pir

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_matrix_core_reads_are_priced_by_their_products(bench):
    # 256 requests over 65,536 rows of 4 KiB in 163 us: 256 * 65536 * 32768 products
    n, B, row, t = 65536, 256, 4096, 163e-6
    size, xors, products = n * row + B * n // 8 + B * row, B * n // 2 * row // 4, B * n * row * 8
    r = bench.plain_roofline(size, xors, products, t)
    assert (r["bound"], r["unit"]) == ("mfma", "TOP/s")
    assert r["peak"] == 5033.16 and r["achieved"] == round(products / t / 1e12, 3)
    assert abs(r["frac"] - products / (256 * 4 * 2048 * 2.4e9) / t) < 1e-4
    # 24 requests: the bytes take longer than the products
    size, xors, products = n * row + 24 * n // 8 + 24 * row, 24 * n // 2 * row // 4, 24 * n * row * 8
    r = bench.plain_roofline(size, xors, products, 60e-6)
    assert (r["bound"], r["unit"]) == ("hbm", "GB/s") and abs(r["frac"] - size / 8e12 / 60e-6) < 1e-4
    # other kernels as before
    r = bench.plain_roofline(n * row, 256 * n // 2 * row // 4, None, 170e-6)
    assert r["bound"] == "alu" and r["peak"] == 78.64


def test_kernel_names(bench):
    plan = {"kind": 1, "tile": 8, "splits": 1, "unroll": 4, "flags": pir.PLAN_ONE_LAUNCH}
    assert bench.kernel_name(plan) == "xorpir_small_kernel"
    assert bench.kernel_name(dict(plan, flags=0)) == "xorpir_tile_kernel"
    assert bench.kernel_name(dict(plan, kind=5, tile=128, flags=0)) == "xorpir_mfma_kernel"
