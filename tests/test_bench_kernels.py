"""The bench names one kernel for a phase only where all its launches are that
kernel, and names kernels that the library has."""
import pytest

import bench
from paper_2311_11943_amd import cqr


def config(name, precision=0, **kw):
    w = bench.WORKLOADS[name]
    return cqr.Config(w["n"], w["n"], w["pr"], w["pr"], w["K"], w["K"], w["b"],
                      cqr.CQR_IN_NODE if w["storage"] == "in" else cqr.CQR_OUT_OF_NODE, precision=precision, **kw)


def test_widths():
    assert [bench.own_width(config(c)) for c in ("c1", "c2", "c3", "c5")] == [16, 64, 512, 512]
    assert bench.own_width(config("c5", 1)) == bench.own_width(config("c5", lookahead=0)) == 256


def test_kernels_of_the_trailing_phases():
    product, update = "trailing_product", "trailing_update"
    # pairs of panels share both phases between kernels; small products have their own
    assert [bench.kernel_of(p, config(c)) for c in ("c1", "c2") for p in (product, update)] == [None] * 4
    # 512 columns at once, subtracted 128 (one launch, but for the last panels) or 256 (a launch each) at a time
    assert [bench.kernel_of(p, config("c3")) for p in (product, update)] == ["tnq_kernel<0>", None]
    assert [bench.kernel_of(p, config("c5")) for p in (product, update)] == ["tnq_kernel<0>", "nnq_kernel<0>"]
    assert [bench.kernel_of(p, config("c5", 1)) for p in (product, update)] == ["tnf_kernel", "nnq_kernel<0>"]
    assert [bench.kernel_of(p, config("c2", 1)) for p in (product, update)] == ["tn_lds_kernel<0, true>", "nnw_kernel<0>"]


@pytest.mark.parametrize("workload", list(bench.WORKLOADS))
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_kernels_exist(workload, precision):
    for phase in cqr.PHASES:
        k = bench.kernel_of(phase, config(workload, precision))
        assert k is None or bench.kernel_source_hash(k), k


def test_roofline_skips_phases_of_several_kernels():
    rep = {p: {"ms": 1.0, "launches": 4, "flops": 1e9, "bytes": 1e6} for p in cqr.PHASES}
    rep["trailing_update"]["ms"] = rep["trailing_product"]["ms"] = 50.0
    assert bench.roofline_of(rep, config("c2"), "fp64", "c2")["phase"] not in ("trailing_update", "trailing_product")
    rep["trailing_update"]["ms"] = 60.0
    r = bench.roofline_of(rep, config("c5"), "fp64", "c5")
    assert r["phase"] == "trailing_update" and r["bound"] == "mfma"
    rep["trailing_update"]["bytes"] = 1e9
    assert bench.roofline_of(rep, config("c5"), "fp64", "c5")["bound"] == "hbm"
