"""CPU tests of how the benchmark names the ungapped kernel, takes its recorded memory
traffic and sets its rate against a peak."""
import os
import sys
import types

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

PEAKS = {"valu_pk_f16": {"rate": 7.0e13}, "lds_b64": {"rate": 1.3e14}}


def test_kernel_is_the_one_the_header_names():
    ws = torch.zeros(256, dtype=torch.uint8)
    for i, name in enumerate(bench.UNGAPPED_KERNELS):
        ws[64:76].view(torch.int32)[2] = i
        assert bench.ungapped_kernel(torch, types.SimpleNamespace(ws=ws)) == name
    text = "".join(open(f).read() for f in bench.UNGAPPED_SRC)
    order = ("kMfma", "kF16", "kI16", "kWaveF16", "kWaveI16")
    assert "enum class Tile { %s };" % ", ".join(order) in text


def test_traffic_goes_stale_with_any_source_of_the_kernel(tmp_path):
    src = [tmp_path / n for n in ("a.hip", "b.h")]
    for f in src:
        f.write_text("one\n")
    names = [str(f) for f in src]
    summary = tmp_path / "t.md"
    summary.write_text("kernel_source_sha256_16: %s\ntraffic_bytes_per_launch: 2e+9\n" % bench.kernel_source_hash(names))
    assert bench.recorded_traffic(str(summary), names) == 2e9
    for f in src:
        f.write_text("two\n")
        assert bench.recorded_traffic(str(summary), names) is None
        f.write_text("one\n")
    assert bench.recorded_traffic(str(summary), names) == 2e9


@pytest.mark.parametrize("kernel", bench.UNGAPPED_KERNELS)
def test_no_fraction_passes_one_at_the_peak(kernel):
    r = bench.ungapped_roofline(kernel, 1_000_000, 1.0, PEAKS)
    assert r["bound"] == ("mfma" if kernel == "k_ungapped_mfma" else "alu")
    # a kernel as fast as its bound allows
    ms = 1.0 * r["frac"]
    top = bench.ungapped_roofline(kernel, 1_000_000, ms, PEAKS)
    assert top["frac"] == pytest.approx(1.0) and top["achieved"] == pytest.approx(top["peak"])
    assert ("lds" in top) == (kernel != "k_ungapped_mfma")
