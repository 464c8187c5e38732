"""Host-side checks of the benchmark's evidence (no GPU): the decay matrices'
products are priced at the six passes they take, and a traffic summary of every
timed span is there to be looked up."""
import os
import re

import pytest

import bench


def test_decay_matrices_take_six_passes():
    net, matrix = 2e11, 3e11
    r = bench.roofline_of("k_none", 2.0, {"mfma_flop": net + matrix, "matrix_flop": matrix, "pairs": 0.0,
                                          "hbm_bytes": 1e6})
    ms = (3 * net + 6 * matrix) / (bench.F16_MFMA_PEAK_TFLOPS * 1e12) * 1e3
    assert r["bound"] == "mfma" and abs(r["lower_bound_ms"]["mfma"] - ms) < 1e-4
    assert abs(r["mfma_passes"] - (3 * net + 6 * matrix) / (net + matrix)) < 1e-3
    counts = {"pairs": 70.0, "matrix_pairs": 50.0, "mlp_flop": 1000.0, "contacted_items": 1.0, "contacted_nodes": 1.0,
              "passive": 1.0}
    for kernel, flop in (("k_step", 300.0), ("k_bwd_decay", 600.0)):
        w = bench.algorithmic_work(kernel, counts, 1, 1, 1, 1, 0)
        assert w["matrix_flop"] == flop and w["pairs"] == 20.0
        assert w["mfma_flop"] - flop == (1000.0 if kernel == "k_step" else 0.0)


@pytest.mark.parametrize("kernel", ["k_step", "k_bwd_decay", "k_bwd", "k_contact", "k_regress"])
def test_a_traffic_summary_is_there(kernel):
    kv = {}
    for ln in open(os.path.join(bench.PROFILES, f"{kernel}_hand4096_hbm_traffic.txt")):
        if ":" in ln and not ln.startswith("#"):
            a, b = ln.split(":", 1)
            kv[a.strip()] = b.strip()
    assert kv["kernel"] == kernel and re.fullmatch("[0-9a-f]{16}", kv["source_digest"])
    assert float(kv["hbm_bytes_per_launch"]) > 0
