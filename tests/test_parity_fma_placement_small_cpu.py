"""The parity fmas of the two-class, full-gradient and fused-field LDS sweeps lie
inside their round-down windows (the check of test_parity_fma_placement_cpu.py on
these sources)."""
import pytest

import test_parity_fma_placement_cpu as placement


@pytest.mark.parametrize("source", ["sweep_dual.hip", "sweep_full.hip", "sweep_fields.hip"])
def test_parity_fmas_inside_the_round_down_window(tmp_path, monkeypatch, source):
    monkeypatch.setattr(placement, "SOURCES", [source])
    placement.test_parity_fmas_inside_the_round_down_window(tmp_path)
