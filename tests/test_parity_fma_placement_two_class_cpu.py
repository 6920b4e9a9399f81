"""The two-class sweep's parity fmas lie inside its round-down window (the check
of test_parity_fma_placement_cpu.py on its own source)."""
import test_parity_fma_placement_cpu as placement


def test_parity_fmas_inside_the_round_down_window(tmp_path, monkeypatch):
    monkeypatch.setattr(placement, "SOURCES", ["sweep_dual.hip"])
    placement.test_parity_fmas_inside_the_round_down_window(tmp_path)
