"""Sweeps of the register-tile plans.  The search for tiles of four wavefronts
stops where it cannot save a sweep; the counts are those of the complete
searches, tiles of four wavefronts where they need fewer."""
import pytest

from paper_1608_00263_amd import circuits as C
from paper_1608_00263_amd import sv

# rows, cols, depth, dtype, register qubits, budget: sweeps, wide
COUNTS = [(2, 5, 20, "c64", 0, 0, 2, False), (3, 4, 16, "c64", 0, 0, 2, False), (3, 4, 16, "c64", 6, 0, 1, False),
          (4, 4, 25, "c128", 0, 0, 4, True), (4, 5, 30, "c64", 0, 0, 5, True), (5, 5, 30, "c64", 0, 0, 5, True),
          (4, 7, 40, "c128", 0, 0, 10, True), (5, 6, 40, "c64", 6, 160, 10, True), (5, 6, 40, "c64", 6, 0, 10, True),
          (5, 7, 40, "c64", 6, 0, 12, True), (1, 23, 40, "c64", 0, 0, 5, True)]


@pytest.mark.parametrize("rows,cols,depth,dtype,tile,budget,sweeps,wide", COUNTS)
def test_sweep_counts(rows, cols, depth, dtype, tile, budget, sweeps, wide):
    text = sv.host_plan_describe(C.make_circuit(rows, cols, depth, seed=5030), dtype, "regtile", 0, tile,
                                 budget=budget)
    assert len(text.splitlines()) == sweeps
    assert text.count("waves=[") == (sweeps if wide else 0)
