"""Register tiles of four wavefronts whose sweeps exchange the wave bits more
than once: every circuit here is asserted to be planned that way, so that the
LDS words of one exchange are used again by the next."""
import re

import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C
from paper_1608_00263_amd import sv

# one tile per state, and four; (qubits, register qubits, dtype, circuit seed)
CASES = [(10, 2, "c64", 900), (12, 2, "c64", 900), (11, 3, "c64", 900), (13, 3, "c64", 901), (12, 4, "c64", 900),
         (14, 4, "c64", 903), (13, 5, "c64", 900), (15, 5, "c64", 901), (14, 6, "c64", 904), (16, 6, "c64", 904),
         (10, 2, "c128", 900), (12, 2, "c128", 900), (11, 3, "c128", 900), (13, 3, "c128", 901),
         (12, 4, "c128", 900), (14, 4, "c128", 903), (13, 5, "c128", 900), (15, 5, "c128", 901)]


def exchange_case(n, tile, dtype, seed):
    circ = C.random_unitary_circuit(n, 200, seed=seed)
    text = sv.host_plan_describe(circ, dtype, "regtile", 0, tile, from_zero=False, budget=2000)
    counts = [int(x) for x in re.findall(r"waves=\[\d+,\d+\] exchanges=\[(\d+)\]", text)]
    assert len(counts) == len(text.splitlines()) and max(counts) >= 2, text
    psi0 = C.random_state(n, seed, dtype=np.complex128)
    return circ, psi0, oracle.apply_circuit(circ, psi0.copy())


@pytest.mark.parametrize("n,tile,dtype,seed", CASES)
def test_repeated_exchanges_replay(n, tile, dtype, seed):
    circ, psi0, want = exchange_case(n, tile, dtype, seed)
    got = sv.host_emulate(circ, psi0, dtype, "regtile", 0, tile, from_zero=False, budget=2000)
    assert np.linalg.norm(got - want) < (1e-5 if dtype == "c64" else 1e-12)


@pytest.mark.gpu
@pytest.mark.parametrize("n,tile,dtype,seed", CASES)
def test_repeated_exchanges_match_reference(n, tile, dtype, seed):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    circ, psi0, want = exchange_case(n, tile, dtype, seed)
    npdt = np.complex64 if dtype == "c64" else np.complex128
    for _ in range(3):
        st = sv.State(n, dtype, tensor=torch.from_numpy(psi0.astype(npdt)).to("cuda"))
        st.apply(circ, "regtile", 0, tile, budget=2000)
        # the amplitude bounds of the parity tests
        assert np.linalg.norm(st.amplitudes() - want) <= (1e-4 if dtype == "c64" else 1e-11)
        st.close()
