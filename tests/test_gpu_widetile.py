"""Register tiles of four wavefronts on the GPU against the FP64 reference, at
the sizes from one tile per state up and every width."""
import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1608_00263_amd import sv  # noqa: E402
from test_library_host import WIDE_CASES, wide_circuits  # noqa: E402


@pytest.mark.parametrize("n,tile,dtype", WIDE_CASES + [(20, 4, "c64"), (21, 6, "c64"), (20, 3, "c128"), (20, 5, "c128")])
def test_wide_tiles_match_reference(n, tile, dtype):
    tol = 1e-4 if dtype == "c64" else 1e-11   # the amplitude bounds of the parity tests
    npdt = np.complex64 if dtype == "c64" else np.complex128
    rnd, chain = wide_circuits(n)
    psi0 = C.random_state(n, 9, dtype=np.complex128)
    want_r = oracle.apply_circuit(rnd, psi0.copy())
    want_c = oracle.apply_circuit(chain)
    for budget in (0, 60, 2000):
        st = sv.State(n, dtype, tensor=torch.from_numpy(psi0.astype(npdt)).to("cuda"))
        st.apply(rnd, "regtile", 0, tile, budget=budget)
        assert np.linalg.norm(st.amplitudes() - want_r) <= tol, budget
        st.apply(chain, "regtile", 0, tile, from_zero=True, budget=budget)
        assert np.linalg.norm(st.amplitudes() - want_c) <= tol, budget
        st.close()
