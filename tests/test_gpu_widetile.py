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


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("tile", [3, 4, 6])
def test_ensembles_of_wide_and_narrow_plans(tile, persistent):
    # one tile per state up to several per item; a depth of 3 needs one sweep
    # and stays on tiles of one wavefront, in the same launches
    shapes = [(2, 7, 30), (4, 4, 20), (3, 6, 24), (4, 5, 20), (3, 5, 3)]
    circs = [C.make_circuit(r, c, d, seed=700 + i) for i, (r, c, d) in enumerate(shapes)]
    states = [sv.State(c.n, "c64") for c in circs]
    for _ in range(2):   # built and replayed
        res = sv.apply_batch(states, circs, mode="regtile", tile=tile, persistent=persistent)
        for c, st, r in zip(circs, states, res):
            ref = oracle.apply_circuit(c)
            want = oracle.stats(oracle.probs(ref))
            # the bounds of the ensembles' parity tests
            assert np.linalg.norm(st.amplitudes() - ref) <= 1e-4
            assert abs(r["entropy"] - want["entropy"]) < 1e-4
            assert abs(r["norm"] - 1.0) < 1e-5
    for st in states:
        st.close()
