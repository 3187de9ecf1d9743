"""Register-tile sweeps of many scaled gates: the add-only and tangent forms let
the amplitudes grow by a power of two that a complex64 sweep must not run out
of, at any sweep budget."""
import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C
from paper_1608_00263_amd import sv
from test_training_plans import gradient_bound

# depths from one sweep whose start value was subnormal on
CASES = [(2, 7, 110, 6, "c64"), (2, 7, 130, 6, "c64"), (3, 4, 200, 4, "c64"), (1, 13, 130, 5, "c64"),
         (2, 7, 200, 6, "c64"), (2, 7, 200, 5, "c128")]
NPDT = {"c64": np.complex64, "c128": np.complex128}


def range_circuits(rows, cols, depth):
    """Without offsets, and with offsets whose cosines are near 1/2."""
    plain = C.make_circuit(rows, cols, depth, seed=1)
    rot = C.make_circuit(rows, cols, depth, seed=1, parametrise=True, theta_seed=2)
    return plain, rot.with_theta(np.random.default_rng(depth).uniform(0.35, 0.5, rot.nparams))


@pytest.mark.parametrize("rows,cols,depth,tile,dtype", CASES)
@pytest.mark.parametrize("budget", [400, 2000])
def test_scaled_forms_replay_in_range(rows, cols, depth, tile, dtype, budget):
    # FP32 coefficients: the bound of the complex64 replays
    tol = 1e-5 if dtype == "c64" else 1e-12
    n = rows * cols
    psi0 = C.random_state(n, 3, dtype=np.complex128)
    for circ in range_circuits(rows, cols, depth):
        got = sv.host_emulate(circ, oracle.zero_state(n), dtype, "regtile", 0, tile, budget=budget)
        assert np.linalg.norm(got - oracle.apply_circuit(circ)) < tol
        got = sv.host_emulate(circ, psi0, dtype, "regtile", 0, tile, from_zero=False, budget=budget)
        assert np.linalg.norm(got - oracle.apply_circuit(circ, psi0.copy())) < tol


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,depth,tile,dtype", CASES)
def test_scaled_forms_stay_in_range(rows, cols, depth, tile, dtype):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tol = 1e-4 if dtype == "c64" else 1e-11   # the amplitude bounds of the parity tests
    n = rows * cols
    psi0 = C.random_state(n, 3, dtype=np.complex128)
    for circ in range_circuits(rows, cols, depth):
        st = sv.State(n, dtype, tensor=torch.from_numpy(psi0.astype(NPDT[dtype])).to("cuda"))
        st.apply(circ, "regtile", 0, tile, budget=2000)
        assert np.linalg.norm(st.amplitudes() - oracle.apply_circuit(circ, psi0.copy())) <= tol
        st.apply(circ, "regtile", 0, tile, from_zero=True, budget=2000)
        assert np.linalg.norm(st.amplitudes() - oracle.apply_circuit(circ)) <= tol
        st.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,eps", [("c64", 2.0 ** -24), ("c128", 2.0 ** -53)])
@pytest.mark.parametrize("ck", [0, 60])
def test_gradient_at_a_large_budget(dtype, eps, ck):
    # the reverse sweeps hold two grown states, their sums products of both
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _, circ = range_circuits(2, 7, 130)
    xs = oracle.sample(oracle.probs(oracle.apply_circuit(circ)), 4000, 17)
    loss0, g0 = oracle.adjoint(circ, xs)
    st = sv.State(circ.n, dtype)
    loss, g = st.backward(circ, xs, checkpoint_c=ck, budget=2000)
    st.close()
    assert abs(loss - loss0) <= (1e-4 if dtype == "c64" else 1e-9)
    assert np.abs(g - g0).max() <= gradient_bound(circ, xs, eps)
