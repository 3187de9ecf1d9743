"""Plans and gradients of circuits with rotation offsets."""
import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C
from paper_1608_00263_amd import sv


@pytest.mark.parametrize("tile", [0, 4, 5, 6])
@pytest.mark.parametrize("rows,cols,depth", [(2, 7, 30), (4, 4, 25), (4, 5, 30)])
def test_offsets_in_single_precision_keep_narrow_tiles(rows, cols, depth, tile):
    # the same circuit takes tiles of four wavefronts without offsets (at some
    # width) and in complex128; with offsets in complex64 it keeps tiles of one
    # wavefront, 6 register qubits unless the caller names a width
    circ = C.make_circuit(rows, cols, depth, seed=6, parametrise=True, theta_seed=7)
    for budget in (0, 160):
        text = sv.host_plan_describe(circ, "c64", "regtile", 0, tile, budget=budget)
        assert "waves=[" not in text
        assert set(l.split(" v=")[1].split()[0] for l in text.splitlines()) == {str(tile or 6)}
    assert "waves=[" in sv.host_plan_describe(circ, "c128", "regtile", 0, 4)


def gradient_case(n_rows, n_cols, depth, seed, k):
    """A parametrised circuit and samples of the circuit without offsets, some
    of them improbable under the offsets."""
    circ = C.make_circuit(n_rows, n_cols, depth, seed=seed, parametrise=True, theta_seed=seed + 1, theta_std=0.2)
    p0 = oracle.probs(oracle.apply_circuit(circ.with_theta(np.zeros(circ.nparams))))
    return circ, oracle.sample(p0, k, seed + 2)


def gradient_bound(circ, xs, eps):
    """Bound on a gradient component.  g_j = -2 Re <mu| D_j |phi> with |D_j| =
    1/2 and mu = sum_i |x_i> phi(x_i) / (k p(x_i)): a relative state error e
    (spread evenly over the amplitudes) turns mu by a share e F of its norm, F
    = sqrt(sum 1/z^2 / sum 1/z) with z = N p(x_i), and the reverse pass adds e
    to both states, so |dg_j| <= |mu| e (F + 3).  e: one rounding of size eps a
    gate, accumulated as a random walk, twice over."""
    p = oracle.probs(oracle.apply_circuit(circ))[xs.astype(np.int64)]
    z = p * 2.0 ** circ.n
    xu, cnt = np.unique(xs, return_counts=True)
    pu = oracle.probs(oracle.apply_circuit(circ))[xu.astype(np.int64)]
    mu = np.sqrt((cnt.astype(float) ** 2 / pu).sum()) / xs.size
    F = np.sqrt((1 / z ** 2).sum() / (1 / z).sum())
    return mu * 2 * eps * np.sqrt(circ.ngates) * (F + 3)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,eps", [("c64", 2.0 ** -24), ("c128", 2.0 ** -53)])
@pytest.mark.parametrize("seed,k", [(110, 300), (120, 5000), (130, 20000)])
def test_gradient_against_double_precision(dtype, eps, seed, k):
    # complex128 forwards take tiles of four wavefronts
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1608_00263_amd.autograd import CircuitCrossEntropy
    circ, xs = gradient_case(4, 4, 25, seed, k)
    loss0, g0 = oracle.adjoint(circ, xs)
    bound = gradient_bound(circ, xs, eps)
    f = CircuitCrossEntropy(circ, xs, dtype)
    theta = torch.tensor(circ.theta, dtype=torch.float64, requires_grad=True)
    for _ in range(2):   # the first step tunes
        theta.grad = None
        f(theta).backward()
        err = np.abs(theta.grad.numpy() - g0).max()
        assert err <= bound, (err, bound)
    f.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_tuned_choice_outlives_new_offsets(dtype):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    circ = C.make_circuit(4, 4, 21, seed=140, parametrise=True, theta_seed=141)
    st = sv.State(circ.n, dtype)
    first = st.autotune(circ)
    assert first[3]
    if dtype == "c64" and first[0] == "regtile":
        assert first[2] in (4, 5, 6)
    for i in range(8):
        assert st.autotune(circ.with_theta(circ.theta + 0.05 * (i + 1))) == first
    st.close()
