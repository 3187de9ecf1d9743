"""GPU reductions at the edges of their work split, against the FP64 reference
on identical inputs."""
import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1608_00263_amd import sv  # noqa: E402


def state_of(n, dtype, seed):
    psi = C.random_state(n, seed, dtype=np.complex64 if dtype == "c64" else np.complex128)
    return psi, sv.State(n, dtype, tensor=torch.from_numpy(psi).to("cuda"))


@pytest.mark.parametrize("k", [1, 255, 256, 257, 4095, 4097, 64 * 256 + 1, 65 * 256, 63 * 4096 + 5, 64 * 4096 + 1,
                               130 * 4096 + 17])
def test_cross_entropy_row_counts(k):
    # partial rows from one to more than two per combining segment, ragged
    n = 11
    psi, st = state_of(n, "c128", 40)
    xs = np.random.default_rng(k).integers(0, 1 << n, k, dtype=np.uint64)
    p = oracle.probs(psi)
    ce, dh, z = st.cross_entropy(xs)
    ce0, dh0, z0 = oracle.cross_entropy(p, xs)
    # k logarithms of a few ulp each, compensated sums
    assert abs(ce - ce0) <= 1e-13 * abs(ce0) and abs(dh - dh0) <= 1e-12 and z == z0
    st.close()


@pytest.mark.parametrize("n", [1, 2, 5, 9, 10, 11, 12, 13, 20, 21, 22])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_moments_across_the_work_split(n, dtype):
    # from less than one amplitude per thread to several loads per thread and
    # all partial rows; probabilities near 1 and 1/2 among them (the bin
    # edges of the table logarithm), exact zeros, and subnormals in complex128
    psi, st = state_of(n, dtype, 50 + n)
    st.close()
    rng = np.random.default_rng(n)
    idx = rng.choice(psi.size, min(psi.size, 24), replace=False)
    special = [0.0, 1.0, np.sqrt(0.5), np.sqrt(1 - 2.0 ** -8), np.sqrt(1 + 2.0 ** -8), np.sqrt(0.69987), 1e-12]
    if dtype == "c128":
        special += [1e-155, 1e-161]
    for i, v in zip(idx[1:], special * 3):
        psi[i] = v
    st = sv.State(n, dtype, tensor=torch.from_numpy(psi).to("cuda"))
    got, want = st.moments(), oracle.stats(oracle.probs(psi))
    both, _ = st.moments_and_sample(0, 1)
    st.close()
    for m in (got, both):
        assert m["zero_count"] == want["zero_count"]
        # logarithms of at most 2 ulp and compensated sums; the entropy may
        # cancel against ln S
        for key in ("norm", "entropy"):
            assert abs(m[key] - want[key]) <= 1e-13 * max(1, abs(np.log(want["norm"])), abs(want[key])), key
        assert m["unif_ce"] == want["unif_ce"] or abs(m["unif_ce"] - want["unif_ce"]) <= 1e-13 * abs(want["unif_ce"])
        np.testing.assert_allclose(m["moments"], want["moments"], rtol=1e-13)
