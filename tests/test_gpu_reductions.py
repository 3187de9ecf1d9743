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
