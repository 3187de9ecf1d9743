"""The sum of ln p of the statistics where it is finite: states without an exact
zero, with probabilities at the edges of the table logarithm's bins and below
the smallest normal number."""
import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1608_00263_amd import sv  # noqa: E402


def state_without_zeros(n, dtype):
    psi = C.random_state(n, 150 + n, dtype=np.complex64 if dtype == "c64" else np.complex128)
    rng = np.random.default_rng(n)
    # p around 1, 1/2, 0.69987 (the lowest z of the table) and the edges of its
    # 256 bins, large and small magnitudes
    edges = np.sqrt(0.69987 + np.arange(0, 256, 17) / 365.7)
    special = np.concatenate([[1.0, np.sqrt(0.5), np.sqrt(1 - 2.0 ** -8), np.sqrt(1 + 2.0 ** -8), np.sqrt(0.69987),
                               1e-12, 1e-18], edges])
    if dtype == "c128":
        special = np.concatenate([special, [1e-155, 3e-158, 1e-161]])   # p subnormal
    idx = rng.permutation(psi.size)[:max(1, min(psi.size - 1, 3 * special.size))]
    for i, v in zip(idx, np.tile(special, 3)):
        psi[i] = v
    return psi


@pytest.mark.parametrize("n", [1, 2, 5, 9, 10, 11, 12, 13, 20, 21, 22])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_log_sums_without_zeros(n, dtype):
    psi = state_without_zeros(n, dtype)
    p = oracle.probs(psi)
    assert (p > 0).all()
    want = oracle.stats(p)
    assert np.isfinite(want["unif_ce"]) and want["zero_count"] == 0
    st = sv.State(n, dtype, tensor=torch.from_numpy(psi).to("cuda"))
    for m in (st.moments(), st.moments_and_sample(0, 1)[0]):
        assert m["zero_count"] == 0
        # logarithms of at most 2 ulp and sums of few roundings an amplitude
        scale = abs(np.log(want["norm"])) + np.abs(np.log(p)).mean()
        assert abs(m["unif_ce"] - want["unif_ce"]) <= 1e-13 * scale
        scale = abs(np.log(want["norm"])) + (p * np.abs(np.log(p))).sum() / want["norm"]
        assert abs(m["entropy"] - want["entropy"]) <= 1e-13 * scale
    st.close()
