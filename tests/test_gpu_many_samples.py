"""Sample counts beyond one launch of the sampler's lookup (2^25 wavefronts)."""
import numpy as np
import pytest

import oracle
from paper_1608_00263_amd import circuits as C

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1608_00263_amd import sv  # noqa: E402

SLICE = 1 << 25


@pytest.mark.parametrize("k", [SLICE - 1, SLICE + 1, 2 * SLICE, 2 * SLICE + 5])
def test_samples_of_every_slice(k):
    # 2 SLICE samples and more do not fit one launch's 2^32 threads
    n, seed = 11, 31
    psi = C.random_state(n, 8, dtype=np.complex64)
    st = sv.State(n, "c64", tensor=torch.from_numpy(psi).to("cuda"))
    xs = st.sample(k, seed)
    st.close()
    p = oracle.probs(psi)
    where = np.unique(np.concatenate([np.arange(0, k, 4099), np.arange(k - 2000, k)] +
                                     [np.arange(b - 2000, min(b + 2000, k)) for b in range(SLICE, k, SLICE)]))
    i = where.astype(np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (i + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    assert z[0] == C.splitmix64_words(seed, 1)[0]
    np.testing.assert_array_equal(xs[where], oracle.sample_from_words(p, z))
    assert int(xs.max()) < 1 << n
    # every slice was written: the share of the likeliest outcome in each
    x = int(p.argmax())
    q = p[x] / p.sum()
    for b in range(0, k, SLICE):
        part = xs[b:b + SLICE]
        assert abs((part == x).sum() - q * part.size) <= 6 * np.sqrt(q * part.size) + 6
