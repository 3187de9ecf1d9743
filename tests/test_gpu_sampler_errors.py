"""A sampler call that fails leaves the caller's array as it was."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1608_00263_amd import sv  # noqa: E402


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("with_stats", [False, True])
@pytest.mark.parametrize("k", [3, 5000])
def test_zero_weights_leave_the_host_array(dtype, with_stats, k):
    n = 12
    st = sv.State(n, dtype)
    st.tensor.zero_()
    st.tensor[5] = 1.0
    assert (st.sample(k, 1) == 5).all()   # the staging memory now holds samples
    st.tensor.zero_()
    out = np.full(k, 0xABCDEF, dtype=np.uint64)
    ptr, seed = ctypes.c_void_p(out.ctypes.data), ctypes.c_uint64(2)
    stats = sv.Stats()
    if with_stats:
        rc = sv.lib().sv_moments_sample(st.h, ctypes.byref(stats), k, seed, ptr, 0)
    else:
        rc = sv.lib().sv_sample(st.h, k, seed, ptr, 0)
    assert rc == sv.SV_ESTATE
    assert (out == 0xABCDEF).all()
    st.tensor[7] = 0.5                    # the next call is served
    assert (st.sample(k, 3) == 7).all()
    st.close()
