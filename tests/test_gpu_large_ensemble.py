"""An ensemble whose round has as many items as a launch has workgroups at most."""
import pytest

from paper_1608_00263_amd import circuits as C

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1608_00263_amd import sv  # noqa: E402


def test_one_instance_of_35_qubits():
    # tiles of four wavefronts with 3 register qubits: 2^24 items a round
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info(0)[0] < 8 * 2 ** 35 + (4 << 30):
        pytest.skip("a 35-qubit complex64 state needs 260 GiB of free device memory")
    circ = C.make_circuit(5, 7, 8, seed=4)
    assert "waves=[" in sv.host_plan_describe(circ, "c64", "regtile", 0, 3)
    st = sv.State(35, "c64")
    print("ensemble of one 35-qubit instance", flush=True)
    got = sv.apply_batch([st], [circ], mode="regtile", tile=3)[0]
    p = st.probs(0, 1 << 12).cpu()
    st.apply(circ, "regtile", 0, 6, from_zero=True)
    want = st.moments()
    q = st.probs(0, 1 << 12).cpu()
    st.close()
    del st
    torch.cuda.empty_cache()
    # the bounds of the ensembles' parity tests
    assert abs(got["norm"] - 1.0) < 1e-5
    assert abs(got["entropy"] - want["entropy"]) < 1e-4
    assert (p - q).abs().max() <= 1e-4 * q.max()
