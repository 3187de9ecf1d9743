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


@pytest.mark.parametrize("n", [1, 4, 8, 9, 10, 11, 13, 16, 22, 23, 24])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_sample_across_the_weight_levels(n, dtype):
    # from a partial unit to several units per chunk and several chunks per
    # group, with runs of empty outcomes
    psi, st = state_of(n, dtype, 60 + n)
    st.close()
    psi[: psi.size // 3] = 0
    psi[psi.size // 2 : psi.size // 2 + psi.size // 8] = 0
    st = sv.State(n, dtype, tensor=torch.from_numpy(psi).to("cuda"))
    want = oracle.sample(oracle.probs(psi), 3000, n)
    np.testing.assert_array_equal(st.sample(3000, n), want)
    np.testing.assert_array_equal(st.moments_and_sample(3000, n)[1], want)
    st.close()


@pytest.mark.parametrize("N", [1, 3, 255, 257, 1023, 1025, 16383, 16385, (1 << 20) + 1, (1 << 24) - 5, (1 << 24) + 77])
def test_sample_from_ragged_levels(N):
    p = C.random_probabilities(N, 70 + N % 97, zeros=N // 5)
    if N > 10:
        p[-1] = 0.0
    words = C.splitmix64_words(N, 2000)
    got = sv.sample_from(torch.from_numpy(p).to("cuda"), torch.from_numpy(words.view(np.int64)).to("cuda"))
    np.testing.assert_array_equal(got.cpu().numpy().view(np.uint64), oracle.sample_from_words(p, words))


@pytest.mark.parametrize("where", [0, 1500, -1])
@pytest.mark.parametrize("bad", [-1e-300, float("nan"), 4.0, float("inf")])
def test_sample_from_one_bad_entry(where, bad):
    p = C.random_probabilities(70001, 5)
    p[where] = bad
    w = torch.zeros(4, dtype=torch.int64, device="cuda")
    with pytest.raises(sv.SVError) as e:
        sv.sample_from(torch.from_numpy(p).to("cuda"), w)
    assert e.value.status == sv.SV_EINVAL


def test_sample_from_total_at_the_limit():
    # weights that sum to 2^64 - 2^11 (accepted; the largest word selects the
    # last outcome) and to 2^64 (refused), entries of 2 and more among them
    top = np.nextafter(4.0, 0.0)
    p = np.zeros(3000)
    p[7], p[2999] = top - 1.0, 1.0
    w = torch.tensor([0, -1], dtype=torch.int64, device="cuda")
    got = sv.sample_from(torch.from_numpy(p).to("cuda"), w).cpu().numpy()
    np.testing.assert_array_equal(got, [7, 2999])
    for q in (4.0 - 1.0, 3.5):
        p[7] = q
        with pytest.raises(sv.SVError) as e:
            sv.sample_from(torch.from_numpy(p).to("cuda"), w)
        assert e.value.status == sv.SV_ERANGE


@pytest.mark.parametrize("n", [31, 32, 33])
def test_sample_wide_sub_buckets(n):
    # sub-buckets of 2^9 and 2^10 entries: a sparse state whose integer CDF is
    # formed on the host
    rng = np.random.default_rng(n)
    idx = np.unique(rng.integers(0, 1 << n, 4000))
    idx = np.unique(np.concatenate([idx, [0, 255, 256, 511, 512, 1023, 1024, (1 << n) - 1]]))
    amp = (rng.standard_normal(idx.size) + 1j * rng.standard_normal(idx.size)) / np.sqrt(2.5 * idx.size)
    amp = amp.astype(np.complex64)
    t = torch.zeros(1 << n, dtype=torch.complex64, device="cuda")
    t[torch.from_numpy(idx).to("cuda")] = torch.from_numpy(amp).to("cuda")
    st = sv.State(n, "c64", tensor=t)
    k, seed = 5000, 9
    xs = st.sample(k, seed)
    m, ys = st.moments_and_sample(k, seed)
    st.close()
    p = amp.real.astype(np.float64) ** 2 + amp.imag.astype(np.float64) ** 2
    cdf = np.cumsum([int(np.floor(np.ldexp(v, 62))) for v in p], dtype=object)
    words = C.splitmix64_words(seed, k)
    want = idx[np.searchsorted(cdf, [(int(r) * int(cdf[-1])) >> 64 for r in words], side="right")]
    np.testing.assert_array_equal(xs, want.astype(np.uint64))
    np.testing.assert_array_equal(ys, xs)
    assert m["zero_count"] == (1 << n) - idx.size
    np.testing.assert_allclose(m["norm"], p.sum(), rtol=1e-12)


@pytest.mark.parametrize("n,nbins,zmin,zmax", [(1, 3, -8.0, 4.0), (9, 1, -1.0, 1.0), (10, 24, -8.0, 4.0),
                                               (11, 255, -8.0, 4.0), (12, 256, -3.0, 1.0), (13, 1024, -8.0, 4.0),
                                               (20, 1024, -20.0, 3.0), (21, 24, 0.5, 0.5 + 1e-13), (22, 7, 6.0, 9.0)])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_pair_histogram_slots(n, nbins, zmin, zmax, dtype):
    # thresholds as arguments and from memory, one to sixteen copies per slot,
    # rows limited by size; zeros, a bin narrower than the logarithm's error
    # and outcomes exactly on thresholds
    a, st = state_of(n, dtype, 80 + n)
    st.close()
    b, _ = state_of(n, dtype, 180 + n)
    if n > 4:
        a[3] = a[7] = 0
        thr = np.ldexp(np.exp(zmin + np.arange(nbins + 1) * ((zmax - zmin) / nbins)), -n)
        m = min(nbins + 1, a.size // 4)
        a[8:8 + m] = np.sqrt(thr[:m])
    sa, sb_ = (sv.State(n, dtype, tensor=torch.from_numpy(x).to("cuda")) for x in (a, b))
    d, h = sv.pair_stats(sa, sb_, nbins, zmin, zmax)
    d0, _ = sv.pair_stats(sa, sb_)
    sa.close()
    sb_.close()
    want, hw = oracle.pair_stats(a, b, nbins, zmin, zmax)
    np.testing.assert_array_equal(h, hw)
    for k, v in want.items():
        for got in (d[k], d0[k]):
            assert (np.isnan(v) and np.isnan(got)) or got == v or abs(got - v) <= 1e-11 * max(1.0, abs(v)), k


@pytest.mark.parametrize("rows,cols,tile", [(3, 6, 1), (3, 6, 2), (3, 6, 3), (3, 6, 4), (3, 6, 5), (1, 19, 5), (4, 5, 4),
                                            (2, 10, 0)])
def test_cycle_statistics_formed_in_the_sweeps(rows, cols, tile):
    # complex128 from 18 qubits up: one to many tiles per wavefront
    circ = C.make_circuit(rows, cols, 14, seed=23)
    st = sv.State(circ.n, "c128")
    got = st.cycle_moments(circ, "regtile", tile)
    psi = st.amplitudes()
    st.close()
    want = oracle.cycle_stats(circ)
    assert np.linalg.norm(psi - oracle.apply_circuit(circ)) <= 1e-11
    assert len(got) == len(want)
    for g, w in zip(got, want):
        # the bound of the per-cycle parity tests on the state's own error
        assert abs(g["norm"] - w["norm"]) <= 1e-11 and abs(g["entropy"] - w["entropy"]) <= 1e-9
        np.testing.assert_allclose(g["moments"], w["moments"], rtol=1e-9)


@pytest.mark.parametrize("nbins", [163, 164])
def test_pair_results_at_the_slot_size(nbins):
    # 505 words fit a 4 KB result slot of 512, 164 bins (514 words) do not
    n = 12
    a, b = (C.random_state(n, s, dtype=np.complex128) for s in (3, 4))
    sa, sb_ = (sv.State(n, "c128", tensor=torch.from_numpy(x).to("cuda")) for x in (a, b))
    _, h = sv.pair_stats(sa, sb_, nbins, -12.0, 4.0)
    sa.close()
    sb_.close()
    np.testing.assert_array_equal(h, oracle.pair_stats(a, b, nbins, -12.0, 4.0)[1])


def test_results_of_more_threads_than_slots():
    # 24 threads for 16 slots, each on a state of its own: exact repeats
    from concurrent.futures import ThreadPoolExecutor

    psis = [C.random_state(10, 40 + i, dtype=np.complex128) for i in range(24)]
    states = [sv.State(10, "c128", tensor=torch.from_numpy(p).to("cuda")) for p in psis]
    alone = [(st.moments()["entropy"], st.sample(50, 5)) for st in states]

    def work(i):
        return [(states[i].moments()["entropy"], states[i].sample(50, 5)) for _ in range(20)]

    with ThreadPoolExecutor(24) as ex:
        for i, rows in enumerate(ex.map(work, range(24))):
            for e, xs in rows:
                assert e == alone[i][0]
                np.testing.assert_array_equal(xs, alone[i][1])
    for st in states:
        st.close()


@pytest.mark.parametrize("rows,cols,depth,dtype", [(2, 3, 63, "c128"), (2, 3, 64, "c64"), (2, 3, 150, "c128"),
                                                   (1, 18, 80, "c128")])
def test_cycle_series_across_the_combined_lists(rows, cols, depth, dtype):
    # 64 points are combined at a time: one list less, one full, several
    circ = C.make_circuit(rows, cols, depth, seed=31)
    st = sv.State(circ.n, dtype)
    got = st.cycle_moments(circ, "regtile")
    st.close()
    want = oracle.cycle_stats(circ)
    assert len(got) == len(want)
    tol = 1e-9 if dtype == "c128" else 1e-4   # the per-cycle parity bounds
    for g, w in zip(got, want):
        assert abs(g["entropy"] - w["entropy"]) <= tol
        np.testing.assert_allclose(g["moments"][:5], w["moments"][:5], rtol=tol if dtype == "c128" else 1e-3)
