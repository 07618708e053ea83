"""Draws through the running sums of the chunks, at the edges of chunks, runs
and waves: bit-exact against the oracle's sampler on the same state."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_09733_amd import inputs as I

pytestmark = pytest.mark.gpu


def _state(n, kind, seed):
    re, im = I.random_state(n, seed)
    if kind == "gaps":           # mass in a few runs and chunks only, zeros between
        keep = np.zeros(1 << n, dtype=bool)
        for b in (0, 63, 64, 1023, 1024 % (1 << n), (1 << n) - 65, (1 << n) - 1):
            keep[b] = True
        re, im = re * keep, im * keep
    elif kind == "front":        # an empty tail: the fallbacks
        re[5:] = 0.0
        im[5:] = 0.0
    return re, im


@pytest.mark.parametrize("n", [10, 11, 12, 14, 16])
@pytest.mark.parametrize("kind", ["random", "gaps", "front"])
def test_draws_equal_the_oracle(n, kind):
    from paper_2608_09733_amd import sv
    re, im = _state(n, kind, n)
    st = sv.State(n)
    st.set_planes(re, im)
    qubits = list(range(n))
    for shots in (1, 257, 5000):
        ref = O.sample(n, re + 1j * im, 7, shots, qubits)
        assert np.array_equal(st.sample(7, shots, qubits), np.asarray(ref, dtype=np.uint64))
    st.close()


@pytest.mark.parametrize("n", [10, 11, 12, 14, 16])
@pytest.mark.parametrize("kind", ["random", "gaps", "front"])
def test_complex64_draws_equal_the_oracle(n, kind):
    from paper_2608_09733_amd import sv
    re, im = (p.astype(np.float32) for p in _state(n, kind, n))
    st = sv.State(n, "c64")
    st.set_planes(re, im)
    qubits = list(range(n))
    psi = re.astype(np.float64) + 1j * im.astype(np.float64)   # the same values
    for shots in (1, 257, 5000):
        ref = O.sample(n, psi, 7, shots, qubits)
        assert np.array_equal(st.sample(7, shots, qubits), np.asarray(ref, dtype=np.uint64))
    st.close()


# A state of 8 GiB is drawn from without running sums up to a quarter as many
# shots as chunks (from 4096 on by whole waves in FP64), with them from there on.
# A shot's draw depends on the seed and its number alone, so the ways agree.
@pytest.mark.parametrize("n,dtype", [(29, "c128"), (30, "c64")])
def test_draws_without_running_sums_are_those_with_them(n, dtype):
    from paper_2608_09733_amd import sv
    circ = I.layered(n, 2, seed=5)
    st = sv.State(n, dtype)
    st.apply(circ.ops, circ.params)
    qubits = list(range(n))
    quarter = 1 << (n - 12)
    want = st.sample(11, quarter, qubits)
    assert len(np.unique(want)) > 1000
    for shots in (1000, 5000, quarter - 1):
        assert np.array_equal(st.sample(11, shots, qubits), want[:shots])
    st.close()
