"""Single-precision rotations at the angles where their scaled form changes:
form 0 while |cos(t / 2)| >= 2^-12 |sin(t / 2)|, form 1 nearer to a flip."""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_09733_amd import inputs as I

pytestmark = pytest.mark.gpu

# An amplitude goes through 4 layers of up to 4 rotations and 2 diagonals a
# stage, each within a few 2^-24 of it: 1e-5 as for every complex64 amplitude.
TOL32 = 1e-5

EDGE = 2.0 * math.atan(2.0 ** 12)   # |c| = 2^-12 |s|
ANGLES = [0.0, math.pi, -math.pi, 3 * math.pi, EDGE * (1 - 1e-9), EDGE * (1 + 1e-9), math.pi - 1e-7,
          math.pi + 2e-4, math.pi / 2, 1.0, 2 * math.pi]


def _circuit(n, pick):
    ops, par = [], []
    for layer in range(4):
        for q in range(n):
            ops.append(I.Op("ry", (q,), params=(len(par),)))
            par.append(1.0 + 0.1 * q if layer == 0 else pick(layer, q))
        for q in range(n - 1):
            ops.append(I.Op("z", (q + 1,), (q,)))
    return I.Circuit(n, ops, np.array(par))


# fewer qubits than a group, a part of a tile, one tile, several
@pytest.mark.parametrize("n", [2, 3, 5, 13, 14, 16])
@pytest.mark.parametrize("group", [0, 5])
@pytest.mark.parametrize("mix", ["flips", "edges"])
def test_rotations_near_a_flip(n, group, mix):
    from paper_2608_09733_amd import sv
    circ = _circuit(n, (lambda l, q: math.pi) if mix == "flips"
                    else lambda l, q: ANGLES[(3 * l + q) % len(ANGLES)])
    st = sv.State(n, "c64")
    if group:
        st.set_tiling(0, 0, group)
    st.run(circ)
    got = st.to_numpy()
    st.close()
    assert np.max(np.abs(got - O.run_circuit(circ))) <= TOL32


def test_gradients_near_a_flip():
    from paper_2608_09733_amd import sv
    n = 9
    circ = _circuit(n, lambda l, q: ANGLES[(3 * l + q) % len(ANGLES)])
    ham = I.tfim(n)
    st = sv.State(n, "c64", adjoint=True)
    e, g = st.adjoint_grad(circ.ops, circ.params, ham)
    st.close()
    er, gr = O.adjoint_grad(circ, ham)
    # sums over 2 n terms of |coefficient| <= 1
    assert abs(e - er) <= 2 * n * TOL32 and np.max(np.abs(g - gr)) <= 2 * n * TOL32


# Amplitudes may be far from 1: between a stage's rotations and its scales they
# grow by at most about 2^14, so 2^100 times a state gives 2^100 times the result.
@pytest.mark.parametrize("n", [5, 13, 16])
@pytest.mark.parametrize("group", [0, 5])
@pytest.mark.parametrize("mixed", [False, True])
def test_large_amplitudes_stay_finite(n, group, mixed):
    from paper_2608_09733_amd import sv
    near = [math.pi - 1e-3, 1.0, math.pi + 2e-3, math.pi - 5e-4, -math.pi + 1e-3]
    circ = _circuit(n, lambda l, q: near[(3 * l + q) % len(near)])
    ops = circ.ops + ([I.Op("rxx", (0, n - 1), params=(0,))] if mixed else [])
    re, im = I.random_state(n, n)
    re, im = re.astype(np.float32), im.astype(np.float32)
    st = sv.State(n, "c64")
    if group:
        st.set_tiling(0, 0, group)
    got = []
    for scale in (np.float32(1), np.float32(2.0 ** 100)):
        st.set_planes(re * scale, im * scale)
        st.apply(ops, circ.params)
        got.append([p / scale for p in st.planes()])
    st.close()
    assert np.isfinite(got[1]).all() and np.array_equal(got[0], got[1])
