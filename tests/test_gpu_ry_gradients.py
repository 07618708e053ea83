"""Gradients of RY rotations taken by their place in a register group: one,
some or all of a stage's group bits, shared angles, rotations without a
parameter of their own beside them, and stages of sweeps that hold other gates."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_09733_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-10   # bar of a double gradient: sums of up to 2 n terms of O(1)


# states smaller than a group and than a tile, one tile, several
@pytest.mark.parametrize("n", [1, 2, 3, 4, 11, 12, 14])
@pytest.mark.parametrize("tiling", [(0, 0, 0), (12, 3, 4)])
@pytest.mark.parametrize("mixed", [False, True])
def test_ry_gradients(n, tiling, mixed):
    from paper_2608_09733_amd import sv
    rng = np.random.default_rng(17 * n + mixed)
    ops, count = [], 0
    for layer in range(5):
        for q in range(n):
            kind = (layer + q) % 4
            if kind == 0:
                ops.append(I.Op("ry", (q,), params=(count,)))
                count += 1
            elif kind == 1:
                ops.append(I.Op("h", (q,)))
            elif kind == 2:
                ops += [I.Op("rz", (q,), params=(count,)), I.Op("ry", (q,), params=(max(count - 1, 0),))]
                count += 1
            if mixed and n > 1 and kind == 3:
                ops.append(I.Op("ry", (q,), ((q + 1) % n,), 1, (count,)))
                ops.append(I.Op("rxx", (q, (q + 1) % n), params=(count + 1,)))
                count += 2
        for q in range(n - 1):
            ops.append(I.Op("x", (q + 1,), (q,)) if layer % 2 else I.Op("z", (q + 1,), (q,)))
    circ = I.Circuit(n, ops, rng.uniform(0, 6, count))
    ham = I.tfim(n) if n > 1 else I.hamiltonian(1, [("X", [0], 0.7), ("Z", [0], 1.0)])
    st = sv.State(n, adjoint=True)
    st.set_adjoint_tiling(*tiling)
    e, g = st.adjoint_grad(circ.ops, circ.params, ham)
    st.close()
    er, gr = O.adjoint_grad(circ, ham)
    assert abs(e - er) <= TOL and np.max(np.abs(g - gr)) <= TOL
