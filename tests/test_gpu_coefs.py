"""Coefficient tables with more factors than the lanes that build them."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2608_09733_amd import inputs as I

pytestmark = pytest.mark.gpu

# max-abs bar of a double amplitude; a table entry is a product of up to 40
# unit factors, each rounded once
TOL = 1e-12


@pytest.mark.parametrize("group,count", [(3, 1), (3, 8), (3, 9), (3, 40), (4, 17), (5, 40)])
def test_tables_of_many_factors(group, count):
    from paper_2608_09733_amd import sv
    n = 7
    rng = np.random.default_rng(count)
    ops = [I.Op("ry", (q,), params=(q,)) for q in range(n)]
    for k in range(count):
        kind = ["rz", "s", "t", "p", "z"][k % 5]
        q = [int(v) for v in rng.permutation(group)[:2]]
        par = (n + k,) if kind in ("rz", "p") else ()
        ops.append(I.Op(kind, (q[0],), (q[1],) if k % 2 else (), k % 4 // 2 if k % 2 else None, par))
    ops += [I.Op("ry", (q,), params=(q,)) for q in range(n)]
    circ = I.Circuit(n, ops, rng.uniform(0, 2 * np.pi, n + count))
    st = sv.State(n)
    st.set_tiling(13, 3, group)
    st.run(circ)
    assert np.max(np.abs(st.to_numpy() - O.run_circuit(circ))) <= TOL
    st.close()
