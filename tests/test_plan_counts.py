"""The plan query counts the sweeps that a call launches: circuits of Kronecker
stages and of all kinds, from |0..0> and from another state."""
import pytest

from paper_2608_09733_amd import inputs as I


# below one tile, a few tiles, on both sides of the size from which a reset
# handle's plan is its own
@pytest.mark.gpu
@pytest.mark.parametrize("n", [6, 14, 20, 25, 26])
@pytest.mark.parametrize("kind", ["layered", "mixed"])
def test_sweeps_counted_are_those_launched(n, kind):
    from paper_2608_09733_amd import sv
    circ = I.layered(n, 8, seed=1) if kind == "layered" else I.random_circuit(n, 90, seed=n)
    oa = sv.OpArray(circ.ops)
    st = sv.State(n)
    st.timing(True)
    for zero in (True, False):   # the second call starts from the first one's state
        st.apply(None, circ.params, op_array=oa)
        launches = st.timing_read()[1]
        assert launches == sv.plan_stats(n, circ.ops, from_zero=zero)[0]
    st.close()


def test_blocks_of_gates_that_are_written_as_others():
    from paper_2608_09733_amd import sv
    # RX = S^dag RY S on three qubits is one Kronecker stage; a double excitation
    # is two fans of three CX around a rotation under three controls, one of
    # which is no part of its register group
    assert sv.plan_stats(12, [I.Op("rx", (q,), params=(q,)) for q in (1, 4, 9)]) == (1, 1)
    assert sv.plan_stats(12, [I.Op("dexc", (1, 4, 9, 11), params=(0,))])[1] > 1
