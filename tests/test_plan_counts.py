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


# The planner counts what every qubit would add to a tile or a group in one pass
# over the pending gates.  These plans are those of a search that counts for one
# qubit at a time: default tiling, two that are set, and from |0..0>.
PLANS = [
    (14, "layered", 8, [(3, 45), (3, 47), (3, 31), (3, 45)]),
    (23, "hea", 6, [(4, 60), (4, 60), (6, 39), (4, 60)]),
    (24, "layered", 20, [(17, 206), (20, 191), (23, 137), (17, 206)]),
    (26, "mixed", 150, [(19, 112), (19, 112), (25, 76), (19, 112)]),
    (27, "qft", 0, [(10, 177), (10, 177), (13, 72), (10, 179)]),
    (30, "layered", 20, [(26, 236), (26, 236), (27, 153), (22, 245)]),
]


@pytest.mark.parametrize("n,kind,arg,counts", PLANS, ids=[f"{p[1]}{p[0]}" for p in PLANS])
def test_plans_are_those_of_the_search_qubit_by_qubit(n, kind, arg, counts):
    from paper_2608_09733_amd import sv
    ops = (I.layered_structure(n, arg) if kind == "layered" else I.hea_structure(n, arg) if kind == "hea"
           else I.qft(n).ops if kind == "qft" else I.random_circuit(n, arg, seed=4).ops)
    assert [sv.plan_stats(n, ops), sv.plan_stats(n, ops, -1, 13, 5, 3), sv.plan_stats(n, ops, -1, 11, 3, 5),
            sv.plan_stats(n, ops, from_zero=True)] == counts


def test_a_state_of_25_qubits_has_a_plan_of_its_own():
    # 6 layers on a state that is not |0..0> took 2.6 ms with the plan from
    # |0..0> and 2.2 with this one; at 24 qubits one plan serves both
    from paper_2608_09733_amd import sv
    for n, one in ((24, True), (25, False)):
        ops = I.layered_structure(n, 6)
        assert (sv.plan_stats(n, ops) == sv.plan_stats(n, ops, from_zero=True)) == one


def test_22_qubits_keep_13_bit_tiles_where_12_bit_ones_take_many_more_sweeps():
    # 10 and 12 layers took 403 and 525 us in 12-bit tiles, 367 and 466 in 13-bit
    # ones; 8 layers are faster in 12-bit ones
    from paper_2608_09733_amd import sv
    for layers, tile, low in ((8, 12, 3), (10, 13, 5), (12, 13, 5)):
        ops = I.layered_structure(22, layers)
        small, whole = sv.plan_stats(22, ops, -1, 12, 3, 3), sv.plan_stats(22, ops, -1, 13, 5, 3)
        assert (3 * small[0] > 4 * whole[0]) == (tile == 13)
        assert sv.plan_stats(22, ops) == sv.plan_stats(22, ops, -1, tile, low, 3)
