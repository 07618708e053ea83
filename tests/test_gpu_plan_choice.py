"""From 26 qubits on a plan is chosen by whether the state is |0..0>: both
plans, and that of a tiling that was set, give the same state."""
import numpy as np
import pytest

from paper_2608_09733_amd import inputs as I

pytestmark = pytest.mark.gpu


# bounds of a double and of a single amplitude, one from each of two plans
@pytest.mark.parametrize("dtype,tol", [("c128", 2e-12), ("c64", 2e-5)])
def test_plans_from_zero_from_a_state_and_of_a_set_tiling_agree(dtype, tol):
    import torch
    from paper_2608_09733_amd import sv
    n = 26
    circ = I.hea(n, 4, seed=5)
    oa = sv.OpArray(circ.ops)
    one = np.zeros(1 << n)
    one[0] = 1.0
    ref = None
    for how in ("zero", "state", "set"):
        st = sv.State(n, dtype)
        if how == "set":
            st.set_tiling(13, 4, 5)
        if how == "state":
            st.set_planes(one, np.zeros(1 << n))
        st.apply(None, circ.params, op_array=oa)
        re, im = st.re.clone(), st.im.clone()
        st.close()
        if ref is None:
            ref = re, im
            assert abs(float((re.double() ** 2 + im.double() ** 2).sum()) - 1.0) <= 1e-5
        assert float((re - ref[0]).abs().max()) <= tol and float((im - ref[1]).abs().max()) <= tol
    torch.cuda.empty_cache()


def test_a_gradient_on_a_full_plan_cache():
    from oracle import oracle as O
    from paper_2608_09733_amd import sv
    n = 4
    st = sv.State(n, adjoint=True)
    for k in range(64):   # as many plans as the handle keeps
        ops = [I.Op("ry", (q,), params=(0,)) for q in range(n)]
        ops += [I.Op("x" if k >> b & 1 else "z", (b % n,), ((b + 1) % n,)) for b in range(6)]
        st.apply(ops, np.array([0.3]))
    circ, ham = I.hea(n, 2, seed=1), I.tfim(n)
    st.reset()
    e, g = st.adjoint_grad(circ.ops, circ.params, ham)
    st.close()
    er, gr = O.adjoint_grad(circ, ham)
    assert abs(e - er) <= 1e-12 and np.max(np.abs(g - gr)) <= 1e-12


def test_gradients_of_as_many_circuits_as_the_cache_holds_keep_their_plans():
    import torch
    from paper_2608_09733_amd import sv
    n, count = 10, 32            # two plans each, 64 in all
    circ, ham = I.hea(n, 40, seed=1), I.tfim(n)
    oas = [sv.OpArray(circ.ops + [I.Op("x" if k >> b & 1 else "z", (b,), (b + 1,)) for b in range(5)])
           for k in range(count)]
    st = sv.State(n, adjoint=True)

    def one(oa):
        st.reset()
        st.adjoint_grad(None, circ.params, ham, op_array=oa)
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    first = one(oas[0])
    free = [one(oa) for oa in oas[1:]][-1]
    used = first - free          # device memory of 62 plans
    assert used > 0
    # dropping them would give that memory back
    assert max(one(oa) for oa in oas) - free < used // 4
    st.close()


@pytest.mark.parametrize("circ", [I.random_circuit(10, 30, seed=0, max_qubits=3), I.layered(11, 2, seed=3),
                                  I.hea(12, 1, seed=3)], ids=["mixed10", "layered11", "hea12"])
def test_a_density_matrix_given_as_zero_takes_the_plan_of_a_reset_one(circ):
    import torch
    from paper_2608_09733_amd import sv
    n = circ.n
    st = sv.State(2 * n)
    st.reset()
    st.dm_apply(circ.ops, circ.params)
    want = st.re.clone(), st.im.clone()
    one = np.zeros(1 << 2 * n)
    one[0] = 1.0
    st.set_planes(one, np.zeros(1 << 2 * n))
    st.dm_apply(circ.ops, circ.params)
    assert torch.equal(st.re, want[0]) and torch.equal(st.im, want[1])
    st.close()
