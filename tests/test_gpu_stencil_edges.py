"""Single H_K^(0) steps on lattices whose last tiles hold rows past them, with states that end at the end of their
memory segment (150^3 x 8 complex128 states are 13 KB short of a multiple of 2 MiB): the bits of fused steps."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k,precision", [(8, 2, 1), (18, 1, 0), (26, 3, 1), (150, 8, 1)])
def test_single_steps_beside_the_end_of_their_memory(N, k, precision):
    import torch
    from paper_2211_10185_amd.solver import Solver
    a = 0.05
    p = S.Problem(N=N, a=a, m=1.5, kinetic=S.K_FDTD, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=k,
                  precision=precision, dt=1.5 * a * a / 8, seed=N)
    print("single steps, N", N, "k", k, "precision", precision, flush=True)
    got = []
    for fused in (True, False):
        s = Solver.from_problem(p, fused_stencil=fused)
        s.set_states_noise(7)
        s.evolve(2, p.dt)
        E = s.energies()
        got.append((E, [torch.view_as_real(s.state_tensor(i)).cpu().numpy().copy() for i in (0, k - 1)]))
        s.close()
    (E, psi), (E1, psi1) = got
    assert np.isfinite(E).all() and np.array_equal(E, E1)
    for x, y in zip(psi, psi1):
        assert np.array_equal(x, y)
