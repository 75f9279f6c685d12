"""Fused H_K^(0) steps at the edges of their tiles (32 x 13 sites, 2 to 32 planes), both precisions: the bits
of single steps."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu

# the smallest lattice, one tile exactly or one site more or less per axis, marches of 2 to 32 planes
# with whole and partial last ones, a last march of one plane, one to eight states, odd chunks
CASES = [(8, 1, 0, False, 2), (10, 8, 1, True, 3), (12, 1, 1, False, 5), (14, 2, 0, True, 4), (26, 1, 0, False, 7),
         (32, 3, 1, False, 4), (34, 2, 0, True, 5), (66, 1, 1, True, 3), (98, 3, 0, False, 4), (130, 1, 0, True, 2),
         (130, 3, 1, False, 2), (194, 2, 0, False, 2), (226, 4, 0, False, 3), (80, 3, 0, False, 3), (96, 3, 0, True, 2),
         (112, 2, 1, False, 3), (88, 5, 1, True, 2)]


@pytest.mark.parametrize("N,k,precision,vc,steps", CASES)
def test_fused_stencil_steps_have_the_bits_of_single_steps(N, k, precision, vc, steps):
    import torch
    from paper_2211_10185_amd.solver import Solver
    a = 0.05
    p = S.Problem(N=N, a=a, m=1.5, kinetic=S.K_FDTD, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=k,
                  vgrid_seed=1031 if vc else None, precision=precision, dt=1.5 * a * a / 8, seed=N)
    print("fused stencil, N", N, "k", k, "precision", precision, "complex V", vc, flush=True)
    got = []
    for fused in (True, False):
        s = Solver.from_problem(p, fused_stencil=fused)
        s.set_states_noise(7)
        s.evolve(steps, p.dt)
        E = s.energies()
        got.append((E, [torch.view_as_real(s.state_tensor(i)).cpu().numpy().copy() for i in range(k)]))
        s.close()
    (E, psi), (E1, psi1) = got
    assert np.isfinite(E).all() and np.array_equal(E, E1)
    for x, y in zip(psi, psi1):
        assert np.array_equal(x, y)
