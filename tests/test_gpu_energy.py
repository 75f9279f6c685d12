"""The FP64 energy measurement against the oracle on states as set: every route of its sums."""
import numpy as np
import pytest

import oracle as O
import synthetic as S

pytestmark = pytest.mark.gpu

# N, kinetic, precision, states, complex V: the sizes without split-x2 kernels (the smallest and the largest),
# the smallest and ragged sizes with them, tiles of one and two planes, the walls' stencil
CASES = [(8, S.K_NR_P2, 1, 3, True), (30, S.K_REL, 0, 2, False), (32, S.K_NR_SIN2, 0, 8, True),
         (36, S.K_REL, 1, 1, False), (50, S.K_NR_P2, 0, 3, True), (90, S.K_REL, 1, 2, True),
         (128, S.K_NR_SIN2, 0, 2, True), (150, S.K_REL, 0, 1, False), (10, S.K_FDTD, 1, 8, True),
         (66, S.K_FDTD, 0, 3, False), (130, S.K_FDTD, 1, 1, True)]


@pytest.mark.parametrize("N,kind,precision,k,vc", CASES)
def test_energies_and_residuals_of_noise_match_oracle(N, kind, precision, k, vc):
    from paper_2211_10185_amd.solver import Solver
    a = 0.05
    p = S.Problem(N=N, a=a, m=1.5, kinetic=kind, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=k,
                  vgrid_seed=1031 if vc else None, precision=precision, dt=1e-4, steps=0, seed=N)
    init = p.init_states()
    print("energies, N", N, "kind", kind, "precision", precision, "k", k, flush=True)
    s = Solver.from_problem(p)
    s.set_states(init)
    r = s.residuals()
    E, psi = s.states()
    G = s.gram()
    s.close()
    start = init if precision else init.astype(np.complex64).astype(np.complex128)
    q, R = np.linalg.qr(start.reshape(k, -1).T)
    # sums of N^3 positive terms in FP64: relative error far below 1e-12
    assert np.allclose(r, np.abs(np.diag(R)), rtol=1e-12, atol=0)
    # the energies of exactly the states that the library returns
    ref = np.array(O.energies(list(psi), p.kinetic, p.a, p.m, O.problem_potential(p)))
    assert np.max(np.abs(E - ref) / np.abs(ref)) < 1e-12, (E, ref)
    assert np.allclose(G, psi.reshape(k, -1).conj() @ psi.reshape(k, -1).T, rtol=0, atol=1e-12)
