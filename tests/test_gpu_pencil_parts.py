"""Pencil passes that exchange real and imaginary parts in turn: the bits of those that exchange whole values."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu

# N, precision, kinetic, states, A/B update: the sizes where variant 0 exchanges parts and variant 1 whole values
# with the same factors and plans; one, two and three stages per line, threads without a position
CASES = [(192, 0, S.K_REL, 1, False), (192, 0, S.K_NR_SIN2, 2, False), (240, 0, S.K_REL, 2, False),
         (240, 0, S.K_NR_P2, 1, False), (216, 1, S.K_REL, 1, False), (216, 1, S.K_NR_SIN2, 2, True)]


@pytest.mark.parametrize("N,precision,kind,k,ab", CASES)
def test_parts_have_the_bits_of_whole_values(N, precision, kind, k, ab):
    import torch
    from paper_2211_10185_amd.solver import Solver
    a = 0.05
    p = S.Problem(N=N, a=a, m=1.5, kinetic=kind, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=k,
                  precision=precision, dt=1.5 * a * a / 8 if ab else a / 8, seed=N,
                  scheme=S.SCHEME_AB if ab else S.SCHEME_SPLIT)
    print("pencil parts, N", N, "precision", precision, "kind", kind, "A/B", ab, flush=True)
    got = []
    for variant in (0, 1):
        s = Solver.from_problem(p, split=True, split_variant=variant, groups=1)
        s.set_states_noise(11)
        s.evolve(3, p.dt)
        E = s.energies()
        got.append((E, [torch.view_as_real(s.state_tensor(i)).cpu().numpy().copy() for i in range(k)]))
        s.close()
    (E, psi), (E1, psi1) = got
    assert np.isfinite(E).all() and np.array_equal(E, E1)
    for x, y in zip(psi, psi1):
        assert np.isfinite(x).all() and np.abs(x).max() > 0 and np.array_equal(x, y)
