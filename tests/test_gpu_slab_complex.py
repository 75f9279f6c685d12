"""Complex potentials at the sizes whose slab pass has threads or fused stages of its own for a complex factor:
against the oracle, and the bits of the size's other tile shape where that has the same factors and line plans."""
import numpy as np
import pytest

import oracle as O
import synthetic as S
from compare import energy_errors, wavefunction_errors

pytestmark = pytest.mark.gpu

# N, precision, kinetic, states, variant, the variant with its bits
CASES = [(150, 0, S.K_REL, 1, 0, 1), (180, 0, S.K_NR_SIN2, 2, 0, 1), (180, 0, S.K_REL, 1, 1, 0),
         (192, 0, S.K_REL, 2, 0, 1), (216, 0, S.K_NR_P2, 2, 0, 1), (216, 1, S.K_REL, 1, 0, 1)]


@pytest.mark.parametrize("N,precision,kind,k,variant,other", CASES)
def test_complex_factor_kernels(N, precision, kind, k, variant, other):
    from paper_2211_10185_amd.solver import Solver
    a = 0.05
    p = S.Problem(N=N, a=a, m=1.5, kinetic=kind, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=k, vgrid_seed=1031,
                  precision=precision, dt=a / 8, steps=3, measure_every=2, seed=N)
    init = p.init_states()
    print("complex factor, N", N, "precision", precision, "kind", kind, "variant", variant, flush=True)
    got = []
    for v in (variant, other):
        s = Solver.from_problem(p, split=True, split_variant=v, groups=1)
        s.enable_kernel_timing(1)
        s.set_states(init)
        s.evolve(p.steps, p.dt)
        got.append(s.states())
        assert min(s.kernel_stats(5)[0], s.kernel_stats(6)[0]) > 0
        s.close()
    (E, psi), (E1, psi1) = got
    assert np.array_equal(E, E1) and np.array_equal(psi, psi1)
    ref = O.solve(p, init=init)
    # the bounds of every comparison with the oracle in each precision
    etol, wtol = ((1e-5, 1e-4), (1e-10, 1e-9))[precision]
    assert np.max(energy_errors(E, ref["energies"])) < etol, (E, ref["energies"])
    assert np.max(wavefunction_errors(psi, ref["states"], ref["energies"])) < wtol
