"""Complex128 on the split-x2 schedule against the oracle: the sizes and tile shapes that the other complex128
tests leave out, and the schedules that a solve of several states takes by default (state groups on streams of
their own, no timing), the A/B update among them."""
import numpy as np
import pytest

import oracle as O
import synthetic as S
from compare import energy_errors, wavefunction_errors

pytestmark = pytest.mark.gpu


def problem(N, kind, vkind, k, ab, steps):
    a, m = 0.05, 1.5
    vp = (0.4, 0.2, a / 2) if vkind == S.V_CORNELL else (1.0,)
    dt = 0.9 * 2 / (np.sqrt(12 / a ** 2 + m * m) - m) if ab and kind == S.K_REL else (m * a * a / 8 if ab else a / 8)
    return S.Problem(N=N, a=a, m=m, kinetic=kind, vkind=vkind, vparams=vp, k=k,
                     vgrid_seed=1031 if vkind == S.V_CORNELL else None, precision=S.PREC_C128, dt=dt, steps=steps,
                     measure_every=2, seed=N + k, scheme=S.SCHEME_AB if ab else S.SCHEME_SPLIT)


def check(p, init, E, psi):
    ref = O.solve(p, init=init)
    # the bounds of every complex128 comparison with the oracle
    assert np.max(energy_errors(E, ref["energies"])) < 1e-10, (E, ref["energies"])
    assert np.max(wavefunction_errors(psi, ref["states"], ref["energies"])) < 1e-9


SHAPES = [(72, S.K_REL, S.V_CORNELL, 2, 0), (72, S.K_NR_P2, S.V_HARMONIC, 1, 1), (80, S.K_NR_SIN2, S.V_HARMONIC, 2, 0),
          (80, S.K_REL, S.V_CORNELL, 1, 1), (180, S.K_REL, S.V_HARMONIC, 1, 0), (216, S.K_NR_SIN2, S.V_CORNELL, 1, 0),
          (216, S.K_REL, S.V_HARMONIC, 1, 1), (240, S.K_REL, S.V_CORNELL, 1, 0)]


@pytest.mark.parametrize("N,kind,vkind,k,variant", SHAPES)
def test_shape_matches_oracle(N, kind, vkind, k, variant):
    from paper_2211_10185_amd.solver import Solver
    p = problem(N, kind, vkind, k, False, 3)
    init = p.init_states()
    print("complex128 shape, N", N, "kind", kind, "variant", variant, flush=True)
    s = Solver.from_problem(p, split=True, split_variant=variant, groups=1)
    s.enable_kernel_timing(1)
    s.set_states(init)
    s.evolve(p.steps, p.dt)
    E, psi = s.states()
    assert min(s.kernel_stats(5)[0], s.kernel_stats(6)[0]) > 0
    s.close()
    check(p, init, E, psi)


# two and three groups, even and uneven ones, of one and of several states each
GROUPS = [(72, S.K_REL, S.V_CORNELL, 3, False), (80, S.K_NR_P2, S.V_HARMONIC, 2, False), (90, S.K_NR_SIN2, S.V_CORNELL, 4, False),
          (100, S.K_REL, S.V_HARMONIC, 5, False), (150, S.K_NR_SIN2, S.V_CORNELL, 2, False),
          (180, S.K_REL, S.V_CORNELL, 3, False), (100, S.K_NR_SIN2, S.V_CORNELL, 3, True), (160, S.K_REL, S.V_HARMONIC, 2, True)]


@pytest.mark.parametrize("N,kind,vkind,k,ab", GROUPS)
def test_default_schedule_of_several_states_matches_oracle(N, kind, vkind, k, ab):
    from paper_2211_10185_amd.solver import Solver
    p = problem(N, kind, vkind, k, ab, 5)
    init = p.init_states()
    s = Solver.from_problem(p)
    print("complex128 default schedule, N", N, "kind", kind, "k", k, "A/B", ab, s.schedule, flush=True)
    assert s.schedule["split"] and s.schedule["groups"] >= 2
    s.set_states(init)
    s.evolve(p.steps, p.dt)      # captured chunks of two steps, replayed, and one of one step
    E, psi = s.states()
    s.close()
    check(p, init, E, psi)


@pytest.mark.parametrize("N,kind,k", [(120, S.K_NR_SIN2, 1), (162, S.K_REL, 2)])
def test_default_ab_schedule_with_the_second_shape_matches_oracle(N, kind, k):
    from paper_2211_10185_amd.solver import Solver
    p = problem(N, kind, S.V_CORNELL, k, True, 3)
    init = p.init_states()
    s = Solver.from_problem(p)
    print("complex128 A/B, N", N, "kind", kind, s.schedule, flush=True)
    assert s.schedule["split"] and s.schedule["split_variant"] == 1
    s.set_states(init)
    s.evolve(p.steps, p.dt)
    E, psi = s.states()
    s.close()
    check(p, init, E, psi)
