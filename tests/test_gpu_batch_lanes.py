"""Batches whose members run on several streams: the bits of each member alone."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu


def members(precision):
    a = 0.05

    def prob(N, kind, k, K, scheme=S.SCHEME_SPLIT):
        return S.Problem(N=N, a=a, m=1.5, kinetic=kind, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=k,
                         precision=precision, dt=1.5 * a * a / 8 if scheme or kind == S.K_FDTD else a / 8, steps=12,
                         measure_every=K, seed=N + kind, scheme=scheme)
    # the stencil, planes (24 and 18 share launches), two split sizes with two members of one, A/B, and sizes
    # in three size groups: more kinds than streams
    return [prob(64, S.K_NR_SIN2, 2, 5), prob(40, S.K_FDTD, 1, 4), prob(24, S.K_REL, 3, 6), prob(18, S.K_NR_P2, 1, 5),
            prob(96, S.K_REL, 1, 5), prob(64, S.K_NR_P2, 1, 3), prob(50, S.K_NR_SIN2, 1, 5, S.SCHEME_AB),
            prob(30, S.K_FDTD, 2, 5)]


@pytest.mark.parametrize("precision", [S.PREC_C64, S.PREC_C128])
def test_batch_on_several_streams_has_the_bits_of_each_member_alone(precision):
    from paper_2211_10185_amd.solver import Solver, batch_energies, batch_evolve
    probs = members(precision)
    print("batch on several streams, precision", precision, flush=True)
    alone = []
    for p in probs:
        s = Solver.from_problem(p)
        s.set_states(p.init_states())
        for _ in range(4):
            s.evolve(12, p.dt)
        alone.append(s.states())
        s.close()
    ss = [Solver.from_problem(p) for p in probs]
    for s, p in zip(ss, probs):
        s.set_states(p.init_states())
    # direct launches, capture, replays, with eager work in between; the member that owns the streams leaves
    # after three rounds and is advanced on its own
    for _ in range(3):
        batch_evolve(ss, 12, [p.dt for p in probs])
        batch_energies(ss)
    ss[0].evolve(12, probs[0].dt)
    out = [ss[0].states()]
    ss[0].close()
    batch_evolve(ss[1:], 12, [p.dt for p in probs[1:]])
    out += [s.states() for s in ss[1:]]
    for s in ss[1:]:
        s.close()
    for (E, psi), (Ea, psia) in zip(out, alone):
        assert np.array_equal(E, Ea) and np.array_equal(psi, psia)
