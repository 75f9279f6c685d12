"""transform_state of a context on the split-x2 schedule: the passes, and so the bits, of the plane schedule
where the size has plane passes."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu

# N, precision, A/B update: the smallest and the largest size of each precision that takes the split-x2
# schedule instead of the plane schedule, odd radices, the A/B update's own variant
CASES = [(32, 0, False), (54, 0, False), (90, 0, False), (32, 1, False), (72, 1, False), (96, 1, False),
         (90, 1, True), (60, 0, True), (108, 0, True), (128, 0, True)]


@pytest.mark.parametrize("N,precision,ab", CASES)
def test_transform_state_has_the_bits_of_the_plane_schedule(N, precision, ab):
    import torch
    from paper_2211_10185_amd.solver import Solver
    a = 0.05
    p = S.Problem(N=N, a=a, m=1.5, kinetic=S.K_NR_SIN2, vkind=S.V_CORNELL, vparams=(0.4, 0.2, a / 2), k=2,
                  precision=precision, dt=1.5 * a * a / 8 if ab else a / 8, seed=N,
                  scheme=S.SCHEME_AB if ab else S.SCHEME_SPLIT)
    print("transform_state, N", N, "precision", precision, "A/B", ab, flush=True)
    got = []
    for split in (True, False):
        s = Solver.from_problem(p, split=split, rowcol=False, split_variant=0, groups=1)
        s.set_states_noise(5)
        s.enable_kernel_timing(1)
        runs = []
        for sign in (-1, +1):
            s.transform_state(1, sign)
            runs.append(torch.view_as_real(s.state_tensor(1)).cpu().numpy().copy())
        # plane and column launches: one of each per transform, no row pass
        launches = [s.kernel_stats(c)[0] for c in (0, 1, 2)]
        got.append((runs, launches))
        s.close()
    assert got[0][1] == got[1][1] == [2, 0, 2]
    for x, y in zip(got[0][0], got[1][0]):
        assert np.isfinite(x).all() and np.array_equal(x, y)
