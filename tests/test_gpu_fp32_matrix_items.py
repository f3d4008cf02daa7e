"""GPU parity of the fp32 matrix-core items at the edges of their tiles (16 tokens, 16 rows of A, 32-value runs of the
contraction, 16 rows of B, 64 columns per wavefront), with the thresholds forced and with the library's own rule on
both sides of its limit, and against the vector-ALU items' error: the parity tests' tolerances are fp32's own."""
import numpy as np
import pytest

from workload import DT_F32, Layout
from helpers import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,d_out", [(8, 8), (24, 56), (128, 64), (136, 264), (1000, 520), (2048, 2048)])
def test_tile_edges(oracle_mod, d_in, d_out):
    ranks = [1, 4, 15, 16, 17, 32, 33, 64, 100]
    groups = [1, 15, 16, 17, 31, 32, 33, 48, 65]
    lay = Layout((d_in, d_in), (d_out, 2 * d_out), DT_F32)
    need = sum(-(-(r * 4 * (2 * d_in + 3 * d_out)) // 16384) for r in ranks)
    case = Case(oracle_mod, lay, ranks, [16.0 / r for r in ranks], 16384, need + 4, seed=21, mfma_min_tokens=1)
    t2a = np.concatenate([np.full(n, a, np.int32) for a, n in enumerate(groups)] + [np.full(3, -1, np.int32)])
    np.random.default_rng(2).shuffle(t2a)
    case.evict(4)  # and one adapter on scattered pages
    case.evict(7)
    case.load(7)
    case.load(4)
    out = case.run(t2a, seed=3)
    for o in out:  # no further from the fp64 sums than fp32 sums in short chains are
        assert np.linalg.norm(o["v_got"] - o["v_ref"]) <= 3e-7 * np.linalg.norm(o["v_ref"])
        # y: v's error as above, a chain of up to 100 products (a chain of 512 has 4.1e-7, errors grow with the root: 1.8e-7), and the
        # final rounding (6e-8 of y, which is up to 1.5 times the delta): together 3.6e-7 of the delta
        delta = o["y_ref"].astype(np.float64) - o["y0"]
        assert np.linalg.norm(o["y_got"].astype(np.float64) - o["y_ref"]) <= 4e-7 * np.linalg.norm(delta)
    case.close()


# below the limit of 64 items; above it, with launches too small for them and large enough
@pytest.mark.parametrize("groups", [[200, 150, 90, 16], [900, 700, 500, 20],
                                    [1500, 1300, 903, 401]])
def test_own_choice(oracle_mod, groups):
    ranks = [16, 33, 8, 64]
    lay = Layout((264, 512), (136, 72), DT_F32)
    need = sum(-(-(r * 4 * (264 + 512 + 136 + 72)) // 4096) for r in ranks)
    case = Case(oracle_mod, lay, ranks, [1.0, -0.5, 2.0, 0.25], 4096, need + 2, seed=22)
    case.run(np.random.default_rng(5).permutation(np.repeat(np.arange(4, dtype=np.int32), groups)), seed=4)
    case.close()
