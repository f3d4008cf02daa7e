"""GPU parity of two small-launch paths: the cooperative shrink with two chunks of d_in under way (contractions of an odd and
an even number of whole chunks per wavefront, with and without a ragged end, 1 .. 4 tokens), and the cooperative
expand of the groups that a panel batch has besides its blocks of 64 tokens (on consecutive and on scattered pages)."""
import numpy as np
import pytest

from workload import DT_BF16, DT_F16, DT_F32, Layout
from helpers import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [DT_BF16, DT_F16, DT_F32])
@pytest.mark.parametrize("d_in", [512, 2048, 2056, 4096, 4608, 6144, 8200])
def test_cooperative_shrink_chunks(oracle_mod, dtype, d_in):
    ranks = [3, 8, 17, 32]
    lay = Layout((d_in,), (72,), dtype)
    elt = 4 if dtype == DT_F32 else 2
    need = sum(-(-(r * elt * (d_in + 72)) // 16384) for r in ranks)
    case = Case(oracle_mod, lay, ranks, [16.0 / r for r in ranks], 16384, need + 2, seed=31)
    case.kernel_modes = ((1 << 30, 8, 1, "pair"), (1 << 30, 8, 1, "delta"))
    case.run(np.array([0, 1, 1, 2, 2, 2, 3, 3, 3, 3, -1, 3], np.int32), seed=8)
    case.close()


@pytest.mark.parametrize("scattered", [False, True])
@pytest.mark.parametrize("dtype", [DT_BF16, DT_F16])
def test_rest_of_a_panel_batch(oracle_mod, dtype, scattered):
    ranks = [64, 8, 33, 5, 16, 100]
    lay = Layout((128, 264, 128), (520, 1032, 136), dtype)
    need = sum(-(-(r * 2 * (520 + 1688)) // 4096) for r in ranks)
    scales = [16.0 / r for r in ranks]
    if scattered:  # all of them: the panel blocks' adapters 0 and 5, and the rest's in front of, between and behind those
        case = Case.scattered(oracle_mod, lay, ranks, scales, 4096, seed=32, max_rank=101)
    else:
        case = Case(oracle_mod, lay, ranks, scales, 4096, need, seed=32, max_rank=101)
    # limits that take the cooperative kernel for the rest, the ordinary one, and the library's own
    case.kernel_modes = ((1 << 30, 1, 0, "pair"), (0, 1, 0, "pair"), (2500, 1, 0, "delta"))
    t2a = np.concatenate([np.repeat(np.arange(6, dtype=np.int32), [200, 3, 1, 40, 7, 70]), np.full(4, -1, np.int32)])
    np.random.default_rng(6).shuffle(t2a)
    case.run(t2a, seed=9)
    case.close()
