"""GPU parity of the panel shrink items (up to 64 tokens x 64 rows of A per workgroup), as such and cut over four
workgroups as in launches that they would not fill the GPU with, at the edges of their tiles:
tokens around 32 / 33 / 64 / 65 / 128, ranks around 16 / 32 / 33 / 64 / 65 / 128 / 129, the shortest contractions (fewer
steps than the kernel keeps in flight), the block of 16 steps whose sums are collected, adapters on consecutive and on
scattered pages, q, k, v that read one x; against the fp64-accumulating oracle with the parity tests' tolerances, and
v bit for bit between one call over all slots and a call over one (the order of the workgroups must not matter)."""
import numpy as np
import pytest

from workload import DT_BF16, DT_F16, Layout
from helpers import Case

pytestmark = pytest.mark.gpu

# (coop limit, panel_min_blocks, mfma_shrink_depth, entry points): the library's own choices; the expand is not the subject
MODES = ((0, 8, 0, "pair"),)


CUT = pytest.mark.parametrize("limit", [0, 1], ids=["panel", "cut"])  # 1: these launches are too small for whole items


def _case(oracle_mod, dtype, d_in, ranks, page, limit, scattered=False):
    n = len(d_in)
    lay = Layout(tuple(d_in), (136,) * n, dtype)
    need = sum(-(-(r * 2 * (sum(d_in) + 136 * n)) // page) for r in ranks)
    scales = [16.0 / r for r in ranks]
    if scattered:
        case = Case.scattered(oracle_mod, lay, ranks, scales, page, seed=11)
    else:
        case = Case(oracle_mod, lay, ranks, scales, page, need, seed=11)
    case.kernel_modes = MODES
    case.gpool.set_option("panel_min_tiles_shrink", limit)
    return case


@CUT
@pytest.mark.parametrize("scattered", [False, True], ids=["consecutive", "scattered"])
@pytest.mark.parametrize("dtype", [DT_BF16, DT_F16])
@pytest.mark.parametrize("d_in", [64, 128, 192, 1024, 1088, 4096])
def test_tile_edges(oracle_mod, dtype, d_in, scattered, limit):
    ranks = [8, 16, 17, 32, 33, 64, 65, 128, 129, 200]
    groups = [33, 64, 65, 100, 128, 129, 192, 33, 63, 97]
    case = _case(oracle_mod, dtype, [d_in], ranks, 4096 if scattered else 16384, limit, scattered)
    t2a = np.concatenate([np.full(n, a, np.int32) for a, n in enumerate(groups)] + [np.full(5, -1, np.int32)])
    np.random.default_rng(3).shuffle(t2a)
    case.run(t2a, seed=5)
    case.close()


@CUT
@pytest.mark.parametrize("dtype", [DT_BF16, DT_F16])
@pytest.mark.parametrize("page", [4096, 65536])
def test_scattered_pages_and_shared_x(oracle_mod, page, dtype, limit):
    ranks = [64, 24, 128, 8, 40, 65]
    case = _case(oracle_mod, dtype, [1024, 1024, 1024, 512], ranks, page, limit, scattered=True)
    t2a = np.repeat(np.arange(6, dtype=np.int32), [70, 64, 40, 130, 33, 200])
    np.random.default_rng(4).shuffle(t2a)
    whole = case.run(t2a, seed=6, share_x=[(0, 1, 2)])
    for s in range(4):
        one = case.run(t2a, slots=[s], seed=6, xs=[whole[s]["x"]])
        assert np.array_equal(one[0]["v_got"], whole[s]["v_got"])
    case.close()


def test_few_tiles_and_odd_contractions_keep_the_split_items(oracle_mod):
    """Below the limit, and where a contraction is no whole number of steps, the split items run; both must stay right."""
    for d_in, limit in ((1000, 0), (1024, 1 << 30), (1024, -1)):
        case = _case(oracle_mod, DT_BF16, [d_in], [16, 100], 16384, limit)
        case.run(np.repeat(np.arange(2, dtype=np.int32), [70, 150]), seed=7)
        case.close()
