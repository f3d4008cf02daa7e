"""The way of a batch's image to the GPU: a small one goes by a kernel on the batch's own stream, the first of a batch object and
a large one by a copy on the pool's side stream."""
import ctypes

import numpy as np
import pytest

from workload import DT_BF16, Layout, make_act
from helpers import Case, raw_to_torch

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime that this process already has loaded."""
    import torch
    torch.cuda.init()
    with open("/proc/self/maps") as f:
        path = next(l.split()[-1] for l in f if "libamdhip64.so" in l)
    return ctypes.CDLL(path)


def test_a_pending_error_of_the_caller_does_not_fail_a_begin(oracle_mod):
    import torch
    lay = Layout((64,), (64,), DT_BF16)
    case = Case(oracle_mod, lay, [8, 16], [1.0, 1.0], 4096, 16, seed=1)
    case.gpool.set_option("batches_per_marker", 1)
    hip = _hip()
    t2a = np.array([0, 1, 1, 0], np.int32)
    for k in range(3):  # the first image goes by the side stream, the later ones by a kernel
        torch.cuda.synchronize()
        assert hip.hipSetDevice(9999) != 0  # an error that nobody has looked at yet
        batch = case.gpool.batch_begin(t2a, case.stream)
        hip.hipGetLastError()
        case.gpool.batch_end(batch)
    case.run(t2a, seed=1)
    case.close()


@pytest.mark.parametrize("tokens", [1, 64, 3000, 30000])
def test_every_way_gives_the_same_result(oracle_mod, tokens):
    """Two batches in turn through one recycled batch object (a kernel up to 128 KiB: 30,000 tokens have more) against the same
    batches as the first of new objects (side stream), bit for bit."""
    import torch
    lay = Layout((64,), (72,), DT_BF16)
    case = Case(oracle_mod, lay, [8, 16, 5], [1.0, 0.5, 2.0], 4096, 16, seed=2)
    pool = case.gpool
    pool.set_option("batches_per_marker", 1)
    rng = np.random.default_rng(tokens)
    x = raw_to_torch(make_act(rng, tokens, 64, DT_BF16), "cuda")
    maps = [rng.integers(-1, 3, tokens).astype(np.int32) for _ in range(2)]
    maps[0][0], maps[1][0] = 0, 1

    def results(batch):
        v = torch.full((tokens, case.max_rank), float("nan"), device="cuda")
        y = torch.zeros((tokens, 72), dtype=torch.int16, device="cuda")
        pool.delta(batch, 0, [x], [v], [y], case.stream)
        return v, y

    open_batches = [pool.batch_begin(m, case.stream) for m in maps]  # open together: two new objects
    want = [results(b) for b in open_batches]
    for b in open_batches:
        pool.batch_end(b)
    for k in range(6):
        torch.cuda.synchronize()
        batch = pool.batch_begin(maps[k % 2], case.stream)
        v, y = results(batch)
        pool.batch_end(batch)
        assert torch.equal(v, want[k % 2][0]) and torch.equal(y, want[k % 2][1])
    assert not torch.equal(want[0][1], want[1][1])
    case.run(maps[0], seed=3)
    case.close()
