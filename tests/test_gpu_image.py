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
