"""Which kernel a batch runs on (scps_get_launch_shape): the forms of paths 0 and 2
on both sides of the lines between them."""
import numpy as np
import pytest

import test_gpu_packed as P
from paper_1705_02180_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1705_02180_amd import scps
    return scps


# chain lengths, replicas, set_launch, what runs
SHAPES = [
    ([20], 48, None, ("wave", 4, 1)),
    ([20], 48, (2, 1), ("wave", 1, 1)),
    ([20], 2048, (2, 8), ("wave", 8, 1)),
    ([20], 2049, None, ("packed", 12, 1)),
    ([20], 2049, (2, 1), ("packed", 3, 1)),
    ([7], 12, None, ("packed", 36, 1)),
    ([7, 8], 12, None, ("wave", 4, 1)),
    ([33], 16, None, ("wave", 4, 1)),
    ([64], 2048, None, ("wave", 4, 1)),
    ([64], 2049, None, ("packed", 4, 1)),
    ([64], 16, (2, 8), ("wave", 8, 1)),
    ([64], 600, None, ("persistent", 1, 1)),
    ([65], 16, None, ("persistent", 1, 1)),
    ([161], 4, None, ("persistent", 1, 1)),       # too little work to split
    ([200], 4, None, ("split", 1, 8)),
    ([200], 64, None, ("split", 1, 4)),
    ([200], 85, None, ("split", 1, 3)),
    ([200], 86, None, ("persistent", 1, 1)),      # two workgroups each would save less than a launch
    ([200], 4, (0, 512), ("persistent", 1, 1)),
    ([200], 4, (1, 0), ("per step", 0, 0)),
    ([560], 128, None, ("split", 1, 2)),
    ([560], 129, None, ("persistent", 1, 1)),
    ([1600], 64, None, ("split", 1, 4)),
    ([1700], 4, None, ("per step", 0, 0)),
]


@pytest.mark.parametrize("sizes,R,launch,want", SHAPES, ids=str)
def test_launch_shape(S, sizes, R, launch, want):
    base = dict(I._base_params())
    w = I.Workload("shape", base, [P._system(n, "all", 3) for n in sizes], np.arange(R, dtype=np.int32) % len(sizes), 1)
    ctx = S.Context.from_workload(w, params=base)
    if launch:
        ctx.set_launch(*launch)
    got = ctx.get_launch_shape()
    path = ctx.get_launch()[0]
    ctx.close()
    assert got == want
    assert path == {"per step": 1, "persistent": 0, "split": 0, "packed": 2, "wave": 2}[want[0]]
