"""The canonical RMSNorm, four waves to a row: widths at
the edges of the 64-group slices (one group, a slice, a slice and a group, four slices and around,
the largest), where waves have no, part of, or several slices of the output."""
import numpy as np
import pytest
import torch

from oracle import mgo
from paper_2605_30218_amd import mg, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [8, 504, 512, 520, 1024, 1544, 2040, 2048, 2056, 3584, 5128, 8184, 8192])
@pytest.mark.parametrize("n", [1, 7])
def test_rmsnorm_bitexact(n, d):
    x, g = synth.random_bf16((n, d), seed=d), synth.random_bf16((d,), seed=d + 1)
    dev = [torch.as_tensor(a.view(np.int16)).cuda() for a in (x, g)]
    y = mg.op_rmsnorm(*dev, 1e-5).cpu().numpy().view(np.uint16)
    for r in range(n):
        np.testing.assert_array_equal(y[r], mgo.rmsnorm(mgo.CANON, x[r], g, 1e-5), err_msg=f"row {r}")
