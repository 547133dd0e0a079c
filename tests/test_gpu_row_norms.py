"""The canonical RMSNorm, four waves to a row: widths at the edges of the 64-group slices (one
group, a slice, a slice and a group, four slices and around, the largest), where waves have no,
part of, or several slices of the output; into a buffer of its own and in place."""
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


@pytest.mark.parametrize("d", [520, 4096, 8192])
def test_rmsnorm_in_place(d):
    n = 256  # enough rows that the waves of a row run apart
    x, g = (torch.as_tensor(synth.random_bf16(s, seed=d).view(np.int16)).cuda() for s in ((n, d), (d,)))
    want = mg.op_rmsnorm(x, g, 1e-5).clone()
    st = mg.load().mg_op_rmsnorm(n, d, x.data_ptr(), g.data_ptr(), 1e-5, x.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert torch.equal(x, want)
