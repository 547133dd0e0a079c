"""The fast path's projection above 64 rows (K % 128 == 0) at the edges of its tiles: row counts
around the 64-row blocks, feature counts around 16-feature tiles and narrow blocks, one and
several 128-element units of K, split K, and the SwiGLU, fp32 and top-2 epilogues against groups of
16 rows, which only the other kernel takes (the same order of every sum, so the same bits)."""
import numpy as np
import pytest
import torch

from oracle import mgo
from paper_2605_30218_amd import mg, synth

from _gpu_common import FEPI_BF16, FastGemmArgs, Pair, dev_i32, fast_gemm_launcher, u16

pytestmark = pytest.mark.gpu


def to_dev(a):
    return torch.as_tensor(a.view(np.int16)).to("cuda")


@pytest.mark.parametrize("n", [65, 80, 127, 128, 129, 192, 193, 251, 256])
@pytest.mark.parametrize("N,K", [(16, 128), (48, 256), (4112, 384), (9232, 512), (37888, 256), (112, 8192), (2064, 4480)])
def test_small_integers_exact(n, N, K):
    """Every partial sum is an integer below 2^24: any order gives the exact sum."""
    X = synth.small_int_bf16((n, K), seed=n)
    W = synth.small_int_bf16((N, K), seed=N)
    Y = mg.op_linear(False, to_dev(X), to_dev(W)).cpu().numpy()
    ref = (torch.as_tensor(mgo.f32_from_bf16(X)).cuda().double() @ torch.as_tensor(mgo.f32_from_bf16(W)).cuda().double().T)
    np.testing.assert_array_equal(Y, ref.cpu().numpy().astype(np.float32))


@pytest.mark.parametrize("n", [16, 17, 33, 64])
@pytest.mark.parametrize("N", [16, 1040, 4096, 4112, 8192, 8208])
def test_few_features_at_up_to_64_rows(n, N):
    """Unsplit outputs on both sides of the 64 blocks of 64 features up to which 17 to 32 rows take it,
    and of the 128 for 33 to 64 rows."""
    X, W = synth.small_int_bf16((n, 512), seed=n), synth.small_int_bf16((N, 512), seed=N)
    Y = mg.op_linear(False, to_dev(X), to_dev(W)).cpu().numpy()
    ref = mgo.f32_from_bf16(X).astype(np.float64) @ mgo.f32_from_bf16(W).astype(np.float64).T
    np.testing.assert_array_equal(Y, ref.astype(np.float32))


@pytest.mark.parametrize("n", [17, 64, 65, 128, 129, 251])
@pytest.mark.parametrize("Nseg", [(16, 0, 0), (4096, 48, 16)])
def test_bf16_epilogue_at_every_row_count(n, Nseg):
    """The bf16 epilogue with its bias, which the wide kernel does not have, is computed above 64 rows
    too.  Small integers: the sum is exact, so the result is its bf16 rounding."""
    K, N = 256, sum(Nseg)
    X, W = synth.small_int_bf16((n, K), seed=n), synth.small_int_bf16((N, K), seed=N)
    b = synth.small_int_bf16((N,), seed=N + 1)
    x, w, bias, y = to_dev(X), to_dev(W), to_dev(b), torch.zeros((n, N), dtype=torch.int16, device="cuda")
    a = FastGemmArgs(X=x.data_ptr(), M=n, K=K, N=N, Y=y.data_ptr(), S=1, n_cu=256)
    j = 0
    for k, seg in enumerate(Nseg):
        a.Nseg[k] = seg
        if seg:
            a.W[k], a.bias[k] = w[j:].data_ptr(), bias[j:].data_ptr()
        j += seg
    assert fast_gemm_launcher("launch_fast_gemm")(a, FEPI_BF16, torch.cuda.current_stream().cuda_stream) == 0
    ref = mgo.f32_from_bf16(X).astype(np.float64) @ mgo.f32_from_bf16(W).astype(np.float64).T + mgo.f32_from_bf16(b)
    want = torch.as_tensor(ref.astype(np.float32)).to(torch.bfloat16).view(torch.int16)
    assert torch.equal(y.cpu(), want)


@pytest.mark.parametrize("F", [128, 400, 1024])
def test_matrix_core_verifier_bits_across_the_kernels(F):
    """The matrix-core verifier's logits, tokens and columns for n rows at once are those of the
    rows in groups of 16, with the logits and without; the groups' tokens come from the other
    kernel's top-2 epilogue, and equal those of its logits.  At 33 rows only the LM head is wide."""
    s = synth.ModelShape("wide", 2, 384, 6, 2, 64, F, 1040, True, 1e4, 1e-5)
    B = 201
    pair = Pair(s, max_batch=B, ctx_cap=48, seed=F)
    e = pair.eng
    synth.fill_synthetic_kv(e.kv_view(), np.arange(pair.n_pages), seed=1)
    rng = np.random.RandomState(F)
    tok, pos = dev_i32(rng.randint(0, s.vocab, B)), dev_i32(rng.randint(0, 48, B))
    pt = dev_i32(pair.pt)

    def run(rows, logits):
        n = len(rows)
        lg = torch.empty((n, s.vocab), device="cuda") if logits else None
        vt = torch.empty(n, dtype=torch.int32, device="cuda")
        vc = torch.empty((n, e.col_elems), dtype=torch.int16, device="cuda")
        e.verify_rows_mfma(n, dev_i32(rows), tok, pos, pt, lg, vt, vc)
        torch.cuda.synchronize()
        return (lg.cpu().numpy().view(np.uint32) if logits else np.zeros((n, 1))), vt.cpu().numpy(), u16(vc)

    groups = [np.arange(r, min(r + 16, B)) for r in range(0, B, 16)]
    parts = [run(g, True) for g in groups]
    want = [np.concatenate([p[k] for p in parts]) for k in range(3)]
    np.testing.assert_array_equal(np.concatenate([run(g, False)[1] for g in groups]), want[1])
    np.testing.assert_array_equal(want[1], want[0].view(np.float32).argmax(1))
    for n in (33, 65, 100, 130, B):
        for logits in (True, False):
            got = run(np.arange(n), logits)
            if logits:
                np.testing.assert_array_equal(got[0], want[0][:n])
            np.testing.assert_array_equal(got[1], want[1][:n])
            np.testing.assert_array_equal(got[2], want[2][:n])
