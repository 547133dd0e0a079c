"""The fast path's attention where its tiling can go wrong: every count of query heads per KV
head (three or two copies of the head columns), both head sizes, contexts around the 16-position
page, the 32-position step and the four waves' shares, rows split over blocks, and more blocks
than the device holds (longest rows first).  The MLP is switched off and the embedding is small,
so a layer's output is its attention through the output projection; the oracle's plain mode runs
the same layer on the same cache.  Every cache slot past a row's position holds NaN: a slot that
is read by mistake shows at once."""
import numpy as np
import pytest
import torch

from oracle import mgo
from paper_2605_30218_amd import synth

from _gpu_common import Pair, dev_i32, normwise, u16

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 34, 48, 49, 64, 65, 97, 127, 128, 129, 130, 160, 161, 255, 257, 513, 600]
SPLIT = [1100, 3, 1025, 1024, 16, 900]  # 70 pages of capacity and few rows: splits of the positions


def check(hd, G, n_kv, ctx, cap, seed=3):
    s = synth.ModelShape("attn", 1, 256, G * n_kv, n_kv, hd, 64, 256, bool(G & 1), 1e4, 1e-5)
    ws = synth.make_weights(s, seed=seed)
    ws[0] = (ws[0].view(torch.bfloat16).float() * 1e-3).to(torch.bfloat16).view(torch.int16)  # the residual: negligible
    ws[12].zero_()                                                                            # w_down: no MLP
    B = len(ctx)
    pair = Pair(s, max_batch=B, ctx_cap=cap, seed=seed, weights=ws)
    pos = np.asarray(ctx, np.int32) - 1
    kv = pair.eng.kv_view()
    synth.fill_synthetic_kv(kv, np.arange(pair.n_pages), seed=seed)
    nan = torch.tensor(0x7fc0, dtype=torch.int16, device="cuda")
    slot = torch.arange(cap, device="cuda")
    pt = torch.as_tensor(pair.pt).long().cuda()
    for r in range(B):
        past = slot[int(pos[r]):]
        kv[:, pt[r, past // 16], :, :, past % 16] = nan
    pair.sync_oracle_cache()
    tok = np.arange(B, dtype=np.int32) % s.vocab
    taps = torch.empty((2, B, s.d_model), dtype=torch.int16, device="cuda")
    logits = torch.empty((B, s.vocab), dtype=torch.float32, device="cuda")
    pair.eng.decode_step_taps(B, dev_i32(tok), dev_i32(pos), dev_i32(pair.pt), logits, taps)
    torch.cuda.synchronize()
    x = u16(taps)
    ref = pair.om.layer(mgo.PLAIN, 0, x[0], pos, pair.pt)
    # attention and projection are each rounded to bf16 once: 2^-9 of the largest value apiece,
    # with room for their sum and the residual's rounding (3 x 2^-9)
    errs = [normwise(mgo.f32_from_bf16(x[1][r]), mgo.f32_from_bf16(ref[r])) for r in range(B)]
    bad = [(c, e) for c, e in zip(ctx, errs) if not e <= 6e-3]
    assert not bad, bad


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("G", range(1, 9))
def test_edges_of_pages_steps_and_waves(hd, G):
    check(hd, G, 2, EDGES, 640)


@pytest.mark.parametrize("hd,G", [(64, 1), (128, 4), (128, 5), (128, 7)])
def test_split_positions(hd, G):
    check(hd, G, 2, SPLIT, 1120)


@pytest.mark.parametrize("hd,G,B", [(64, 1, 256), (64, 6, 129), (128, 5, 131)])
def test_longest_rows_first(hd, G, B):
    rng = np.random.RandomState(B)
    check(hd, G, 4, [int(c) for c in rng.randint(1, 120, B)], 128)
