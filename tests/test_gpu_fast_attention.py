"""The fast path's attention where its tiling can go wrong: every count of query heads per KV
head (three or two copies of the head columns), both head sizes, contexts around the 16-position
page, the 32-position step and the four waves' shares, rows split over blocks (an inner split that
ends on half a step among them), more blocks than the device holds (longest rows first), more
pages in one block than its LDS holds, and rows that share pages.  The MLP is switched off and the embedding is small,
so a layer's output is its attention through the output projection; the oracle's plain mode runs
the same layer on the same cache.  Every cache slot past a row's position holds NaN: a slot that
is read by mistake shows at once."""
import numpy as np
import pytest
import torch

from oracle import mgo
from paper_2605_30218_amd import mg, synth

from _gpu_common import Pair, dev_i32, normwise, u16

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 34, 48, 49, 64, 65, 97, 127, 128, 129, 130, 160, 161, 255, 257, 513, 600]
SPLIT = [1100, 3, 1025, 1024, 16, 900]  # 70 pages of capacity and few rows: splits of the positions
# 68 pages in 4 splits of 17: each ends after the first page of a 32-position step
ODD_SPLIT = [1088, 273, 274, 288, 289, 545, 546, 560, 561, 817, 818, 833, 5]


class SharedPrefix(Pair):
    """A Pair whose rows share their first `shared` pages and have the others for themselves."""

    def __init__(self, shape, max_batch, ctx_cap, shared, seed, weights):
        self.shape, self.max_batch, self.maxp = shape, max_batch, ctx_cap // 16
        own = self.maxp - shared
        self.n_pages = shared + own * max_batch
        perm = np.random.RandomState(seed).permutation(self.n_pages).astype(np.int32)
        self.pt = np.concatenate([np.tile(perm[:shared], (max_batch, 1)), perm[shared:].reshape(max_batch, own)], 1)
        self.eng = mg.Engine(shape, weights, max_batch, self.maxp, self.n_pages)
        self.om = mgo.OracleModel(shape, synth.weights_to_numpy(weights), max_batch, self.maxp, self.n_pages)


def check(hd, G, n_kv, ctx, cap, seed=3, shared=0, tol=6e-3):
    s = synth.ModelShape("attn", 1, 256, G * n_kv, n_kv, hd, 64, 256, bool(G & 1), 1e4, 1e-5)
    ws = synth.make_weights(s, seed=seed)
    ws[0] = (ws[0].view(torch.bfloat16).float() * 1e-3).to(torch.bfloat16).view(torch.int16)  # the residual: negligible
    ws[12].zero_()                                                                            # w_down: no MLP
    B = len(ctx)
    pair = SharedPrefix(s, B, cap, shared, seed, ws) if shared else Pair(s, max_batch=B, ctx_cap=cap, seed=seed, weights=ws)
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
    bad = [(c, e) for c, e in zip(ctx, errs) if not e <= tol]
    assert not bad, bad


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("G", range(1, 9))
def test_edges_of_pages_steps_and_waves(hd, G):
    check(hd, G, 2, EDGES, 640)


@pytest.mark.parametrize("hd,G", [(64, 1), (128, 4), (128, 5), (128, 7)])
def test_split_positions(hd, G):
    check(hd, G, 2, SPLIT, 1120)


@pytest.mark.parametrize("hd,G", [(64, 1), (128, 4), (128, 5), (128, 7)])
def test_split_ends_on_half_a_step(hd, G):
    check(hd, G, 2, ODD_SPLIT, 1088)


@pytest.mark.parametrize("hd,G", [(64, 2), (128, 4), (128, 7)])
def test_split_positions_of_a_full_device(hd, G):
    """32 rows x 2 KV heads x 4 splits: a block per CU and more, whose K/V loads are streamed."""
    rng = np.random.RandomState(G)
    check(hd, G, 2, ODD_SPLIT + [int(c) for c in rng.randint(1, 1089, 32 - len(ODD_SPLIT))], 1088)


@pytest.mark.parametrize("hd,G", [(64, 1), (128, 2)])
def test_more_pages_than_the_block_holds(hd, G):
    """512 (row, KV head) blocks are not split: contexts above 16384 positions, whose page indices
    are read from memory, next to the longest one whose indices fit.  Of 64 rows x 256 outputs one or
    two of the largest round to neighbouring bf16 values on the two sides: a step of 2^-7 of the value, and 2^-9
    for what the attention's own rounding moves before (a page left out of 17000 positions would show
    as 3e-2, sqrt(16 / 17000))."""
    B = 64
    ctx = [16385, 16386, 16401, 17600] + [int(c) for c in np.random.RandomState(hd).randint(16386, 17601, B - 4)]
    check(hd, G, 8, ctx, 17600, shared=1020, tol=2.0 ** -7 + 2.0 ** -9)


@pytest.mark.parametrize("hd,G,B", [(64, 2, 40), (128, 4, 140)])
def test_rows_that_share_pages(hd, G, B):
    rng = np.random.RandomState(B)
    check(hd, G, 4, [int(c) for c in rng.randint(129, 241, B)], 240, shared=8)


@pytest.mark.parametrize("value", [0x7f80, 0xff80])
def test_an_infinity_in_v_reaches_the_gate_as_nan(value):
    """A probability is multiplied as the sum of three terms, of which the lower may be zero, so an
    infinite V gives the attention a NaN where one product would give an infinity.  The next norm
    makes NaN of either: the row's logits are NaN, as the oracle's, and its gate fires; the other
    rows are as without."""
    s, B, cap = synth.TINY, 6, 64
    pair = Pair(s, max_batch=B, ctx_cap=cap, seed=9)
    ctx = np.asarray([33, 64, 17, 40, 49, 20], np.int32)
    kv = pair.eng.kv_view()
    synth.fill_synthetic_kv(kv, np.arange(pair.n_pages), seed=9)
    inf = torch.tensor(value - 65536 if value & 0x8000 else value, dtype=torch.int16, device="cuda")
    bad = [1, 4]
    for r in bad:
        kv[0, int(pair.pt[r, 1]), 1, 0, 5, 7] = inf  # position 21: layer 0, V of head 0, one value
    pair.sync_oracle_cache()
    tok = np.arange(B, dtype=np.int32)
    lg = torch.empty((B, s.vocab), dtype=torch.float32, device="cuda")
    pair.eng.decode_step(B, dev_i32(tok), dev_i32(ctx - 1), dev_i32(pair.pt), lg)
    i32 = dict(dtype=torch.int32, device="cuda")
    top1, rows, n = torch.empty(B, **i32), torch.empty(B, **i32), torch.empty(1, **i32)
    margin, gate = torch.empty(B, device="cuda"), torch.empty(B, dtype=torch.uint8, device="cuda")
    pair.eng.margin_gate(B, lg, None, 0.0, top1, margin, gate, rows, n)
    torch.cuda.synchronize()
    got, ref = lg.cpu().numpy(), pair.om.decode_step(mgo.PLAIN, tok, ctx - 1, pair.pt)
    for r in range(B):
        assert np.isnan(got[r]).all() == np.isnan(ref[r]).all() == (r in bad), r
        if r not in bad:
            assert normwise(got[r], ref[r]) <= 1e-2
    assert np.isnan(margin.cpu().numpy()).tolist() == [r in bad for r in range(B)]
    assert gate.cpu().tolist() == [int(r in bad) for r in range(B)] and rows.cpu().tolist()[:int(n)] == bad


@pytest.mark.parametrize("hd,G,B", [(64, 1, 256), (64, 6, 129), (128, 5, 131), (128, 4, 130), (128, 7, 133)])
@pytest.mark.parametrize("cap,hi", [(128, 120), (512, 120), (528, 528)])
def test_longest_rows_first(hd, G, B, cap, hi):
    """512 positions of capacity and more: the longest first (many rows of equal length among them; and
    1 to capacity positions); below, the rows' own order."""
    rng = np.random.RandomState(B)
    ctx = [int(c) for c in rng.randint(1, hi, B)]
    ctx[B // 2], ctx[B // 3] = hi, 1
    check(hd, G, 4, ctx, cap)
