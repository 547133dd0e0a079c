"""The margin gate where its slices are few enough for one launch, and on both sides of that limit:
against the oracle, called again and again with other shapes in between (a launch leaves its
arrival counter at zero), and replayed from a graph between eager calls."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import mgo
from paper_2605_30218_amd import mg, synth

from _gpu_common import dev_i32

pytestmark = pytest.mark.gpu

# one row (64 slices), odd and tiny vocabularies, 256 slice states exactly, one slice a row, halved
# slices (by the word too), and past the limits: (8, 128257), (9, 128256), (48, 32064) by the slices' length,
# (200, 8192) by their number
SHAPES = [(1, 128256), (1, 2), (2, 5), (3, 1023), (4, 128257), (5, 128256), (5, 110001), (8, 128257), (9, 128256),
          (16, 32064), (17, 32064), (48, 32064), (64, 4096), (65, 4096), (128, 3000), (200, 8192), (256, 40)]


def logits(B, V, seed):
    rng = np.random.RandomState(seed)
    L = rng.standard_normal((B, V)).astype(np.float32)
    L[0, V - 1] = L[0].max()                       # ties: the lowest index wins
    if B > 1:
        L[1] = 0.25                                # all equal
    if B > 2:
        L[2, V // 2] = np.nan
    if B > 3:
        L[3] = -np.inf
    if B > 4:
        L[4] = np.finfo(np.float32).min
        L[4, V // 3] = np.inf
    return L


def outputs(B):
    return [torch.full((B,), -7, dtype=torch.int32, device="cuda"), torch.full((B,), -7.0, device="cuda"),
            torch.full((B,), 9, dtype=torch.uint8, device="cuda"), torch.full((B,), -7, dtype=torch.int32, device="cuda"),
            torch.full((1,), -7, dtype=torch.int32, device="cuda")]


def check(out, L, prot, tau):
    t, m, g, r = mgo.OracleModel.margin_gate(L, prot, tau)
    n = int(out[4].cpu())
    np.testing.assert_array_equal(out[0].cpu().numpy(), t)
    gm = out[1].cpu().numpy()
    np.testing.assert_array_equal(np.isnan(gm), np.isnan(m))
    np.testing.assert_array_equal(gm[~np.isnan(m)].view(np.uint32), m[~np.isnan(m)].view(np.uint32))
    np.testing.assert_array_equal(out[2].cpu().numpy(), g)
    np.testing.assert_array_equal(out[3].cpu().numpy()[:n], r)
    assert n == len(r)


def test_against_the_oracle_in_turn():
    for rnd in range(3):
        for B, V in SHAPES:
            L = logits(B, V, 10 * rnd + B)
            prot = (np.arange(B) % 5 != 3).astype(np.uint8)
            out = outputs(B)
            mg.margin_gate_noalloc(B, V, torch.as_tensor(L).cuda(), torch.as_tensor(prot).cuda(), 0.3, *out)
            torch.cuda.synchronize()
            check(out, L, prot, 0.3)


@pytest.mark.parametrize("B,V", [(1, 128256), (5, 4096)])
def test_graph_replays(B, V):
    L = [logits(B, V, s) for s in range(4)]
    buf = torch.as_tensor(L[0]).cuda()
    out = outputs(B)
    mg.margin_gate_noalloc(B, V, buf, None, 0.3, *out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mg.margin_gate_noalloc(B, V, buf, None, 0.3, *out)
    for k in range(4):
        buf.copy_(torch.as_tensor(L[k]))
        g.replay()
        torch.cuda.synchronize()
        check(out, L[k], None, 0.3)
        other = outputs(B)
        mg.margin_gate_noalloc(B, V, torch.as_tensor(L[k - 1]).cuda(), None, 0.3, *other)  # eager, in between
        torch.cuda.synchronize()
        check(other, L[k - 1], None, 0.3)


@pytest.mark.parametrize("B,V,launches", [(1, 128256, 1), (16, 4096, 1), (17, 4096, 2), (64, 4096, 2), (4, 32000, 1),
                                          (16, 32000, 2), (8, 128256, 2), (1, 131071, 1), (1, 152063, 2)])
def test_launches_in_a_graph(B, V, launches):
    """In a graph no launch costs the host anything, and above 64 slice states the single launch
    takes more of the GPU than the two: a captured gate is one launch up to there, two above (and
    for slices above 2048 values of rows that are no 16-byte multiple)."""
    L = [logits(B, V, s) for s in range(3)]
    buf = torch.as_tensor(L[0]).cuda()
    out = outputs(B)
    hip = ctypes.CDLL("libamdhip64.so")
    side = torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t(0)
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(side.cuda_stream), 2) == 0  # hipStreamCaptureModeRelaxed
    mg.margin_gate_noalloc(B, V, buf, None, 0.3, *out, stream=side)
    assert hip.hipStreamEndCapture(ctypes.c_void_p(side.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    run = ctypes.c_void_p()
    assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
    assert n.value == launches
    for k in range(3):
        buf.copy_(torch.as_tensor(L[k]))
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(run, ctypes.c_void_p(side.cuda_stream)) == 0
        torch.cuda.synchronize()
        check(out, L[k], None, 0.3)
    assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0


def test_contexts_that_take_turns_on_one_workspace():
    """Two contexts of one model for different batches over the same workspace, used in turn: neither's
    scratch is where the other keeps its gate's counters (a counter that is overwritten would leave the
    gate's outputs as they were)."""
    s = synth.TINY
    ws = synth.make_weights(s, seed=2)
    big, pages = 64, 4
    pt, n_pages = synth.make_page_table([16 * pages] * big, s.page_size, pages, seed=3)
    # (2 items of prefill: the small context's plan then ends inside the normalised rows of the big one's step)
    engs = [mg.Engine(s, ws, b, pages, n_pages, max_prefill=m) for b, m in ((big, 0), (2, 2))]
    assert engs[0].workspace.numel() >= engs[1].workspace.numel()
    lib, small = engs[1].lib, engs[1]
    lib.mg_destroy(small.ctx)
    assert lib.mg_create(ctypes.byref(small.cfg), small._wtab, small.kv_pool.data_ptr(), small.kv_pool.numel() * 2,
                         engs[0].workspace.data_ptr(), small.workspace.numel(), ctypes.byref(small.ctx)) == 0
    tok, pos, ptd = dev_i32(np.arange(big) % s.vocab), dev_i32(np.full(big, 16 * pages - 1)), dev_i32(pt)
    for rnd in range(3):
        for e, B in zip(engs, (big, 2)):
            lg = torch.empty((B, s.vocab), dtype=torch.float32, device="cuda")
            e.decode_step(B, tok, pos, ptd, lg)
            for f, n in zip(engs, (B, min(B, 2))):  # either context's gate after either one's step
                out = outputs(n)
                f.margin_gate(n, lg, None, 0.3, *out)
                torch.cuda.synchronize()
                check(out, lg[:n].cpu().numpy(), None, 0.3)
