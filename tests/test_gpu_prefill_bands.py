"""The canonical prefill over more rows than one band of the matrix-core GEMV's block order (8 row
tiles of 32): whole bands, a last band of one tile and of several, feature groups that do not
divide over the 8 XCDs (688 outputs), against the same prompts in calls of at most 64 items --
bit for bit, as an item's result depends on neither the call nor its place in it."""
import numpy as np
import pytest

from paper_2605_30218_amd import mg, synth
from paper_2605_30218_amd.runtime import prefill_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("items", [256, 257, 300, 513, 700, 1024])
def test_prefill_cache_independent_of_items_per_call(items):
    s, R = synth.TINY, 16
    ws = synth.make_weights(s, seed=4)
    length = -(-items // R) + 1
    pt, n_pages = synth.make_page_table([length + 16] * R, s.page_size, -(-(length + 16) // s.page_size), seed=6)
    prompts = synth.make_prompts(R, [length - (r >= (items - 1) % R + 1) for r in range(R)], s.vocab, seed=items)
    assert sum(len(p) - 1 for p in prompts) == items
    caches = []
    for per_call in (1024, 64):
        eng = mg.Engine(s, ws, R, pt.shape[1], n_pages)
        prefill_rows(eng, prompts, pt, max_items=per_call)
        caches.append(eng.kv_pool.cpu().numpy())
        eng.close()
    assert np.any(caches[0])
    np.testing.assert_array_equal(caches[0], caches[1])
