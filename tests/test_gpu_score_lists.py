"""k-lists of the matrix-core path around the sizes where their place and their
merge change: 32 entries (the longest with an LDS tail), blocks of 64 entries
in the wave-wide merge, more entries than a slice has rows; and rows in
ascending order of one query's scores, so that every block of 384 rows beats all before it
and fills the queues, against the oracle (acceptance rule of oracle/accept.py)."""
import numpy as np
import pytest

import synth
from gpu_harness import check_dedup, check_delivery, check_unique_topk, note, run_merge

pytestmark = pytest.mark.gpu


def _f32(bits: np.ndarray) -> np.ndarray:
    return (bits.astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("k", [32, 33, 64, 65, 129, 400])
@pytest.mark.parametrize("n_corpus,requests", [(30_000, 2048), (90_001, 40)])
def test_ascending_rows(k, n_corpus, requests):
    # 329 distinct queries in slices of one tile, and a single partial query tile
    w = synth.make("ridge1m", n_corpus=1, with_corpus=False)
    keys = w.keys[:requests]
    q, _ = synth.gaussian_rows(w.seed, synth.S_QUERY, 0, 64, "bf16",
                               row_ids=w.template_ids[:requests])
    c, _ = synth.gaussian_rows(w.seed, synth.S_CORPUS, n_corpus, 64, "bf16")
    c = c[np.argsort(_f32(c) @ _f32(q[0]))]
    note(f"ascending rows k={k} N={n_corpus} requests={requests}")
    m = run_merge(keys, q, c, k)
    ref = check_dedup(m, keys)
    check_unique_topk(m, ref, q, c, k, sel=np.arange(0, ref["n_unique"], 7))
    check_delivery(m, requests)


@pytest.mark.parametrize("enc", ["bf16", "fp8"])
@pytest.mark.parametrize("k", [33, 100])
def test_ascending_rows_in_long_slices(enc, k):
    # 2,197 distinct queries: 14 slices of 41 tiles, past the first publication
    # of order statistics by running items
    w = synth.make("fp8_20m", n_corpus=1, with_corpus=False)
    q, _ = synth.gaussian_rows(w.seed, synth.S_QUERY, 0, 32, "bf16", row_ids=w.template_ids)
    c, sc = synth.gaussian_rows(w.seed, synth.S_CORPUS, 220_000, 32, enc)
    by, _ = synth.gaussian_rows(w.seed, synth.S_CORPUS, 220_000, 32, "bf16")
    order = np.argsort(_f32(by) @ _f32(q[0]))
    c = c[order]
    scale = sc[order] if enc == "fp8" else None
    note(f"ascending rows, long slices, {enc} k={k}")
    m = run_merge(w.keys, q, c, k, scale=scale)
    ref = check_dedup(m, w.keys)
    check_unique_topk(m, ref, q, c, k, scale=scale, sel=np.arange(0, ref["n_unique"], 60))
    check_delivery(m, w.R)
