"""The arg-max that the acceptance takes from the output head's partial results, against the logits of the same call: blocks of one
node up to the largest, ragged batches whose rows start anywhere in a line of partial results, few and many column groups.  The
head compares sums before the row's scale (positive) is applied and the logits after it; columns whose logits differ by no more than
one rounding step (2^-22 of the value, twice 2^-23) may come out in either order, anything else is exact."""
import numpy as np
import pytest
import torch

import synth
from tests.helpers import announce

pytestmark = pytest.mark.gpu
SHAPE = synth.workload.ModelShape("accept-head", 1, 256, 2, 1, 128, 192, 8224, 10000.0, "bf16")       # 257 column tiles: the last part has one
SEED = 31


@pytest.mark.parametrize("ns", [(1,), (2, 1, 3), (8,) * 5, (64,), (33, 64, 5, 17), (64,) * 3, (9, 64, 64, 64, 64, 64)])
def test_argmax_of_every_row(ns):
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    announce(f"arg-max of the rows of blocks {ns}")
    rng = np.random.default_rng(len(ns) + ns[0])
    B, k, lens = len(ns), max(ns), [int(x) for x in np.random.default_rng(3).integers(1, 40, len(ns))]
    model = harness.build_model(SHAPE, SEED)
    batch = harness.Batch(model, SHAPE, [p + k for p in lens], max_rows=max(sum(ns), 64), seed=SEED)
    batch.prefill([rng.integers(0, SHAPE.vocab, p) for p in lens])
    tok = rng.integers(0, SHAPE.vocab, (B, k)).astype(np.int32)
    out = sev.verify_ex(model, batch.kv, lens, torch.tensor(tok, device="cuda"), k, draft_lens=list(ns), want_argmax=True, want_logits=True)
    torch.cuda.synchronize()
    logits, got = out["logits"].cpu().numpy(), out["row_argmax"].cpu().numpy()
    best = logits.max(axis=1)
    taken = logits[np.arange(len(got)), got]
    assert np.all(best - taken <= 2.0 ** -22 * np.abs(best))
    assert np.mean(got == logits.argmax(axis=1)) > 0.99 or len(got) < 100 and np.sum(got != logits.argmax(axis=1)) <= 1
