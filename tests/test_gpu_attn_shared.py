"""The attention of requests with many query rows (four row groups per block, K/V through LDS): row counts around the block
of 128 rows and its waves, prefixes around a page and a page pair, whole sequences and chunks, chains and trees, ragged
batches that mix both sizes of blocks, against the oracle.  Also an appended block whose rows see only part of it.
Tolerances as for every bf16 path here: the logits of a two-plane forward are within 3e-2 (mean 3e-3), measured 1e-3."""
import numpy as np
import pytest
import torch

import synth
from oracle import verify_oracle as vo
from tests.helpers import announce, oracle_model

pytestmark = pytest.mark.gpu
SHAPE, SEED = synth.MINI_BF16.with_layers(2), 909           # 4 query heads per KV head: 24 nodes are 96 rows, 32 are 128


@pytest.fixture(scope="module")
def setup():
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    return sev, harness, harness.build_model(SHAPE, SEED), oracle_model(SHAPE, SEED, dtype=np.float32)


@pytest.mark.parametrize("lens,ns,tree", [
    ([1], (24,), False), ([15, 16, 17], (32, 31, 25), False), ([31, 33], (64, 64), True), ([700, 5, 130], (64, 57, 32), True),
    ([1500], (33,), False), ([257, 90], (64, 24), False), ([64, 480, 31, 9], (32, 64, 63, 24), True)])
def test_blocks(setup, lens, ns, tree):
    sev, harness, model, om = setup
    rng = np.random.default_rng(sum(lens) + len(ns))
    B, k = len(ns), max(ns)
    announce(f"shared attention: prefixes {lens}, nodes {ns}, trees {tree}")
    prompts = [rng.integers(0, SHAPE.vocab, p) for p in lens]
    batch = harness.Batch(model, SHAPE, [p + k for p in lens], max_rows=max(sum(ns), 128), seed=SEED)
    batch.prefill(prompts)
    caches = [vo.prefill(om, p, len(p) + k) for p in prompts]
    for b, p in enumerate(lens):                             # prefilled in chunks of at most 128 rows or sum(ns)
        for got, ref in zip(batch.export_kv(b, 1, 0, p), (caches[b].K[1][:p], caches[b].V[1][:p])):
            assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 2e-3)
    par = np.full((B, k), -1, dtype=np.int32)
    tok = rng.integers(0, SHAPE.vocab, (B, k)).astype(np.int32)
    for b, n in enumerate(ns):
        par[b, :n] = [int(rng.integers(max(-1, j - 6), j)) if tree else j - 1 for j in range(n)]
    out = sev.verify_ex(model, batch.kv, lens, torch.tensor(tok, device="cuda"), k, draft_lens=list(ns),
                        parents=torch.tensor(par, device="cuda") if tree else None, want_argmax=True, want_logits=True)
    torch.cuda.synchronize()
    want = np.concatenate(vo.forward_blocks(om, caches, [tok[b, :n] for b, n in enumerate(ns)], [par[b, :n] for b, n in enumerate(ns)])[0])
    diff = np.abs(out["logits"].cpu().numpy() - want)
    announce(f"  logits max {diff.max():.2e} mean {diff.mean():.2e}")
    assert diff.max() < 3e-2 and diff.mean() < 3e-3


def test_long_prompt_equals_small_chunks(setup):
    """A prompt of 2600 tokens in chunks of 1024 rows (whole sequences up to 2048 and chunks of them beyond) against the same
    prompt appended 8 tokens at a time, which takes the attention of small blocks."""
    sev, harness, model, om = setup
    rng = np.random.default_rng(3)
    prompt = rng.integers(0, SHAPE.vocab, 2600)
    announce("shared attention: prompt of 2600, chunks of 1024 against blocks of 8")
    a = harness.Batch(model, SHAPE, [2608], max_rows=1024, seed=SEED)
    a.prefill([prompt])
    b = harness.Batch(model, SHAPE, [2608], max_rows=8, seed=SEED)
    b.prefill([prompt])
    for got, ref in zip(a.export_kv(0, 1, 0, 2600), b.export_kv(0, 1, 0, 2600)):
        assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 2e-3)
