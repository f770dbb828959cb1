"""The attention of requests with many query rows (four row groups per block, K/V through LDS): row counts around the block
of 128 rows and its waves, prefixes around a page and a page pair, whole sequences and chunks, chains and trees, ragged
batches that mix both sizes of blocks, against the oracle.  Also an appended block whose rows see only part of it.
The variant is forced through the tuning variable SEV_TUNE_QUAD (pages per chunk, 0: one row group per block), and left to
the library once.
Tolerances: entries of the bf16 cache that lie between two values may be rounded the other way, which leaves the logits
1e-4 off on average and 7e-4 at most over these cases; the bounds are four times that.  Nothing else has fewer than 16 bits."""
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


BATCHES = [([1], (24,), False), ([15, 16, 17], (32, 31, 25), False), ([31, 33], (64, 64), True), ([700, 5, 130], (64, 57, 32), True),
           ([1500], (33,), False), ([257, 90], (64, 24), False), ([64, 480, 31, 9], (32, 64, 63, 24), True)]
# chunks of 3 pages that end before, at, behind and inside the draft block; several chunks of 8 and 24 pages, trees and chains,
# and whole sequences where the library would split; the same blocks by one row group, in sets of equal requests (1, 3 and 8
# of them) and unequal ones
FORCED = [(3, [60, 95, 96, 97], (64, 33, 24, 48), True), (3, [47, 48, 1], (64, 1, 64), False), (8, [700, 5, 130], (64, 57, 32), True),
          (8, [257, 127, 128, 129], (64, 24, 33, 64), True), (24, [1500, 383, 384], (33, 64, 24), True), (24, [1500, 385], (64, 24), False),
          (256, [700, 5, 130], (64, 57, 32), True), (256, [1500], (33,), False), (0, [31] * 8, (24,) * 8, True), (0, [200] * 3, (64,) * 3, True),
          (0, [40], (64,), False), (0, [900] * 8, (33,) * 8, True), (0, [700, 5, 130], (64, 57, 32), True)]


@pytest.mark.parametrize("quad,lens,ns,tree", [(None, *x) for x in BATCHES] + FORCED)
def test_blocks(setup, monkeypatch, quad, lens, ns, tree):
    sev, harness, model, om = setup
    if quad is not None:
        monkeypatch.setenv("SEV_TUNE_QUAD", str(quad))
    rng = np.random.default_rng(sum(lens) + len(ns))
    B, k = len(ns), max(ns)
    announce(f"shared attention ({quad}): prefixes {lens}, nodes {ns}, trees {tree}")
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
    assert diff.max() < 3e-3 and diff.mean() < 5e-4


def test_planes_and_variants(setup, monkeypatch):
    """One layer, where no rounded cache entry feeds another layer: every variant is within 2.6e-5 of the oracle on average
    (bound 6e-5; with q held in one bf16 plane it would be 1.3e-4, with the probabilities 5.5e-4), and the variants, which differ
    in the order of their float32 sums alone, are within 1.7e-5 of each other (bound four times that)."""
    sev, harness, _, _ = setup
    shape = SHAPE.with_layers(1)
    model, om = harness.build_model(shape, SEED), oracle_model(shape, SEED, dtype=np.float32)
    for lens, ns in (([700, 5, 130], (64, 57, 32)), ([60, 95, 96, 97], (64, 33, 24, 48))):
        rng = np.random.default_rng(sum(lens))
        prompts = [rng.integers(0, shape.vocab, p) for p in lens]
        tok = rng.integers(0, shape.vocab, (len(lens), 64)).astype(np.int32)
        caches = [vo.prefill(om, p, len(p) + 64) for p in prompts]
        want = np.concatenate(vo.forward_blocks(om, caches, [tok[b, :n] for b, n in enumerate(ns)], [vo.chain_parents(n) for n in ns])[0])
        plain = None
        for quad in ("0", "3", "24", "256"):
            monkeypatch.setenv("SEV_TUNE_QUAD", quad)
            announce(f"one layer, attention variant {quad}: prefixes {lens}, nodes {ns}")
            batch = harness.Batch(model, shape, [p + 64 for p in lens], max_rows=sum(ns), seed=SEED)
            batch.prefill(prompts)
            got = sev.verify_ex(model, batch.kv, lens, torch.tensor(tok, device="cuda"), 64, draft_lens=list(ns),
                                want_logits=True)["logits"].cpu().numpy()
            plain = got if plain is None else plain
            assert np.abs(got - want).mean() < 6e-5 and np.abs(got - plain).max() < 7e-5


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


@pytest.mark.parametrize("cp,lens,ns", [(8, [500, 60, 1], (5, 3, 8)), (8, [635, 636], (5, 4)), (4, [505, 500, 3], (7, 8, 1)), (4, [570], (24,)), (2, [700, 250, 33], (9, 17, 8))])
def test_merge_of_many_chunks(setup, monkeypatch, cp, lens, ns):
    """1, 4 and 5, 8 and 9, 36, and 45, 17 and 3 chunks of cp pages per request, groups of query rows that end inside and at the end of a
    merge block's 8 rows (4 query heads x 1 to 24 nodes)."""
    sev, harness, model, om = setup
    monkeypatch.setenv("SEV_TUNE_CP", str(cp))
    monkeypatch.setenv("SEV_TUNE_QUAD", "0")
    rng = np.random.default_rng(sum(lens) + cp)
    B, k = len(ns), max(ns)
    announce(f"merge: chunks of {cp} pages, prefixes {lens}, nodes {ns}")
    prompts = [rng.integers(0, SHAPE.vocab, p) for p in lens]
    batch = harness.Batch(model, SHAPE, [p + k for p in lens], max_rows=128, seed=SEED)
    batch.prefill(prompts)
    caches = [vo.prefill(om, p, len(p) + k) for p in prompts]
    tok = rng.integers(0, SHAPE.vocab, (B, k)).astype(np.int32)
    out = sev.verify_ex(model, batch.kv, lens, torch.tensor(tok, device="cuda"), k, draft_lens=list(ns), want_logits=True)
    torch.cuda.synchronize()
    want = np.concatenate(vo.forward_blocks(om, caches, [tok[b, :n] for b, n in enumerate(ns)], [vo.chain_parents(n) for n in ns])[0])
    diff = np.abs(out["logits"].cpu().numpy() - want)
    announce(f"  logits max {diff.max():.2e} mean {diff.mean():.2e}")
    assert diff.max() < 2.8e-3 and diff.mean() < 4e-4
