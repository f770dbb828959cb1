"""GEMM blocks whose waves share a column tile (64 x 192 for QKV, 128 x 448 for gate/up) and the 128 x 384 QKV block, forced on
a small model through the tuning variables, against the oracle: 225 rows (the last row tile holds one row), a gate/up matrix of
88 column tiles (the last block has 4 of 14) and 32 QKV tiles (2 of 6 in the last block of six, 8 of 12), whole and split K.
Tolerances: keys and values are rounded to bf16 (one step is 2^-7 of the value) and may lie one step apart.  Everything else
keeps 16 bits and more, so the logits (of order one) are off by what such flips leave: 1e-4 on average and 1e-3 at most,
whichever shapes are taken, and the bounds are four times that."""
import numpy as np
import pytest
import torch

import synth
from oracle import verify_oracle as vo
from tests.helpers import announce, oracle_model

pytestmark = pytest.mark.gpu
SHAPE = synth.workload.ModelShape("gemm-shapes", 2, 512, 6, 1, 128, 1408, 4224, 500000.0, "bf16")
SEED = 77


@pytest.fixture(scope="module")
def setup():
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    om = oracle_model(SHAPE, SEED, dtype=np.float32, gains=True)
    rng = np.random.default_rng(5)
    lens = [int(x) for x in rng.integers(3, 40, 15)]
    prompts = [rng.integers(0, SHAPE.vocab, p) for p in lens]
    tok = rng.integers(0, SHAPE.vocab, (15, 15)).astype(np.int32)
    caches = [vo.prefill(om, p, len(p) + 15) for p in prompts]
    want = np.concatenate(vo.forward_blocks(om, caches, list(tok), [vo.chain_parents(15)] * 15)[0])
    return sev, harness, harness.build_model(SHAPE, SEED, gains=True), lens, prompts, tok, caches, want


@pytest.mark.parametrize("qkv,gate_up", [("", ""), ("2,15,1,4", "4,35,1,4"), ("2,15,3,4", "4,35,2,4"), ("4,3,1,4", "4,4,1,4"), ("4,3,2,4", "4,2,1,4"), ("4,4,1,4", "4,4,1,4")])
def test_forced_shapes(setup, monkeypatch, qkv, gate_up):
    sev, harness, model, lens, prompts, tok, caches, want = setup
    if qkv:
        monkeypatch.setenv("SEV_TUNE_QKV", qkv)
        monkeypatch.setenv("SEV_TUNE_GU", gate_up)
    announce(f"GEMM shapes: QKV {qkv or 'automatic'}, gate/up {gate_up or 'automatic'}")
    batch = harness.Batch(model, SHAPE, [p + 15 for p in lens], max_rows=225, seed=SEED)
    batch.prefill(prompts)
    for b, p in enumerate(lens):
        for got, ref in zip(batch.export_kv(b, 1, 0, p), (caches[b].K[1][:p], caches[b].V[1][:p])):
            assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-3)
    out = sev.verify_ex(model, batch.kv, lens, torch.tensor(tok, device="cuda"), 15, want_argmax=True, want_logits=True)
    torch.cuda.synchronize()
    diff = np.abs(out["logits"].cpu().numpy() - want)
    announce(f"  logits max {diff.max():.2e} mean {diff.mean():.2e}")
    assert diff.max() < 4e-3 and diff.mean() < 4e-4


@pytest.mark.parametrize("requests,shape", [(15, "-1,1,1,4"), (15, "-3,1,2,4"), (15, "-3,2,1,4"), (15, "-5,1,1,4"), (15, "-5,2,3,4"), (7, "-7,1,2,4"), (7, "-7,2,1,4"), (3, "-3,1,1,4"), (1, "-1,2,3,4"),
                                            (15, "-5,3,1,4"), (15, "-5,4,2,4"), (5, "-5,4,1,4"), (6, "-6,3,2,4"), (6, "-6,4,1,4"), (7, "-7,3,1,4"), (7, "-7,4,3,4"), (10, "-10,3,2,4"),
                                            (15, "-1,0,1,4"), (15, "-2,0,1,4"), (3, "-2,0,1,4"), (1, "-1,0,1,4")])
def test_blocks_of_an_odd_number_of_row_units(setup, monkeypatch, requests, shape):
    """Blocks of 16, 48, 80 and 112 rows, narrow (two k-steps of activations per stage) and wide (one, its last load by half of the threads),
    and wide ones of 96 and 160, whole and split K, on all four projections: 225, 150, 105, 90, 75, 45 and 15 rows.  Also blocks of one
    column tile whose waves share K (16, 24 and 44 steps, the last not a multiple of their batch).  Same bounds as above."""
    sev, harness, model, lens, prompts, tok, caches, want = setup
    for name in ("SEV_TUNE_QKV", "SEV_TUNE_O", "SEV_TUNE_GU", "SEV_TUNE_DOWN"):
        monkeypatch.setenv(name, shape)
    announce(f"GEMM row units {shape}, {requests} requests of 15")
    batch = harness.Batch(model, SHAPE, [p + 15 for p in lens], max_rows=225, seed=SEED)
    batch.prefill(prompts)
    out = sev.verify_ex(model, batch.kv, lens[:requests], torch.tensor(tok[:requests], device="cuda"), 15, want_logits=True)
    torch.cuda.synchronize()
    diff = np.abs(out["logits"].cpu().numpy() - want[:15 * requests])
    announce(f"  logits max {diff.max():.2e} mean {diff.mean():.2e}")
    assert diff.max() < 4e-3 and diff.mean() < 4e-4


LM_SHAPE = synth.workload.ModelShape("lm-shapes", 1, 256, 2, 1, 128, 512, 128256, 500000.0, "bf16")


@pytest.mark.parametrize("requests", [5, 6, 7, 8, 9, 31])
def test_head_blocks(requests):
    """The output head over a vocabulary that fills the chip several times, in blocks of 80 to 160 rows (75, 90, 105, 120, 135 and 465 rows of 4008
    column tiles, which neither 16 nor 12 divide evenly among the blocks): logits, and the arg-max of every row of them.  Same bounds as above."""
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    om = oracle_model(LM_SHAPE, SEED, dtype=np.float32, gains=True)
    rng = np.random.default_rng(requests)
    prompts = [rng.integers(0, LM_SHAPE.vocab, 3) for _ in range(requests)]
    tok = rng.integers(0, LM_SHAPE.vocab, (requests, 15)).astype(np.int32)
    caches = [vo.prefill(om, p, len(p) + 15) for p in prompts]
    want = np.concatenate(vo.forward_blocks(om, caches, list(tok), [vo.chain_parents(15)] * requests)[0])
    announce(f"LM head, {15 * requests} rows")
    batch = harness.Batch(harness.build_model(LM_SHAPE, SEED, gains=True), LM_SHAPE, [18] * requests, max_rows=15 * requests, seed=SEED)
    batch.prefill(prompts)
    out = sev.verify_ex(batch.model, batch.kv, [3] * requests, torch.tensor(tok, device="cuda"), 15, want_argmax=True, want_logits=True)
    torch.cuda.synchronize()
    got = out["logits"].cpu().numpy()
    diff = np.abs(got - want)
    announce(f"  logits max {diff.max():.2e} mean {diff.mean():.2e}")
    assert diff.max() < 4e-3 and diff.mean() < 4e-4
    assert np.array_equal(out["row_argmax"].cpu().numpy(), got.argmax(axis=1))


@pytest.mark.parametrize("d,ffn,rows", [(64, 64, 3), (128, 320, 17), (192, 1088, 40)])
def test_narrow_blocks_of_few_steps(monkeypatch, d, ffn, rows):
    """Blocks of one column tile whose waves have 0 or 1, 1 to 3, and 8 or 9 k-steps each (2 to 34 of them), on matrices of 2 to 68 column
    tiles and 3, 17 and 40 rows; the head likewise.  Same bounds as above."""
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    shape = synth.workload.ModelShape("narrow", 2, d, 2, 1, 128, ffn, 1056, 500000.0, "bf16")
    for name in ("SEV_TUNE_QKV", "SEV_TUNE_O", "SEV_TUNE_GU", "SEV_TUNE_DOWN"):
        monkeypatch.setenv(name, "-2,0,1,4" if rows > 16 else "-1,0,1,4")
    om = oracle_model(shape, SEED, dtype=np.float32, gains=True)
    rng = np.random.default_rng(rows)
    prompt, tok = rng.integers(0, shape.vocab, 5), rng.integers(0, shape.vocab, (1, rows)).astype(np.int32)
    cache = vo.prefill(om, prompt, 5 + rows)
    want = vo.forward_blocks(om, [cache], list(tok), [vo.chain_parents(rows)])[0][0]
    announce(f"narrow blocks: model {d} wide, feed-forward {ffn}, {rows} rows")
    batch = harness.Batch(harness.build_model(shape, SEED, gains=True), shape, [5 + rows], max_rows=64, seed=SEED)
    batch.prefill([prompt])
    out = sev.verify_ex(batch.model, batch.kv, [5], torch.tensor(tok, device="cuda"), rows, want_argmax=True, want_logits=True)
    torch.cuda.synchronize()
    got = out["logits"].cpu().numpy()
    diff = np.abs(got - want)
    announce(f"  logits max {diff.max():.2e} mean {diff.mean():.2e}")
    assert diff.max() < 4e-3 and diff.mean() < 4e-4
    assert np.array_equal(out["row_argmax"].cpu().numpy(), got.argmax(axis=1))
