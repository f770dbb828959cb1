"""sev_prefill over batches of unequal prompts: row budgets that cut prompts anywhere, chunks that end no prompt, one, or
several, a one-token prompt, prefixes that are already there.  K/V against the oracle's prefill (relative rms: 2e-4 in layer
0, where only float32 sums differ, 8e-3 in the deeper layers, whose one-step flips of the rounded cache feed each other) and
the next token, which comes from the last row alone, where the oracle's arg-max is firm."""
import numpy as np
import pytest
import torch

import synth
from oracle import verify_oracle as vo
from tests.helpers import oracle_model, announce

pytestmark = pytest.mark.gpu
SHAPE, SEED, LENS = synth.MINI_BF16, 606, [5, 130, 1, 64, 33]


@pytest.fixture(scope="module")
def setup():
    from paper_2505_17052_amd import harness
    om = oracle_model(SHAPE, SEED, dtype=np.float32)
    rng = np.random.default_rng(9)
    prompts = [rng.integers(0, SHAPE.vocab, n) for n in LENS]
    caches, firm = [], []
    for p in prompts:
        caches.append(vo.prefill(om, p, len(p)))
        t = np.sort(vo.forward_blocks(om, [vo.Cache(om, len(p))], [p], [vo.chain_parents(len(p))])[0][0][-1])[-2:]
        firm.append(t[1] - t[0] >= 0.05)
    return harness, harness.build_model(SHAPE, SEED), prompts, caches, firm


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("budget,split", [(5, 0), (32, 0), (64, 0), (65, 0), (232, 0), (512, 0), (48, 1), (512, 1)])
def test_ragged_prompts(setup, budget, split):
    harness, model, prompts, caches, firm = setup
    announce(f"prefill chunks: prompts {LENS}, {budget} rows, {'in two calls' if split else 'in one call'}")
    batch = harness.Batch(model, SHAPE, [n + 4 for n in LENS], max_rows=budget, seed=SEED)
    if split:                                                # the second call continues the first one's prefixes
        batch.prefill([p[:len(p) // 2] for p in prompts if len(p) > 1], [b for b, p in enumerate(prompts) if len(p) > 1])
        batch.prefill([p[len(p) // 2:] for p in prompts])
    else:
        batch.prefill(prompts)
    for b, n in enumerate(LENS):
        length, nxt, flags = batch.kv.get_state(b)
        assert (length, flags) == (n, 0)
        if firm[b]:
            assert nxt == caches[b].next_tok
        for l in range(SHAPE.n_layers):
            k, v = batch.export_kv(b, l, 0, n)
            assert _rel(k, caches[b].K[l][:n]) < (2e-4 if l == 0 else 8e-3) and _rel(v, caches[b].V[l][:n]) < (2e-4 if l == 0 else 8e-3)


def test_token_array_beyond_32_bits(setup):
    """Prompts in a token array of more than 2^31 entries (rows of 2^30 + 16 and more), the last of them behind entry 2^31:
    the caches and next tokens of the same prompts in an array that just holds them, bit for bit."""
    harness, model, prompts, caches, firm = setup
    import paper_2505_17052_amd as sev
    for B, t_max in ((2, 2 ** 30 + 16), (3, 2 ** 30 + 16)):
        announce(f"prefill: {B} prompts in rows of {t_max} tokens")
        lens = LENS[:B]
        got = []
        wide = torch.empty((B, t_max), dtype=torch.int32, device="cuda")
        narrow = torch.zeros((B, max(lens)), dtype=torch.int32, device="cuda")
        for tokens in (wide, narrow):
            for b, p in enumerate(prompts[:B]):
                tokens[b, :len(p)] = torch.tensor(p.astype(np.int32), device="cuda")
            batch = harness.Batch(model, SHAPE, [n + 4 for n in lens], max_rows=48, seed=SEED)
            sev.prefill(model, batch.kv, [0] * B, lens, tokens)
            got.append([x for b, n in enumerate(lens) for x in (*batch.export_kv(b, SHAPE.n_layers - 1, 0, n), *batch.kv.get_state(b))])
        assert all(np.array_equal(a, b) for a, b in zip(*got))
