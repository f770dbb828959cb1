"""The float32 path over the shapes it accepts (odd model widths, head sizes that are no multiple of four, grouped heads, an
odd vocabulary) and over block sizes around its row tiles (4, 8, 16 rows per wave, from 17 rows on 32 per block and 64 where
the matrix is wide), chains, trees and prefill, against the
64-bit oracle.  A logit is a sum of d products after layers of such sums: with float32 rounding (6e-8) on values of order one
and up to 700 terms in any order, 1e-4 leaves a factor of about ten."""
import numpy as np
import pytest
import torch

import synth
from oracle import verify_oracle as vo
from tests.helpers import announce, oracle_model

pytestmark = pytest.mark.gpu
TOL = 1e-4

#        layers d   Hq Hkv hd  ffn  vocab
SHAPES = [(1, 33, 2, 1, 6, 50, 97), (2, 64, 4, 2, 34, 44, 130), (1, 100, 3, 3, 32, 129, 61), (2, 68, 2, 1, 128, 70, 256), (1, 48, 2, 2, 200, 36, 64),
          (1, 256, 4, 4, 64, 688, 1024), (1, 33, 2, 1, 6, 50, 8191), (1, 64, 2, 1, 32, 40, 8200)]


def _shape(i):
    L, d, hq, hkv, hd, f, v = SHAPES[i]
    return synth.workload.ModelShape(f"f32-{i}", L, d, hq, hkv, hd, f, v, 10000.0, "f32", init_std=0.1)


@pytest.mark.parametrize("i,ns,tree", [(0, (1,), False), (0, (5, 12), True), (1, (3, 4, 9), False), (2, (64, 33), True), (3, (4,), True), (4, (16, 1), False),
                                       (4, (7,), True), (5, (8,), False), (5, (60, 64), True), (5, (16,), True), (5, (17,), False), (5, (32, 1), True),
                                       (6, (17,), True), (6, (64, 1), False), (7, (64,), True), (7, (64, 64, 2), False)])
def test_logits(i, ns, tree):
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    shape, seed = _shape(i), 90 + i
    rng = np.random.default_rng(1000 + i + len(ns))
    B, k = len(ns), max(ns)
    lens = [int(x) for x in rng.integers(1, 150, B)]
    announce(f"float32 {SHAPES[i]}, blocks {ns}, prefixes {lens}, trees {tree}")
    model, om = harness.build_model(shape, seed, gains=True), oracle_model(shape, seed, gains=True)
    prompts = [rng.integers(0, shape.vocab, p) for p in lens]
    batch = harness.Batch(model, shape, [p + k for p in lens], max_rows=max(sum(ns), 70), seed=seed)
    batch.prefill(prompts)                                   # chunks of at most 70 rows
    caches = [vo.prefill(om, p, len(p) + k) for p in prompts]
    for b, p in enumerate(lens):
        K, V = batch.export_kv(b, shape.n_layers - 1, 0, p)
        assert np.abs(K - caches[b].K[-1][:p]).max() < TOL and np.abs(V - caches[b].V[-1][:p]).max() < TOL
    par = np.full((B, k), -1, dtype=np.int32)
    tok = rng.integers(0, shape.vocab, (B, k)).astype(np.int32)
    for b, n in enumerate(ns):
        par[b, :n] = [int(rng.integers(max(-1, j - 5), j)) if tree else j - 1 for j in range(n)]
    out = sev.verify_ex(model, batch.kv, lens, torch.tensor(tok, device="cuda"), k, draft_lens=list(ns),
                        parents=torch.tensor(par, device="cuda") if tree else None, want_argmax=True, want_logits=True)
    torch.cuda.synchronize()
    got = out["logits"].cpu().numpy()
    want = np.concatenate(vo.forward_blocks(om, caches, [tok[b, :n] for b, n in enumerate(ns)], [par[b, :n] for b, n in enumerate(ns)])[0])
    assert np.abs(got - want).max() < TOL
    assert np.array_equal(out["row_argmax"].cpu().numpy(), np.argmax(got, axis=-1))


@pytest.mark.parametrize("n", [5, 17, 64])
def test_infinite_weights(n):
    """An infinite weight makes its column's logits infinite, of the sign of the activation it meets, and leaves every other
    column alone, whichever kernel the row count takes (a sum that turned infinite early must not end as NaN)."""
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    shape, seed = _shape(5), 95
    model, om = harness.build_model(shape, seed), oracle_model(shape, seed)
    head = synth.WeightSource(shape, seed).tensor("lm_head").copy()
    head[7, 5], head[9, 200], head[1023, 255] = np.inf, -np.inf, np.inf
    model.load_tensor("lm_head", 0, torch.from_numpy(head).cuda())
    plain = om.tensor
    om = vo.Model(shape.n_layers, shape.d_model, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.d_ffn, shape.vocab, shape.rope_base,
                  shape.rms_eps, tensor=lambda name, layer=0: head if name == "lm_head" else plain(name, layer), dtype=np.float64)
    rng = np.random.default_rng(n)
    prompt, tok = rng.integers(0, shape.vocab, 9), rng.integers(0, shape.vocab, (1, n)).astype(np.int32)
    announce(f"float32, infinite head weights, {n} rows")
    batch = harness.Batch(model, shape, [9 + n], max_rows=70, seed=seed)
    batch.prefill([prompt])
    got = sev.verify_ex(model, batch.kv, [9], torch.tensor(tok, device="cuda"), n, want_logits=True)["logits"].cpu().numpy()
    want = vo.forward_blocks(om, [vo.prefill(om, prompt, 9 + n)], [tok[0]], [vo.chain_parents(n)])[0][0]
    infinite = np.isinf(want)
    assert infinite[:, [7, 9, 1023]].all() and infinite.sum() == 3 * n
    assert np.array_equal(got[infinite], want[infinite]) and np.abs(got[~infinite] - want[~infinite]).max() < TOL
