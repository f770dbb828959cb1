"""The call plan (rows, ancestor sets, work items) and the acceptance walk at the edges of their blocks: block lengths around
the 16 rows of a plan block, the deepest tree (64 levels), the widest, ragged batches up to 256 requests.  Decisions are
compared with the oracle's acceptance on the GPU's own arg-max (whole numbers: exact); a tree that is a chain must give the
chain's logits bit for bit."""
import numpy as np
import pytest
import torch

import synth
from oracle import verify_oracle as vo
from tests.helpers import announce

pytestmark = pytest.mark.gpu
SHAPE, SEED = synth.MINI_BF16, 606


@pytest.fixture(scope="module")
def setup():
    import paper_2505_17052_amd as sev
    from paper_2505_17052_amd import harness
    return sev, harness, harness.build_model(SHAPE, SEED)


def _tree(rng, n, kind):
    if kind == "deep":
        return np.arange(-1, n - 1)
    if kind == "wide":
        return np.array([-1] + [0] * (n - 1))
    if kind == "roots":
        return np.full(n, -1)
    return np.array([-1] + [int(rng.integers(max(-1, i - 9), i)) for i in range(1, n)])


@pytest.mark.parametrize("ns,kinds", [((1,), ("deep",)), ((64,), ("deep",)), ((15, 16, 17, 64), ("random",)), ((64, 2, 33), ("wide", "roots", "random")),
                                      ((31, 32, 63, 1), ("deep", "random")), ((3,) * 256, ("random", "wide"))])
def test_tree_decisions(setup, ns, kinds):
    sev, harness, model = setup
    rng = np.random.default_rng(len(ns) * 100 + ns[0])
    B, k = len(ns), max(ns)
    lens = [int(x) for x in rng.integers(1, 70, B)]
    announce(f"plan: {B} requests, nodes {sorted(set(ns))}, {kinds}")
    batch = harness.Batch(model, SHAPE, [p + k for p in lens], max_rows=sum(ns), seed=SEED)
    batch.prefill([rng.integers(0, SHAPE.vocab, p) for p in lens])
    nxt = [batch.kv.get_state(b)[1] for b in range(B)]
    par = np.full((B, k), -1, dtype=np.int32)
    tok = rng.integers(0, SHAPE.vocab, (B, k)).astype(np.int32)
    for b, n in enumerate(ns):
        par[b, :n] = _tree(rng, n, kinds[b % len(kinds)])
    dev = lambda x: torch.tensor(x, device="cuda")
    right = rng.random((B, k)) < 0.8
    for rounds in range(5):                                  # each round makes one more level follow the model's own arg-max
        out = sev.verify_ex(model, batch.kv, lens, dev(tok), k, draft_lens=ns, parents=dev(par), want_path=True, want_argmax=True)
        am, row0 = out["row_argmax"].cpu().numpy(), np.concatenate([[0], np.cumsum(ns)])
        path = out["accept_path"].cpu().numpy()
        for b, n in enumerate(ns):
            rows = am[row0[b]:row0[b] + n]
            want_len, want_tok, want_path = vo.accept_tree(tok[b, :n], par[b, :n], nxt[b], rows)
            assert int(out["accept_len"][b]) == want_len and int(out["bonus_token"][b]) == want_tok
            assert path[b].tolist() == list(want_path) + [-1] * (k - want_len)
            for i in range(n):
                if right[b, i]:
                    tok[b, i] = nxt[b] if par[b, i] < 0 else rows[par[b, i]]
    assert batch.kv.get_state(0)[2] == 0
    if ns == (64,) or ns == (1,):                            # a chain given as a tree: the same rows, masks and positions
        a = sev.verify_ex(model, batch.kv, lens, dev(tok), k, parents=dev(par), want_logits=True)
        c = sev.verify_ex(model, batch.kv, lens, dev(tok), k, want_logits=True)
        assert torch.equal(a["logits"], c["logits"])


def test_malformed_parents_are_flagged(setup):
    sev, harness, model = setup
    batch = harness.Batch(model, SHAPE, [80], max_rows=64, seed=SEED)
    batch.prefill([np.arange(5)])
    par = np.array([[-1, 0, 2, 1]], dtype=np.int32)          # node 2 names itself
    announce("plan: malformed parents")
    out = sev.verify_ex(model, batch.kv, [5], torch.zeros((1, 4), dtype=torch.int32, device="cuda"), 4, parents=torch.tensor(par, device="cuda"))
    torch.cuda.synchronize()
    assert batch.kv.get_state(0)[2] & 2 and 0 <= int(out["accept_len"][0]) <= 4


def test_commit_of_captured_blocks(setup):
    """A tree's accepted K/V move at the commit also where the block or the commit itself was captured before, and other blocks
    came between (bit for bit what the eager calls leave)."""
    sev, harness, model = setup
    announce("commit: captured tree block, captured commit")
    P, k = 21, 3
    batch = harness.Batch(model, SHAPE, [P + k], max_rows=32, seed=SEED)
    batch.prefill([np.arange(P) % SHAPE.vocab])
    nxt = batch.kv.get_state(0)[1]
    dev = lambda x: torch.tensor([x], dtype=torch.int32, device="cuda")
    par, other = dev([-1, -1, 1]), dev([1, 2, 3])
    tok = dev([(nxt + 1) % SHAPE.vocab, nxt, 0])
    tok[0, 2] = sev.verify_ex(model, batch.kv, [P], tok, k, parents=par, want_argmax=True)["row_argmax"][1]
    tree = lambda: sev.verify_ex(model, batch.kv, [P], tok, k, parents=par)

    def moved():
        out = [x for l in range(SHAPE.n_layers) for x in batch.export_kv(0, l, P, 2)]
        assert batch.kv.get_state(0)[0] == P + 2
        batch.kv.set_state(None, [P], [nxt])
        sev.verify_ex(model, batch.kv, [P], other, k)           # a chain writes over the block
        return out

    assert int(tree()["accept_len"][0]) == 2
    sev.kv_commit(batch.kv, None, 1)
    want = moved()
    block, commit = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(commit):
        sev.kv_commit(batch.kv, None, 1)
    for _ in range(3):
        tree()
        commit.replay()
        assert all(np.array_equal(a, b) for a, b in zip(moved(), want))
    with torch.cuda.graph(block):
        tree()
    for _ in range(3):
        sev.verify_ex(model, batch.kv, [P], other, k)
        block.replay()
        sev.kv_commit(batch.kv, None, 1)
        assert all(np.array_equal(a, b) for a, b in zip(moved(), want))


@pytest.mark.parametrize("captured", ["chain", "sampled", "prefill"])
def test_commit_after_a_capture_that_never_ran(setup, captured):
    """Capturing a chain block runs nothing: a tree that is pending on the slot stays pending, and its commit still moves the
    accepted K/V (bit for bit what the uninterrupted sequence leaves)."""
    sev, harness, model = setup
    announce(f"commit: eager tree, captured {captured}, eager commit")
    P, k = 21, 3
    batch = harness.Batch(model, SHAPE, [P + k], max_rows=32, seed=SEED)
    batch.prefill([np.arange(P) % SHAPE.vocab])
    nxt = batch.kv.get_state(0)[1]
    dev = lambda x: torch.tensor([x], dtype=torch.int32, device="cuda")
    par, chain = dev([-1, -1, 1]), dev([1, 2, 3])
    tok = dev([(nxt + 1) % SHAPE.vocab, nxt, 0])
    tok[0, 2] = sev.verify_ex(model, batch.kv, [P], tok, k, parents=par, want_argmax=True)["row_argmax"][1]
    q, u = torch.full((k, SHAPE.vocab), 1.0 / SHAPE.vocab, device="cuda"), torch.full((1, k), 0.5, device="cuda")
    call = {"chain": lambda: sev.verify_ex(model, batch.kv, [P], chain, k),
            "sampled": lambda: sev.verify_sample(model, batch.kv, [P], chain, k, q, u, u[:, 0].contiguous(), 1.0),
            "prefill": lambda: sev.prefill(model, batch.kv, [P], [k], chain)}[captured]

    def committed(interrupt):
        batch.kv.set_state(None, [P], [nxt])
        sev.verify_ex(model, batch.kv, [P], chain, k)           # a chain: the block's old K/V are gone
        assert int(sev.verify_ex(model, batch.kv, [P], tok, k, parents=par)["accept_len"][0]) == 2
        if interrupt:
            with torch.cuda.graph(torch.cuda.CUDAGraph()):
                call()
        sev.kv_commit(batch.kv, None, 1)
        assert batch.kv.get_state(0)[0] == P + 2
        return [x for l in range(SHAPE.n_layers) for x in batch.export_kv(0, l, P, 2)]

    want = committed(False)
    assert all(np.array_equal(a, b) for a, b in zip(committed(True), want))


def test_prefill_of_more_prompts_than_rows_is_refused(setup):
    sev, harness, model = setup
    batch = harness.Batch(model, SHAPE, [16] * 3, max_rows=2, seed=SEED)
    with pytest.raises(Exception, match="max_rows"):
        sev.prefill(model, batch.kv, [0] * 3, [1] * 3, torch.zeros((3, 1), dtype=torch.int32, device="cuda"))
