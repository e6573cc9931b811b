"""The nucleus cut among more equal logits than the row-level step tells apart one by one: a second look at the lists then gives
what every slice keeps.  Spread over the row, all in its first slice, or all at its end; more of them than a slice lists; with
other logits in between their neighbours, and with a top-k among them too."""
import numpy as np
import pytest

from gpu_checks import compare_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [8000, 9000, 50257, 128256, 262144])  # 1, 2, 8, 8 and 16 slices
def test_the_cut_among_many_equal_logits(oracle, vocab, filters):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding as B
    B.load()
    print(f"many ties: vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab + 77)
    counts = [c for c in (65, 512, 513, 1000, 3000, 6000, 20000) if c < vocab - 100]
    rows = 3 * len(counts)
    x = np.full((rows, vocab), -30.0, np.float32)
    for r in range(rows):
        many, tied = counts[r // 3], np.float32((4.0, -6.0, 0.3)[r % 3])
        where = rng.permutation(vocab) if r % 3 == 0 else np.arange(vocab) if r % 3 == 1 else np.arange(vocab)[::-1]
        x[r, where[:many]] = tied
        x[r, where[many]] = tied + np.float32(np.log(many))             # half of the mass above the ties' level
        x[r, where[many + 1:many + 41]] = tied + rng.uniform(-0.03, 0.03, 40).astype(np.float32)
    t, top_p = np.ones(rows, np.float32), np.full(rows, 0.7, np.float32)
    u = rng.random(rows, dtype=np.float32)
    top_k = rng.choice(np.array([0, 30, 5000], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 1e-6], np.float32), rows) if filters else None
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((B.sample_tokens_workspace_size(rows, vocab),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(tokens.cpu().numpy(), o, u, vocab)
