"""A logit that is not a number has probability zero, like one of -inf, on rows with and without a cut or a filter, and
greedy ones: the other tokens are drawn as if it were not there."""
import numpy as np
import pytest

from gpu_checks import compare_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [1000, 9001, 50256, 262144])
def test_nan_logits_are_never_drawn_and_change_nothing_else(oracle, vocab, filters):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding as B
    B.load()
    rows = 16
    print(f"NaN logits: vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab + 3)
    x = (rng.standard_normal((rows, vocab)) * 3.0).astype(np.float32)
    gone = np.zeros((rows, vocab), bool)
    gone[np.arange(rows), rng.integers(0, vocab, rows)] = True     # one in every row
    gone[1, : vocab // 3] = gone[2, ::5] = gone[3, -1] = gone[5, -3:] = gone[6, 0] = True
    t = np.array([1.0, 0.7, 0.4, 1.0] * 4, np.float32)
    top_p = np.array([1.0] * 8 + [0.9] * 8, np.float32)
    t[7] = 0.0
    u = rng.random(rows, dtype=np.float32)
    top_k = rng.choice(np.array([0, 7, 300], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 0.02], np.float32), rows) if filters else None
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((max(256, B.sample_tokens_workspace_size(rows, vocab)),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(np.where(gone, np.float32(np.nan), x)), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    masked = np.where(gone, np.float32(-np.inf), x)
    o = oracle.sample_tokens_filtered(masked, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(masked, t, top_p, u)
    compare_tokens(tokens.cpu().numpy(), o, u, vocab)
