"""Shapes either side of the lines of the launch plan: a prefix pass of 256 and 128 workgroups (by the length of a split
and by the suffix bound), chunk sizes below and from 2048 (sample, KV head) pairs on, V marked as streamed or not,
splits turned from prompt to prompt (2, 3, 4, 6, 8 splits of ragged prompts)."""
import numpy as np
import pytest

from gpu_checks import check_attention
from paper_2502_02534_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding, device
    binding.load()
    return device


# (samples, prefix, suffix bound, tokens per split, splits, tokens per chunk, chunks)
SHAPES = [(48, 2000, 20, 128, 16, 64, 1), (48, 2000, 700, 128, 16, 96, 8),
          (33, 3000, 480, 128, 24, 64, 8), (33, 3000, 500, 192, 16, 64, 8),      # the stream outlasts 128 workgroups
          (33, 8192, 940, 512, 16, 96, 10), (33, 8193, 940, 320, 26, 96, 10),    # 512 tokens a split in 128 workgroups
          (80, 4000, 450, 512, 8, 96, 5),
          (16, 2000, 250, 128, 16, 64, 4),
          (255, 300, 500, 128, 3, 192, 3), (256, 300, 330, 128, 3, 352, 1),      # 2040 and 2048 pairs
          (9, 0, 500, 128, 0, 64, 8)]


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("samples,prefix,suffix,split,splits,chunk,chunks", SHAPES)
def test_either_side_of_the_plans_lines(dev, oracle, samples, prefix, suffix, split, splits, chunk, chunks, page):
    from paper_2502_02534_amd import binding as B
    spec = W.small_spec(num_q_heads=16, num_kv_heads=8, samples_per_prompt=samples, prefix_len=(prefix, prefix),
                        suffix_len=(0, suffix), page_size=page)
    inp = W.make_attn_inputs(0, spec=spec, seed=1700 + samples, poison_padding=True)
    desc = B.make_desc(dtype=B.SPD_BF16, num_q_heads=16, num_kv_heads=8, head_dim=128, num_prompts=1, num_samples=samples,
                       max_samples_per_prompt=samples, page_size=page)
    assert B.spd_attn_plan(desc, prefix, inp.max_suffix_len) == (split, splits, chunk, chunks)
    print(f"{samples} samples, prefix {prefix} in {splits} splits, suffix {suffix} in chunks of {chunk}, page {page}", flush=True)
    rows = np.sort(np.random.default_rng(samples).choice(samples * 16, min(samples * 16, 160), replace=False))
    check_attention(dev, oracle, inp, rows=rows)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("prompts,heads,longest", [(2, 8, 900), (3, 8, 1500), (5, 4, 900), (4, 2, 2500), (7, 1, 3000), (1, 8, 700)])
def test_splits_of_ragged_prompts(dev, oracle, dtype, d, prompts, heads, longest):
    spec = W.small_spec(dtype=dtype, head_dim=d, num_q_heads=2 * heads, num_kv_heads=heads, num_prompts=prompts, samples_per_prompt=9,
                        prefix_len=(1, longest), suffix_len=(0, 40), page_size=16 if prompts % 2 else 0)
    print(f"{dtype} {d}: {prompts} prompts of up to {longest} tokens, {heads} KV heads", flush=True)
    check_attention(dev, oracle, W.make_attn_inputs(0, spec=spec, seed=1800 + prompts, poison_padding=True))


@pytest.mark.parametrize("prefix", [0, 40])
def test_streamed_keys(dev, oracle, prefix):
    """From 1 GiB of contiguous KV on, by its bounds, K is marked as streamed too: the suffix kernel by itself, and beside a prefix."""
    samples = 345
    spec = W.small_spec(num_q_heads=16, num_kv_heads=8, samples_per_prompt=samples, prefix_len=(prefix, prefix), suffix_len=(0, 800))
    inp = W.make_attn_inputs(0, spec=spec, seed=1900 + prefix, poison_padding=True)
    assert 2.0 * samples * inp.max_suffix_len * 8 * 128 * 2 >= 2**30
    print(f"{samples} samples, prefix {prefix}, suffix up to {inp.max_suffix_len}", flush=True)
    rows = np.sort(np.random.default_rng(prefix).choice(samples * 16, 160, replace=False))
    check_attention(dev, oracle, inp, rows=rows)
