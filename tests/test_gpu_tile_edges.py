"""Sizes where the tiled kernels change course: prefix lengths either side of the 32-token tiles and, in single
splits, of the five-slot rings, a reference maximum that has to be raised late, and merges of every kind (all lanes
on one row with few and with more than 64 slots, four rows per wavefront)."""
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


# 260 samples of 2 heads: five 128-row workgroups and splits of 128 or 192 tokens, or three samples and splits of
# 128 tokens (whole prompts in one split: test_single_splits_around_the_ring)
LENGTHS = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 159, 160, 161, 191, 193, 224, 257, 383]


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("length", LENGTHS)
def test_prefix_lengths_around_tiles_and_rings(dev, oracle, length, page):
    spec = W.small_spec(num_q_heads=64, num_kv_heads=32, samples_per_prompt=260 if length % 2 else 3, prefix_len=(length, length),
                        suffix_len=(0, 3), page_size=page)
    print(f"prefix length {length}, page {page}, {spec.samples_per_prompt} samples", flush=True)
    inp = W.make_attn_inputs(0, spec=spec, seed=1200 + length, poison_padding=True)
    rows = np.random.default_rng(length).choice(spec.num_samples * 64, 96, replace=False)
    check_attention(dev, oracle, inp, rows=np.sort(rows))


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("at", [0, 40, 65, 130, 199])
def test_a_late_dominant_key_raises_the_reference(dev, oracle, dtype, d, at):
    """One key twenty times as long as the others, in the first tile, in later ones and in the last.  (64 channels: the
    items are shared so that a wavefront holds one tile, and the states meet in LDS; later tiles of a wavefront
    of the general kernel are raised in test_gpu_rows.py.)"""
    spec = W.small_spec(dtype=dtype, head_dim=d, num_q_heads=8, num_kv_heads=2, samples_per_prompt=40, prefix_len=(200, 200),
                        suffix_len=(70, 70))
    inp = W.make_attn_inputs(0, spec=spec, seed=1300 + at)
    for k, t in ((inp.k_prefix, at), (inp.k_suffix.reshape(-1, 2, d), at % 70)):
        row = W.bf16_bits_to_f32(k[t]) if dtype == "bf16" else k[t]
        k[t] = W.f32_to_bf16_bits(row * 20) if dtype == "bf16" else row * 20
    print(f"dominant key at {at}, {dtype} {d}", flush=True)
    check_attention(dev, oracle, inp)


MERGES = [
    dict(num_q_heads=2, num_kv_heads=1, samples_per_prompt=1, prefix_len=(8192, 8192), suffix_len=(2048, 2048)),   # 64 + 32 slots
    dict(num_q_heads=2, num_kv_heads=1, samples_per_prompt=2, prefix_len=(300, 300), suffix_len=(0, 0)),           # 3 slots
    dict(num_q_heads=8, num_kv_heads=4, samples_per_prompt=1030, prefix_len=(70, 70), suffix_len=(0, 90)),         # 8240 rows, few slots
    dict(num_q_heads=8, num_kv_heads=1, samples_per_prompt=1025, prefix_len=(300, 300), suffix_len=(0, 330)),      # 8200 rows, more
    dict(dtype="f32", head_dim=256, num_q_heads=2, num_kv_heads=1, samples_per_prompt=3, prefix_len=(4096, 4096), suffix_len=(0, 9)),
    dict(dtype="f32", head_dim=64, num_q_heads=8, num_kv_heads=1, samples_per_prompt=1024, prefix_len=(40, 40), suffix_len=(0, 20)),
]


@pytest.mark.parametrize("i", range(len(MERGES)))
def test_merges_of_every_kind(dev, oracle, i):
    print(f"merge case {i}: {MERGES[i]}", flush=True)
    spec = W.small_spec(**MERGES[i])
    n = spec.num_samples * spec.num_q_heads
    rows = None if n <= 64 else np.sort(np.random.default_rng(i).choice(n, 160, replace=False))
    check_attention(dev, oracle, W.make_attn_inputs(0, spec=spec, seed=1400 + i, poison_padding=True), rows=rows)


@pytest.mark.parametrize("samples,prefix,suffix,slots", [(127, 70, 60, 2), (128, 70, 60, 2), (255, 300, 330, 7), (256, 300, 330, 5)])
def test_merges_either_side_of_sharing_a_rows_slots(dev, oracle, samples, prefix, suffix, slots):
    """From 1024 rows of up to four slots, and from 2048 of up to eight, a row's slots are no longer shared out."""
    spec = W.small_spec(num_q_heads=8, num_kv_heads=4, samples_per_prompt=samples, prefix_len=(prefix, prefix), suffix_len=(0, suffix))
    inp = W.make_attn_inputs(0, spec=spec, seed=1500 + samples, poison_padding=True)
    from paper_2502_02534_amd import binding as B
    plan = B.spd_attn_plan(dev.upload_attn(inp).desc, prefix, suffix)
    assert plan[1] + plan[3] == slots
    rows = np.sort(np.random.default_rng(samples).choice(spec.num_samples * 8, 160, replace=False))
    check_attention(dev, oracle, inp, rows=rows)


# 8 prompts x 32 KV heads give a workgroup per CU without splits, so a four-wavefront workgroup walks all tiles:
# one ring (five tiles) full, one more, twice round
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("length", [33, 64, 65, 97, 129, 159, 160, 161, 191, 192, 193, 224, 225, 320, 321, 352, 353])
def test_single_splits_around_the_ring(dev, oracle, length, page):
    from paper_2502_02534_amd import binding as B
    spec = W.small_spec(num_q_heads=32, num_kv_heads=32, num_prompts=8, samples_per_prompt=5, prefix_len=(length, length),
                        suffix_len=(0, 3), page_size=page)
    inp = W.make_attn_inputs(0, spec=spec, seed=1600 + length, poison_padding=True)
    d = dev.upload_attn(inp)
    split, splits, _, _ = B.spd_attn_plan(d.desc, length, 3)
    assert splits == 1 and split >= length
    print(f"one split of {length} tokens, page {page}", flush=True)
    rows = np.sort(np.random.default_rng(length).choice(spec.num_samples * 32, 96, replace=False))
    check_attention(dev, oracle, inp, rows=rows)
