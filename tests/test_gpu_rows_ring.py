"""The general kernel from LDS (bf16, 64 channels): lengths either side of its 32-token tiles and of the two tiles
copied ahead, one to four wavefronts on an item, 16 and 32 query rows per wavefront, paged and contiguous KV."""
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


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("length", [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 129, 161, 257, 400])
def test_lengths_around_tiles(dev, oracle, length, page):
    for prompts, spp, heads in ((1, 3, 2), (2, 11, 2), (3, 40, 1)):
        spec = W.small_spec(dtype="bf16", head_dim=64, num_q_heads=4 * heads, num_kv_heads=heads, num_prompts=prompts,
                            samples_per_prompt=spp, prefix_len=(length, length), suffix_len=(max(0, length - 1) % 150, length % 150),
                            page_size=page)
        print(f"length {length}, page {page}, {prompts} x {spp} samples", flush=True)
        check_attention(dev, oracle, W.make_attn_inputs(0, spec=spec, seed=1500 + length, poison_padding=True))


@pytest.mark.parametrize("spp,prefix,suffix", [(300, 700, 130), (700, 100, 700)])
def test_one_wavefront_per_item(dev, oracle, spp, prefix, suffix):
    """So many items that none is shared: whole splits and chunks by one wavefront, many tiles each."""
    spec = W.small_spec(dtype="bf16", head_dim=64, num_q_heads=8, num_kv_heads=8, num_prompts=2, samples_per_prompt=spp,
                        prefix_len=(prefix // 2, prefix), suffix_len=(0, suffix), page_size=16)
    inp = W.make_attn_inputs(0, spec=spec, seed=1600 + spp, poison_padding=True)
    rows = np.sort(np.random.default_rng(spp).choice(spec.num_samples * 8, 128, replace=False))
    print(f"2 x {spp} samples, prefix {prefix}, suffix {suffix}", flush=True)
    check_attention(dev, oracle, inp, rows=rows)
