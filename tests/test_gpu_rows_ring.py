"""The general kernel on bf16 with 64 channels, from registers (short chunks) and from LDS (chunks of 256 tokens and
more, a wavefront each): lengths either side of its 32-token tiles and of the two tiles copied ahead, one to four
wavefronts on an item, 16 and 32 query rows per wavefront, paged and contiguous KV."""
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


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("heads,spp", [(8, 65), (16, 65), (8, 5)])     # 65, 130 and 5 query rows a prompt and KV head
@pytest.mark.parametrize("length", [1, 31, 32, 33, 63, 64, 65, 95, 97, 129, 321, 600])
def test_lengths_around_tiles_through_lds(dev, oracle, length, heads, spp, page):
    from paper_2502_02534_amd import binding as B
    prompts, bound = (130 + spp - 1) // spp, 600
    spec = W.small_spec(dtype="bf16", head_dim=64, num_q_heads=heads, num_kv_heads=8, num_prompts=prompts, samples_per_prompt=spp,
                        prefix_len=(length, length), suffix_len=(max(0, length - 70), length if page else bound), page_size=page)
    inp = W.make_attn_inputs(0, spec=spec, seed=2300 + length, poison_padding=True)
    if page == 0:  # slots of the bound, lengths around `length`
        inp.suffix_lens[:] = np.minimum(inp.suffix_lens, np.random.default_rng(length).integers(max(0, length - 70), length + 1, spec.num_samples))
        for n, filled in enumerate(inp.suffix_lens):
            inp.k_suffix[n, filled:] = inp.v_suffix[n, filled:] = 0x7FC1
    inp.max_suffix_len = bound
    desc = B.make_desc(dtype=B.SPD_BF16, num_q_heads=heads, num_kv_heads=8, head_dim=64, num_prompts=prompts,
                       num_samples=spec.num_samples, max_samples_per_prompt=spp, page_size=page)
    _, _, chunk, chunks = B.spd_attn_plan(desc, inp.max_prefix_len, bound)
    assert chunk >= 256 and spec.num_samples * 8 * chunks > 1024     # long chunks, too many to be shared
    rows = np.sort(np.random.default_rng(length).choice(spec.num_samples * heads, 96, replace=False))
    print(f"length {length}, page {page}, {prompts} x {spp} samples, {heads} heads", flush=True)
    check_attention(dev, oracle, inp, rows=rows)
