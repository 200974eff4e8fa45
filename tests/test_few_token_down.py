"""The down projection of a few tokens on the matrix cores: which of its kernels a call runs, and lists longer than the waves' own kernel
holds the channel numbers of at a time, against plain float64."""
import re

import pytest
import torch

from test_row_loads import _kernels, layer  # noqa: F401 (fixture)
from test_streamed_rows import BF16, F32, _hidden


# waves on their own up to 8 tokens; up to 16 where a slab is one group of every wave's, or with masks over a long list
@pytest.mark.gpu
@pytest.mark.parametrize("layer,T,own_masks,kernel", [
    ((3072, 6144), 10, False, "staged1"), ((3072, 6144), 16, True, "staged1"), ((3072, 6144), 17, False, "staged2"),
    ((3072, 6144), 31, True, "staged2"), ((4096, 8184), 9, True, "staged1"), ((4096, 8192), 9, True, "waves8"),
    ((4096, 8192), 8, False, "waves4"), ((4096, 8192), 9, False, "staged1"), ((2048, 6144), 10, False, "waves8"),
    ((2048, 6145), 16, False, "staged1"), ((2048, 6144), 10, True, "staged1")], indirect=["layer"])
def test_kernel_by_tokens(layer, T, own_masks, kernel):  # noqa: F811
    pop, h, m, x, y = layer
    mask = torch.ones((T if own_masks else 1, m), dtype=torch.uint8, device="cuda")
    names = _kernels(lambda s: pop.pop_pruned_ffn(h, x[:T], T, mask, mask.shape[0], y[:T], F32, stream=s))
    found = [re.search(r"skinny_(down|staged)_kernelIN3pop\d+\w+?BF16ELi(\d)ELb(\d)E", n) or
             re.search(r"skinny_(down|staged)_kernelINS_\d+\w+?BF16ELi(\d)ELb(\d)E", n) for n in names]
    (m_,) = [f for f in found if f]
    assert ("waves" if m_.group(1) == "down" else "staged") + m_.group(2) == kernel and int(m_.group(3)) == own_masks


# Two slabs (d 12288); the waves' own kernel holds 4096 channel numbers of a slab at a time, so lists of 8192 and fewer channels are one
# part a slab, longer ones two, the second of one channel, of 33 (a group of each wave's begun), of 2304
@pytest.mark.gpu
@pytest.mark.parametrize("n", [8190, 8192, 8194, 8258, 12800])
def test_long_lists(n):
    from paper_2602_06822_amd import binding as pop
    d, m = 12288, 12904
    gen = torch.Generator(device="cuda").manual_seed(n)
    wg, wu, wd = ((0.02 * torch.randn(s, generator=gen, device="cuda")).bfloat16() for s in ((m, d), (m, d), (d, m)))
    h = pop.pop_layer_create(d, m, BF16, wg, wu, wd, 32, 6)
    try:
        active = torch.randperm(m, generator=gen, device="cuda")[:n]
        x = torch.randn((17, d), generator=gen, device="cuda").bfloat16()
        own = torch.zeros((17, m), dtype=torch.uint8, device="cuda")
        own[:, active] = (torch.rand((17, n), generator=gen, device="cuda") < 0.7).to(torch.uint8)
        own[0, active] = 1  # (the list is the channels active in any row)
        one = own[:1].contiguous()
        hid = _hidden(x, wg, wu)
        down = wd.double().t()
        for T, mask in ((6, own[:6]), (12, own[:12]), (8, one), (12, one), (17, own)):
            y = torch.full((T, d), 7.0, device="cuda")
            pop.pop_pruned_ffn(h, x[:T].contiguous(), T, mask.contiguous(), mask.shape[0], y, F32)
            torch.cuda.synchronize()
            ref = (hid[:T] * mask) @ down
            # (float32 sums: 2^-24 of the running sum a product, some 1600 of them a wave, random signs: 40 * 6e-8, and expf's few ulp)
            err = float((y - ref).abs().max() / ref.abs().max())
            assert err < 1e-5, (T, mask.shape[0], err)
    finally:
        pop.pop_layer_destroy(h)
