"""The prompt's own forward pass with H kept by channel: its down projection reads rows of H and of the weights by the list of
active channels.  Sizes at the edges of its tiles, against plain float64; its counted waits in the listing."""
import re

import pytest
import torch

from test_asm_waits import counted_waits, loads_in_flight, most_left_in_flight, product_hazards
from test_streamed_rows import BF16, F32, _functions, _hidden, _listing, needs_hipcc


@needs_hipcc
def test_waits_of_the_row_kernels(tmp_path):
    """Two operands by channel: a k-step loads its channel numbers' 64 entries once, five loads before its wait, and reads the numbers
    a step earlier than down_gemm_dma_kernel does, so the same count is the largest that leaves no needed load in flight."""
    found = _listing(tmp_path, "pop_down_gemm.hip", "down_gemm_rows_kernel")
    assert len(found) == 10
    for name, code in found.items():
        mf = int(re.search(r"ILi(\d)E", name).group(1))
        assert not loads_in_flight(code)[1] and not product_hazards(code)[1], name
        na, nb = {5: 2, 4: 3, 3: 3}.get(mf, 4), 3 if mf == 4 else 4
        (before, after, left, products), = counted_waits(code)
        assert (before, after, products, left) == (5, 2 * mf, 16 * mf, most_left_in_flight(na, nb, 2 * mf, 4, True)), name
    found = _listing(tmp_path, "pop_prefill.hip", "prefill_rows_kernel")
    assert len(found) == 10
    for name, code in found.items():
        mf = int(re.search(r"ILi(\d)E", name).group(1))
        assert not loads_in_flight(code)[1] and not product_hazards(code)[1], name
        loops = counted_waits(code)
        assert sorted(p // (2 * mf) for _, _, _, p in loops) == [4, 6, 7, 8, 10, 11, 12], (name, loops)
        for before, after, left, products in loops:
            f = products // (2 * mf)
            na, nb = (3, 3) if mf == 4 and f <= 8 else (2 if mf >= 4 else (3 if mf >= 2 else 4), 3 if mf >= 3 else (4 if mf == 2 else 5))
            assert (before, after, left) == ((f + 1) // 2, 2 * mf, most_left_in_flight(na, nb, 2 * mf, (f + 1) // 2, False))


def _m0_of_the_compiler(lines):
    """Instructions outside inline assembly that name m0."""
    inside, found = False, []
    for line in lines:
        if "ASMSTART" in line or "ASMEND" in line:
            inside = "ASMSTART" in line
        elif not inside and re.search(r"\bm0\b", line.split(";")[0]):
            found.append(line.strip())
    return found


@needs_hipcc
def test_row_kernels_have_m0_to_themselves():
    """Their direct loads set m0 in inline assembly, which cannot tell the compiler so: it must have no use for it of its own."""
    assert _m0_of_the_compiler(["\ts_mov_b32 m0, s3", ";ASMSTART", "\ts_mov_b32 m0, s4", ";ASMEND"]) == ["s_mov_b32 m0, s3"]
    found = _functions("pop_down_gemm.hip", "down_gemm_rows_kernel")
    assert len(found) == 10
    for name, lines in found.items():
        assert any("ASMSTART" in x for x in lines) and sum("m0" in x for x in lines) > 20, name
        assert not _m0_of_the_compiler(lines), name


# (d, m, active channels, prompts run one after the other on one layer: a longer one leaves its rows behind)
CASES = [(128, 193, 130, (320, 33, 64, 319, 32)), (128, 64, 1, (65, 40)), (384, 700, 64, (257, 63, 256)),
         (1152, 333, 65, (129, 128, 191, 193)), (256, 1000, 1000, (520, 100)), (256, 90, 0, (70,)),
         (512, 2050, 1300, (1500, 321, 48))]


@pytest.mark.gpu
@pytest.mark.parametrize("d,m,active,prompts", CASES)
@pytest.mark.parametrize("ydtype", [F32, BF16])
def test_forward_pass_by_channel(d, m, active, prompts, ydtype):
    from paper_2602_06822_amd import binding as pop
    gen = torch.Generator(device="cuda").manual_seed(d + m + active)
    wg, wu, wd = ((0.05 * torch.randn(s, generator=gen, device="cuda")).bfloat16() for s in ((m, d), (m, d), (d, m)))
    h = pop.pop_layer_create(d, m, BF16, wg, wu, wd, max(prompts), 1)
    try:
        for T in prompts:
            x = torch.randn((T, d), generator=gen, device="cuda").bfloat16()
            y = torch.full((T + 1, d), 7.0, device="cuda", dtype=torch.float32 if ydtype == F32 else torch.bfloat16)
            mask = torch.zeros(m, dtype=torch.uint8, device="cuda")
            pop.pop_prefill_forward(h, x, T, active // 2, active - active // 2, active - active // 2, y[:T], ydtype, mask=mask)
            torch.cuda.synchronize()
            assert int(mask.sum()) == active and bool((y[T] == 7.0).all())
            ref = (_hidden(x, wg, wu) * mask) @ wd.double().t()
            # H rounded to bf16 (2^-9 relative per term, in quadrature: 4e-3 of the largest result), a bf16 result another 2^-9
            err = float((y[:T].double() - ref).abs().max()) / max(float(ref.abs().max()), 1e-30)
            assert err < (4e-3 if ydtype == F32 else 8e-3) if active else err == 0.0, (T, err)
    finally:
        pop.pop_layer_destroy(h)

