"""Weight rows of large bf16 layers are loaded past the caches.  The rule is the size of the layer, so a layer just above it
is the layer just below it plus one channel of zeros, which no score, selection or output may notice; against plain float64."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest
import torch

from test_asm_waits import CSRC, ROOT, counted_waits, loads_in_flight, most_left_in_flight, parse, product_hazards

BF16, F32 = 1, 0
needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


@functools.lru_cache(maxsize=None)
def _assembly(src):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, src + ".s")
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
                        os.path.join(CSRC, src), "-o", out], check=True, capture_output=True, timeout=900)
        with open(out) as text:
            return text.read()


def _functions(src, kernel):
    """Lines of every instantiation of a kernel."""
    return {m.group(1): m.group(2).split("\n")[1:] for m in
            re.finditer(r"^(_ZN3pop\d+" + kernel + r"I\w+):(.*?)^\.Lfunc_end", _assembly(src), re.M | re.S)}


def _listing(tmp_path, src, kernel):
    return {name: parse(lines) for name, lines in _functions(src, kernel).items()}


@needs_hipcc
def test_waits_of_the_streaming_prompt_kernels(tmp_path):
    """The counted waits and wait states of prefill_stream_kernel and down_gemm_stream_kernel, as of the kernels they vary."""
    found = _listing(tmp_path, "pop_prefill.hip", "prefill_stream_kernel")
    assert len(found) == 5 * 3 + 2
    for name, code in found.items():
        mf, mode = (int(v) for v in re.search(r"ILi(\d)ELi(\d)E", name).groups())
        assert not loads_in_flight(code)[1] and not product_hazards(code)[1], name
        loops = counted_waits(code)
        assert sorted(p // (2 * mf) for _, _, _, p in loops) == [4, 6, 7, 8, 10, 11, 12], (name, loops)
        for before, after, left, products in loops:
            f = products // (2 * mf)
            deep = mf == 4 and f <= 8 and mode in (0, 2)
            na, nb = (3, 3) if deep else (2 if mf >= 4 else (3 if mf >= 2 else 4), 3 if mf >= 3 else (4 if mf == 2 else 5))
            assert (before, after, left) == ((f + 1) // 2, 2 * mf, most_left_in_flight(na, nb, 2 * mf, (f + 1) // 2, False))
    found = _listing(tmp_path, "pop_down_gemm.hip", "down_gemm_stream_kernel")
    assert len(found) == 5
    for name, code in found.items():
        mf = int(re.search(r"ILi(\d)E", name).group(1))
        assert not loads_in_flight(code)[1] and not product_hazards(code)[1], name
        na, nb = {5: 2, 4: 3, 3: 3}.get(mf, 4), 3 if mf == 4 else 4
        (before, after, left, products), = counted_waits(code)
        assert (before, after, products, left) == (5, 2 * mf, 16 * mf, most_left_in_flight(na, nb, 2 * mf, 4, True)), name


def _hidden(x, wg, wu):
    g = x.double() @ wg.double().t()
    return g / (1.0 + torch.exp(-g)) * (x.double() @ wu.double().t())


# (d, channels of the smaller layer, what runs, rows of x): the larger layer has the first size that streams
CASES = ([(2048, 5461, "step", b) for b in (1, 2, 3, 8)] +
         [(4096, 5461, "forward", t) for t in (24, 40, 300, 400)] + [(4096, 5461, "input_side", 40)] + [(4096, 10239, "forward", t) for t in (128, 512)] +
         [(4096, 8191, "ffn", t) for t in (12, 40)] + [(4096, 10239, "ffn", t) for t in (2, 12, 40)] +
         [(2048, 6826, "step", b) for b in (1, 2, 3, 8)])


@pytest.mark.gpu
@pytest.mark.parametrize("d,m,kind,T", CASES)
def test_a_channel_of_zeros_changes_nothing(d, m, kind, T):
    from paper_2602_06822_amd import binding as pop
    gen = torch.Generator(device="cuda").manual_seed(d + m + T)
    wg, wu, wd = ((0.02 * torch.randn(s, generator=gen, device="cuda")).bfloat16() for s in ((m, d), (m, d), (d, m)))
    x = torch.randn((T, d), generator=gen, device="cuda").bfloat16()
    prompt = torch.randn((64, d), generator=gen, device="cuda").bfloat16()
    n_ret, n_cand, k = int(0.6 * m), int(0.1 * m), int(0.05 * m)
    results = []
    for extra in (0, 1):
        def pad(w, rows):
            return torch.cat([w, w.new_zeros((extra, d) if rows else (d, extra))], 0 if rows else 1).contiguous()
        h = pop.pop_layer_create(d, m + extra, BF16, pad(wg, True), pad(wu, True), pad(wd, False), 512, 8)
        try:
            y = torch.empty((T, d), device="cuda")
            mask = torch.zeros((max(T, 1), m + extra), dtype=torch.uint8, device="cuda")
            scores = torch.empty(m + extra, device="cuda")
            if kind == "step":
                pop.pop_prefill_partition(h, prompt, 64, n_ret, n_cand, scores)
                pop.pop_decode_step(h, x, T, [k] * T, y, F32, mask=mask)
                out = [scores[:m], mask[:, :m], y]
            elif kind == "ffn":
                mask[0, :n_ret] = 1
                pop.pop_pruned_ffn(h, x, T, mask[:1], 1, y, F32)
                out = [mask[:1, :m], y]
            else:
                if kind == "input_side":
                    pop.pop_layer_set_importance(h, pop.POP_IMPORTANCE_INPUT_SIDE)
                pop.pop_prefill_forward(h, x, T, n_ret, n_cand, k, y, F32, scores, mask=mask[0])
                out = [scores[:m], mask[:1, :m], y]
            torch.cuda.synchronize()
            pop.pop_layer_sync_status(h)
        finally:
            pop.pop_layer_destroy(h)
        results.append(out)
    for a, b in zip(*results):
        assert torch.equal(a, b)
    mask, y = results[1][-2].bool(), results[1][-1]
    ref = (_hidden(x, wg, wu) * mask) @ wd.double().t()
    # (a prompt's H is rounded to bf16: 2^-9 relative per term, adding up in quadrature over the active channels)
    assert float((y - ref).abs().max() / ref.abs().max()) < (4e-3 if T >= 32 else 1e-4)
