"""Which calls load weight rows past the caches: the rule is the size of the layer and what the call reads of it, once or again.
A call's kernels are read from its captured (never launched) graph, by name."""
import ctypes
import re

import pytest
import torch

BF16, F32 = 1, 0


class _KernelNode(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint)]


def _kernels(call):
    """Names of the kernels that call(stream) launches."""
    hip = ctypes.CDLL("libamdhip64.so.7")  # (the one that torch has loaded)
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(stream.cuda_stream)  # (scratch is allocated)
    torch.cuda.synchronize()
    graph, s = ctypes.c_void_p(), ctypes.c_void_p(stream.cuda_stream)
    assert hip.hipStreamBeginCapture(s, 2) == 0
    call(stream.cuda_stream)
    assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    count = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    names = []
    for node in nodes:
        kind, p = ctypes.c_int(), _KernelNode()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0 and kind.value == 0
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        names.append(hip.hipKernelNameRefByPtr(p.func, s).decode())
    assert hip.hipGraphDestroy(graph) == 0
    return names


_PAST = re.compile(r"StreamBF16|prefill_stream_kernel|down_gemm_stream_kernel|(prefill|down_gemm)_rows_kernelILi\dELb1E")
_ROWS = re.compile(r"probe_(step_)?read_kernel|decode_fused_kernel|gateup\w*_kernel|skinny_\w+_kernel|down_kernel|down_gemm_\w*(rows|dma|stream|bf16)_kernel|"
                   r"prefill_(mma|deep|stream|rows|bf16)_kernel|input_side_scores_kernel")


def _past_the_caches(call):
    """For every kernel of the call that reads weight rows, in order: whether past the caches."""
    return [bool(_PAST.search(n)) for n in _kernels(call) if _ROWS.search(n)]


@pytest.fixture
def layer(request):
    from paper_2602_06822_amd import binding as pop
    d, m = request.param
    w = [torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((m, d), (m, d), (d, m))]
    h = pop.pop_layer_create(d, m, BF16, *w, 1024, 8)
    x = torch.zeros((512, d), dtype=torch.bfloat16, device="cuda")
    y = torch.empty((512, d), device="cuda")
    try:
        yield pop, h, m, x, y
    finally:
        torch.cuda.synchronize()
        pop.pop_layer_destroy(h)


# (d, m of 67, 94, 201 and 251 MB of weights; tokens): with half of the channels active, six layers in turn gain from 80 MiB on in decode steps,
# three in a stand-alone FFN from 240 MiB on
FFN = [((2048, 5504), False), ((2560, 6144), False), ((4096, 8192), False), ((4096, 10240), True)]


@pytest.mark.gpu
@pytest.mark.parametrize("layer,past", FFN, indirect=["layer"])
@pytest.mark.parametrize("T", [1, 2, 8, 12, 24, 40])
@pytest.mark.parametrize("own_masks", [False, True])
def test_stand_alone_ffn(layer, past, T, own_masks):
    pop, h, m, x, y = layer
    mask = torch.ones((T if own_masks else 1, m), dtype=torch.uint8, device="cuda")
    got = _past_the_caches(lambda s: pop.pop_pruned_ffn(h, x[:T], T, mask, mask.shape[0], y[:T], F32, stream=s))
    assert got == [past, past]


@pytest.mark.gpu
@pytest.mark.parametrize("layer,past", [((2048, 6826), False), ((2048, 6827), True)], indirect=["layer"])
@pytest.mark.parametrize("B", [1, 2, 3, 8])
def test_decode_step(layer, past, B):
    pop, h, m, x, y = layer
    n_ret, n_cand = m // 2, m // 8
    pop.pop_prefill_partition(h, x[:64], 64, n_ret, n_cand)
    got = _past_the_caches(lambda s: pop.pop_decode_step(h, x[:B], B, [n_cand // 2] * B, y[:B], F32, stream=s))
    assert got and all(g == past for g in got)


# Gate and up rows that the same call reads again (input-side scores and the forward pass after them, an FFN of several passes) are left in the
# cache up to layers of 240 MiB and 384 MiB
@pytest.mark.gpu
@pytest.mark.parametrize("layer,past", [((4096, 8192), False), ((4096, 10240), True), ((4104, 8000), False), ((4104, 12000), True)], indirect=["layer"])
@pytest.mark.parametrize("T", [4, 24, 40])
def test_rows_read_again(layer, past, T):
    pop, h, m, x, y = layer
    by_64 = x.shape[1] % 64 == 0  # (other widths have no direct loads: tokens eight at a time, or the register-staged kernels)
    n_ret, n_cand = m // 2, m // 8

    def forward(s):
        pop.pop_prefill_forward(h, x[:T], T, n_ret, n_cand, n_cand // 2, y[:T], F32, stream=s)

    pop.pop_layer_set_importance(h, pop.POP_IMPORTANCE_INPUT_SIDE)
    scores, *ffn = _past_the_caches(forward)
    assert scores == past
    if T >= 32:
        # (the register-staged contraction over a list: a form for either tile, one of which has nothing to do)
        assert ffn == ([past, past] if by_64 else [False, False, False])
    else:
        passes = 1 if by_64 else (T + 7) // 8
        assert ffn == [past and passes == 1] * 2 * passes
    mask = torch.ones((1, m), dtype=torch.uint8, device="cuda")
    got = _past_the_caches(lambda s: pop.pop_pruned_ffn(h, x[:T], T, mask, 1, y[:T], F32, stream=s))
    if T < 32 and not by_64:
        assert got == [past and passes == 1] * 2 * passes
    pop.pop_layer_set_importance(h, pop.POP_IMPORTANCE_OUTPUT_SIDE)
    if T < 32 and not by_64:
        scores, *ffn = _past_the_caches(forward)
        assert not scores and ffn == [past and passes == 1] * 2 * passes


# A partition reads gate and up alone: from 144 MiB of weights on (up to 31 tokens, as the forward pass, from 128), and where two token tiles
# share a chunk of channels from 240
@pytest.mark.gpu
@pytest.mark.parametrize("layer,T,want", [
    ((3200, 7200), 16, True), ((3200, 7200), 40, False), ((4096, 6400), 40, True), ((4096, 6400), 128, False),
    ((4096, 8192), 240, False), ((4096, 10240), 240, True), ((4096, 10240), 1024, False),
    # (the second tile seven eighths full, half on rows of up to 8 KB where a compute unit runs one tile)
    ((5120, 13824), 64, True), ((5120, 13824), 65, False), ((5120, 13824), 119, False), ((5120, 13824), 120, True),
    ((6144, 8192), 224, False), ((6144, 8192), 240, True), ((4096, 10240), 95, False), ((4096, 10240), 96, True), ((4096, 10240), 160, False)], indirect=["layer"])
def test_prompt(layer, T, want):
    pop, h, m, x, y = layer
    x = torch.zeros((T, x.shape[1]), dtype=torch.bfloat16, device="cuda")
    y = torch.empty(x.shape, device="cuda")
    n_ret, n_cand = m // 2, m // 8
    got = _past_the_caches(lambda s: pop.pop_prefill_partition(h, x, T, n_ret, n_cand, stream=s))
    assert got == [want]
    contraction, down = _past_the_caches(lambda s: pop.pop_prefill_forward(h, x, T, n_ret, n_cand, n_cand // 2, y, F32, stream=s))
    # (all of gate and up and most of down: one token tile from 128 MiB on)
    assert contraction == (want or T == 40) and down == (T <= 320)


@pytest.mark.gpu
@pytest.mark.parametrize("layer,want", [((3200, 7200), False), ((4096, 6400), True)], indirect=["layer"])
def test_input_side_partition(layer, want):
    pop, h, m, x, y = layer
    pop.pop_layer_set_importance(h, pop.POP_IMPORTANCE_INPUT_SIDE)
    assert _past_the_caches(lambda s: pop.pop_prefill_partition(h, x[:100], 100, m // 2, m // 8, stream=s)) == [want]


# The bare reads that a step is held against load as the step does
@pytest.mark.gpu
@pytest.mark.parametrize("layer,past", [((2048, 6826), False), ((2048, 6827), True)], indirect=["layer"])
def test_probe_reads(layer, past):
    pop, h, m, x, y = layer
    sink = torch.zeros(1, dtype=torch.int32, device="cuda")
    pop.pop_prefill_partition(h, x[:64], 64, m // 2, m // 8)
    assert _past_the_caches(lambda s: pop.pop_probe_step_read(h, m // 16, 256, sink, stream=s)) == [past]
    buf = torch.zeros(6 * 2048 * m, dtype=torch.uint8, device="cuda")
    assert _past_the_caches(lambda s: pop.pop_probe_read(buf, buf.numel(), 256, sink, stream=s)) == [past]
