"""GPU tests of the weight quantizer that reads large matrices once (csrc/quant_weights.hip): codes and gamma are those of the two
passes bit for bit, whatever the sample says of the matrix.  bitnet_quantize_weights_static has no room for notes and always
takes the two passes, which the parity tests compare with the oracle."""
import pytest

from paper_2402_17764_amd import binding as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _normal(N, K, dtype, seed, scale=0.02):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.empty((N, K), dtype=dtype, device="cuda").normal_(0.0, scale, generator=g)


def _two_passes(W):
    packed = torch.empty(B.packed_bytes(*W.shape), dtype=torch.uint8, device="cuda")
    return B.quantize_weights_static(W, packed, torch.empty(1, device="cuda"))


def _check(W, what):
    N, K = W.shape
    assert B.quantize_weights_workspace(N, K) > 32768
    print("once", what, N, K, W.dtype, flush=True)
    ref, gamma = _two_passes(W)
    small = torch.empty(32768, dtype=torch.uint8, device="cuda")
    for ws in (None, torch.full((B.quantize_weights_workspace(N, K),), 0xFF, dtype=torch.uint8, device="cuda"), small):
        p, g = B.quantize_weights(W, workspace=ws)
        assert torch.equal(g.view(torch.int32), gamma.view(torch.int32)) and torch.equal(p, ref)


# whole and partial last row blocks and items, rows of any length, one item a row block
@pytest.mark.parametrize("dtype,N,K", [(torch.float32, 9600, 3200), (torch.float32, 5005, 5124), (torch.float32, 6007, 4301), (torch.float32, 400001, 64),
                                       (torch.float32, 17, 1 << 18 | 0), (torch.float32, 90, 262143),
                                       (torch.float32, 1100003, 100), (torch.bfloat16, 700001, 250), (torch.bfloat16, 16384, 4112), (torch.bfloat16, 15001, 5001), (torch.bfloat16, 1100003, 63), (torch.bfloat16, 300, 262144 - 8)])
def test_normal_weights(gpu_lib, dtype, N, K):
    W = _normal(N, K, dtype, N + K)
    if W.numel() * W.element_size() >= (128 if dtype == torch.bfloat16 else 96) << 20:
        _check(W, "normal")
    else:                                                  # below the line: the two passes
        ref, gamma = _two_passes(W)
        p, g = B.quantize_weights(W)
        assert torch.equal(p, ref) and torch.equal(g, gamma)


def _cases(W):
    N, K = W.shape
    dtype = W.dtype
    outlier = W.clone()
    outlier[N // 2 + 1, K // 3] = 2.0e6                    # a weight that no sample sees and that most of the mean hangs on
    yield "outlier", outlier
    u = torch.rand((N, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(7))
    s = torch.where(W < 0, -1.0, 1.0)
    yield "at the threshold", (torch.where(u < 0.5, 1.0, 1.0 / 3.0) * s).to(dtype)       # gamma 2/3: half of the weights are noted
    yield "at the threshold in bf16", (torch.where(u < 1.0 / 3.0, 1.0, 0.25) * s).to(dtype)     # gamma 1/2
    yield "one magnitude", (0.75 * s).to(dtype)
    yield "two neighbours", (torch.where(u < 0.5, 1.0, 1.0078125) * s).to(dtype)
    yield "zeros", torch.zeros_like(W)
    almost = torch.zeros_like(W)
    almost[N - 1, K - 1] = -3.0
    yield "one weight", almost
    yield "half zeros", torch.where(u < 0.5, torch.zeros_like(W), W)
    rows = W.clone()
    rows[: N // 3] *= 1e-3
    rows[N - 40:] *= 300.0
    yield "rows of different scales", rows
    spread = (W.double() * torch.exp2(torch.randint(-40, 40, (1, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(8)).double())).to(dtype)
    yield "columns over 80 binades", spread
    yield "near the smallest floats", (W.double() * 2.0 ** -126).to(dtype)
    yield "near the largest floats", (W.double() * 2.0 ** 124).to(dtype)
    yield "ternary already", (torch.where(u < 0.4, 0.0, 0.013) * s).to(dtype)


@pytest.mark.parametrize("dtype,N,K", [(torch.float32, 6160, 4100), (torch.float32, 6003, 4301), (torch.bfloat16, 16400, 4104), (torch.bfloat16, 15001, 5001)])
def test_matrices_that_the_sample_does_not_describe(gpu_lib, dtype, N, K):
    for what, W in _cases(_normal(N, K, dtype, 5)):
        _check(W, what)


@pytest.mark.parametrize("dtype,N,K", [(torch.float32, 6160, 4100), (torch.bfloat16, 15001, 5001)])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
def test_not_finite(gpu_lib, dtype, N, K, value):
    """one such weight, which no sample sees, one in every 61 columns, which every sample sees, and nothing else"""
    for step in (0, 61, 1):
        W = _normal(N, K, dtype, 6)
        if step:
            W[:, ::step] = value
        else:
            W[N // 2 + 1, K // 3] = value
        print("once", value, step, N, K, dtype, flush=True)
        ref, gamma = _two_passes(W)
        p, g = B.quantize_weights(W)
        assert torch.equal(p, ref)
        assert torch.equal(g, gamma) or (torch.isnan(g).all() and torch.isnan(gamma).all())


@pytest.mark.parametrize("dtype,rows,K", [(torch.float32, [3200, 3200, 3200], 3200), (torch.float32, [6400, 800, 1013], 4100),
                                          (torch.bfloat16, [16000, 16, 16384], 2304), (torch.bfloat16, [1024] * 17 + [2048], 4096)])
def test_segments(gpu_lib, dtype, rows, K):
    W = _normal(sum(rows), K, dtype, 11)
    at = 0
    for i, n in enumerate(rows):
        W[at:at + n] *= 1.0 + i                            # a gamma of its own for each
        at += n
    print("once, segments", rows, K, dtype, flush=True)
    full, gammas = B.quantize_weights_segmented(W, rows)
    small = torch.empty(32768, dtype=torch.uint8, device="cuda")
    p, g = B.quantize_weights_segmented(W, rows, workspace=small)
    assert torch.equal(p, full) and torch.equal(g.view(torch.int32), gammas.view(torch.int32))
    at = 0
    codes = B.unpack_weights(full, sum(rows), K)
    for n in rows:
        packed, gamma = _two_passes(W[at:at + n].contiguous())
        assert (gammas[at // 16:(at + n + 15) // 16] == gamma).all()
        assert torch.equal(codes[at:at + n], B.unpack_weights(packed, n, K))
        at += n


def test_captured_and_on_two_streams(gpu_lib):
    """three launches that share nothing but their workspace: replays on changed weights, and two streams at once"""
    W = [_normal(9600, 3200, torch.float32, s) for s in (1, 2)]
    V = W[0].clone()
    n = B.quantize_weights_workspace(9600, 3200)
    ws = [torch.empty(n, dtype=torch.uint8, device="cuda") for _ in W]
    out = [(torch.empty(B.packed_bytes(9600, 3200), dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")) for _ in W]
    ref = [_two_passes(w) for w in W]
    B.quantize_weights(V, packed=out[0][0], gamma=out[0][1], workspace=ws[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.quantize_weights(V, packed=out[0][0], gamma=out[0][1], workspace=ws[0])
    for k in (1, 0, 1):
        V.copy_(W[k])
        graph.replay()
        assert torch.equal(out[0][0], ref[k][0]) and torch.equal(out[0][1], ref[k][1])
    streams = [torch.cuda.Stream() for _ in W]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        for k, s in enumerate(streams):
            with torch.cuda.stream(s):
                B.quantize_weights(W[k], packed=out[k][0], gamma=out[k][1], workspace=ws[k])
    torch.cuda.synchronize()
    for k in range(2):
        assert torch.equal(out[k][0], ref[k][0]) and torch.equal(out[k][1], ref[k][1])


def _bounds(W, rows):
    """what the sample said of each segment, out of the scratch (csrc/quant_weights.hip, kBoundsAt): gamma's bounds, empty where it says nothing"""
    N, K = W.shape
    ws = torch.zeros(B.quantize_weights_workspace(N, K), dtype=torch.uint8, device="cuda")
    _, gammas = B.quantize_weights_segmented(W, rows, workspace=ws)
    at = (1024 + 16) * 16 + (256 + 16) * 16 + (1024 + 16) * 4
    return ws[at:at + 16 * len(rows)].view(torch.float32).view(-1, 4).cpu(), gammas


@pytest.mark.parametrize("dtype,rows,K", [(torch.float32, [3200] * 3, 3200), (torch.bfloat16, [8192], 8192), (torch.float32, [7001], 4099), (torch.bfloat16, [28672], 8192)])
@pytest.mark.parametrize("deviation,block", [(0.1, 1), (0.3, 1), (0.5, 1), (0.5, 128)])
def test_rows_of_different_scale_are_read_once(gpu_lib, dtype, rows, K, deviation, block):
    """rows, or heads of 128 rows, whose scales deviate: the sample bounds gamma all the same"""
    W = _normal(sum(rows), K, dtype, 21)
    blocks = -(-W.shape[0] // block)
    scale = torch.exp(deviation * torch.randn((blocks, 1), device="cuda", generator=torch.Generator(device="cuda").manual_seed(22)))
    W.mul_(scale.repeat_interleave(block, 0)[: W.shape[0]].to(dtype))
    print("once, rows of different scale", rows, K, dtype, deviation, block, flush=True)
    bounds, gammas = _bounds(W, rows)
    at = 0
    for n, (lo, hi, _, _) in zip(rows, bounds.tolist()):
        assert lo <= gammas[at // 16].item() <= hi
        at += n


def _times(calls, rounds=5):
    """us of each of the calls, the best of several rounds in turn"""
    best = [float("inf")] * len(calls)
    for r in range(rounds + 1):
        for i, call in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(6):
                call()
            b.record()
            torch.cuda.synchronize()
            if r:                                          # the first round warms up
                best[i] = min(best[i], a.elapsed_time(b) * 1e3 / 6)
    return best


def _cost_of_failing(W):
    """the time of quantize_weights over that of the two passes"""
    N, K = W.shape
    packed, gamma = torch.empty(B.packed_bytes(N, K), dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")
    ws = torch.empty(B.quantize_weights_workspace(N, K), dtype=torch.uint8, device="cuda")
    two, once = _times([lambda: B.quantize_weights_static(W, packed, gamma), lambda: B.quantize_weights(W, packed=packed, gamma=gamma, workspace=ws)])
    print("once, cost of failing: %.1f us, %.1f in two passes" % (once, two), flush=True)
    return once / two


def test_cost_without_bounds(gpu_lib):
    """rows whose scales spread so far that the sample says nothing: added up, then coded, not coded twice (1.09 of the two passes; coded twice 1.23)"""
    W = _normal(57344, 8192, torch.bfloat16, 31)
    W.mul_(torch.exp(2.0 * torch.randn((57344, 1), device="cuda", generator=torch.Generator(device="cuda").manual_seed(32))).to(torch.bfloat16))
    assert _cost_of_failing(W) < 1.16


def test_cost_of_full_pads(gpu_lib):
    """a value of two thirds of the weights right at the threshold: once a pad is full nothing is noted any more (1.15 of the two passes; noted to
    the end 1.7)"""
    W = _normal(57344, 8192, torch.bfloat16, 33)
    for rows in W.split(4096):
        u = torch.rand(rows.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(34))
        rows.copy_(torch.where(u < 1.0 / 3.0, 1.0, 0.25) * torch.where(rows < 0, -1.0, 1.0))         # gamma 0.5
    assert _cost_of_failing(W) < 1.4


@pytest.mark.parametrize("dtype,N,K,once", [(torch.float32, 400001, 64, False), (torch.float32, 1700000, 64, False), (torch.float32, 1100003, 100, True),
                                            (torch.float32, 101000, 260, False), (torch.float32, 102400, 256, True), (torch.bfloat16, 530000, 128, False),
                                            (torch.bfloat16, 266000, 256, False), (torch.bfloat16, 53200, 1280, False), (torch.bfloat16, 820000, 256, True),
                                            (torch.bfloat16, 16700, 4100, True)])
def test_narrow_matrices_are_read_twice(gpu_lib, dtype, N, K, once):
    """where the lanes past a row's end cost more than the second read; the bounds in the scratch are written by the single read alone"""
    W = _normal(N, K, dtype, 41)
    ws = torch.full((B.quantize_weights_workspace(N, K),), 0xFF, dtype=torch.uint8, device="cuda")
    print("once, narrow", N, K, dtype, flush=True)
    B.quantize_weights(W, workspace=ws)
    at = (1024 + 16) * 16 + (256 + 16) * 16 + (1024 + 16) * 4
    assert bool((ws[at:at + 16] == 0xFF).all()) != once


def test_scratch_is_allocated_where_it_is_used(gpu_lib):
    """the notes' room belongs to the 2-bit format: 5-trit calls and |W| sums allocate the partial sums alone"""
    W = _normal(9600, 3200, torch.float32, 51)
    packed, gamma = torch.empty(B.packed_bytes(9600, 3200, B.PACK_TRIT5), dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    for call in (lambda: B.quantize_weights(W, B.PACK_TRIT5, packed, gamma), lambda: B.abs_sum(W, out)):
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        call()
        assert torch.cuda.max_memory_allocated() - before <= 32768
