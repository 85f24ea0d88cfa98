"""GPU tests of single kernel forms at the sizes where each can go wrong -- the edges of its tiles, its remainders, the
smallest and largest of its range -- against the CPU oracle (bit for bit: codes, scales, accumulators) or, where a form
stands in for a slower one, against that one on the same inputs."""
import numpy as np
import pytest

import oracle
from layout_ref import decode_2bit
from paper_2402_17764_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def dev_bf16(bits_u16):
    return torch.from_numpy(bits_u16.view(np.int16).copy()).cuda().view(torch.bfloat16)


def check_packed(gpu_lib, W, packed, gamma):
    N, K = W.shape
    codes_ref, gamma_ref = oracle.quantize_weights(W)
    assert gamma.cpu().numpy()[0].tobytes() == np.float32(gamma_ref).tobytes(), "gamma bits differ"
    dec, pad_zero = decode_2bit(packed.cpu().numpy(), N, K)
    assert pad_zero and np.array_equal(dec, codes_ref)


# the bf16 packing pass with 16-byte loads (K a multiple of 8): items of two K steps -- less than one, one, two, three steps,
# partial last quads, rows that do not fill a row block, more items than workgroups
@pytest.mark.parametrize("N,K", [(1, 8), (16, 64), (17, 256), (33, 264), (100, 512), (16, 520), (15, 776), (250, 4104), (2056, 8200)])
def test_pack_bf16_rows_of_eight(gpu_lib, N, K):
    W, bits = synth.to_bf16(synth.weights(N, K, config=2, layer=N % 5))
    packed, gamma = gpu_lib.quantize_weights(dev_bf16(bits).view(N, K))
    check_packed(gpu_lib, W, packed, gamma)


# segments quantized side by side: very unequal ones, more than one launch takes (16), rows of every load width
@pytest.mark.parametrize("rows,K,bf16", [([16] * 17 + [5], 40, False), ([4096, 16, 7], 264, True), ([16, 2048, 512, 512], 1030, False),
                                         ([3200, 3200, 3200], 520, True), ([48] * 35, 77, True)])
def test_segments_side_by_side(gpu_lib, rows, K, bf16):
    N = sum(rows)
    W = synth.weights(N, K, config=1, layer=len(rows)) * np.repeat(np.linspace(0.5, 2.0, len(rows)), rows).astype(np.float32)[:, None]
    bits = None
    if bf16:
        W, bits = synth.to_bf16(W)
    packed, gamma_rb = gpu_lib.quantize_weights_segmented(dev_bf16(bits).view(N, K) if bf16 else dev(W), rows)
    dec, pad_zero = decode_2bit(packed.cpu().numpy(), N, K)
    assert pad_zero
    g, row = gamma_rb.cpu().numpy(), 0
    for r in rows:
        codes_ref, gamma_ref = oracle.quantize_weights(np.ascontiguousarray(W[row:row + r]))
        assert np.array_equal(dec[row:row + r], codes_ref)
        blocks = g[row // 16:(row + r + 15) // 16]
        assert np.all(blocks.view(np.uint32) == np.float32(gamma_ref).view(np.uint32))
        row += r


# x_q rows of any length and alignment: the decode form (up to 16 tokens, both its launch shapes, K below one 16-byte piece,
# below and above one K step) and the tiles of the GEMM (two K groups, four waves, 64 x 256), each with ragged rows and tokens
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (1, 40, 7), (3, 100, 255), (16, 33, 1001), (2, 16400, 259), (1, 300, 4097),
                                   (17, 130, 5), (64, 128, 255), (65, 129, 257), (77, 1003, 2050), (100, 3000, 513), (200, 1000, 3333),
                                   (1030, 2500, 301), (700, 25000, 77), (16, 50, 8001),
                                   # more than 16 tokens in tiles over the grid: a full and a partial last tile, K beyond 64 KiB of
                                   # LDS, the most workgroups of the form and one more
                                   (32, 70, 333), (40, 1900, 3900), (33, 100, 5000), (8192, 16, 33), (8193, 16, 33),
                                   # the most LDS a decode workgroup takes
                                   (33, 100, 4863), (1, 40, 81407),
                                   # K a multiple of 16, whole K steps among them, which the second call below brings here unaligned
                                   (16, 100, 256), (3, 500, 272), (40, 300, 256), (2, 300, 4096), (300, 1000, 272), (100, 3000, 4096),
                                   (2000, 9000, 256),
                                   # the shortest rows these forms are chosen for (below, a thread per output is faster)
                                   (5, 300, 15), (16, 500, 13), (3000, 1100, 1), (3000, 1100, 3)])
@pytest.mark.parametrize("y", ["I32", "F32", "BF16"])
def test_rows_of_any_length(gpu_lib, M, N, K, y):
    packed, gamma = gpu_lib.quantize_weights(dev(synth.weights(N, K, config=1, layer=M % 7)))
    xq, sx = gpu_lib.quantize_acts(dev(synth.activations(M, K, config=1, layer=N % 7)))
    yt = getattr(gpu_lib, y)
    # one byte past an aligned address (that nothing behind x_q is read is the business of the address replica on the CPU)
    buf = torch.empty(M * K + 1, dtype=torch.int8, device="cuda")
    buf[1:] = xq.reshape(-1)
    big = torch.full((M * N + 64,), 7, dtype=gpu_lib._OUT[yt], device="cuda")
    want = gpu_lib.linear(xq, sx, packed, gamma, N, y_dtype=yt, kernel=gpu_lib.KERNEL_REFERENCE)
    assert torch.equal(gpu_lib.linear(xq, sx, packed, gamma, N, y_dtype=yt), want)
    assert torch.equal(gpu_lib.linear(buf[1:].view(M, K), sx, packed, gamma, N, y_dtype=yt, y=big[:M * N].view(M, N)), want)
    assert bool((big[M * N:] == 7).all())


@pytest.mark.parametrize("M,N,K", [(5, 100, 130), (40, 300, 1030)])
def test_rows_of_any_length_with_a_gamma_per_block(gpu_lib, M, N, K):
    rows = [48, N - 48]
    packed, gamma_rb = gpu_lib.quantize_weights_segmented(dev(synth.weights(N, K, config=1, layer=1)), rows)
    xq, sx = gpu_lib.quantize_acts(dev(synth.activations(M, K, config=1, layer=2)))
    want = gpu_lib.linear_segmented(xq, sx, packed, gamma_rb, N, kernel=gpu_lib.KERNEL_REFERENCE)
    got = gpu_lib.linear_segmented(xq, sx, packed, gamma_rb, N)
    assert torch.allclose(got, want, rtol=3 * 2.0 ** -23, atol=0.0)      # gamma * (s_x / 127) or (gamma * s_x) / 127: two roundings


def test_native_marshalling_checks_its_arguments(gpu_lib):
    """What binding.py's entry points refuse, and that a non-default stream, given outputs and keyword arguments arrive."""
    B, M, N, K = gpu_lib, 3, 64, 128
    packed, gamma = B.quantize_weights(dev(synth.weights(N, K)))
    x = dev(synth.activations(M, K))
    xq, sx = B.quantize_acts(x)
    f64 = x.double()
    for call, err in [(lambda: B.quantize_acts(f64), TypeError), (lambda: B.quantize_acts(x.t()), ValueError),
                      (lambda: B.quantize_acts(x[0]), ValueError), (lambda: B.quantize_acts(x, xq=xq.int()), TypeError),
                      (lambda: B.rmsnorm_quantize(x, g=torch.ones(K - 1, device="cuda")), ValueError),
                      (lambda: B.rmsnorm_quantize(x, eps="a"), ValueError),
                      (lambda: B.rmsnorm_quantize(x, eps=-1.0), B.BitnetError),
                      (lambda: B.swiglu_quantize(x[:, :127].contiguous()), ValueError),
                      (lambda: B.linear(x, sx, packed, gamma, N), TypeError), (lambda: B.linear(xq, sx.double(), packed, gamma, N), TypeError),
                      (lambda: B.linear(xq, sx, packed, gamma, N, y_dtype=9), KeyError),
                      (lambda: B.linear(xq, sx, packed, gamma, N, y_dtype=torch.float32), KeyError), (lambda: B.linear_fused(x, packed, gamma, N, y_dtype="F32"), KeyError),
                      (lambda: B.linear(xq, sx, packed, gamma, 16.5), TypeError),
                      (lambda: B.linear(xq, sx, packed, gamma, 0), B.BitnetError),
                      (lambda: B.linear(xq, sx, packed, gamma, N, y=torch.empty(M, N, device="cuda", dtype=torch.bfloat16)), TypeError),
                      (lambda: B.linear(xq, sx, packed, gamma, N, fmt=7), B.BitnetError),
                      (lambda: B.linear(xq, sx, packed, gamma, N, kernel=77), B.BitnetError),
                      (lambda: B.linear_segmented(xq, sx, packed, gamma, N), ValueError),
                      (lambda: B.linear_fused_segmented(x, packed, gamma, N), ValueError),
                      (lambda: B.rmsnorm_linear_fused(x, None, 1e-6, packed, gamma, N, segmented=True), ValueError),
                      (lambda: B.ffn_gate_up_fused(x, packed, gamma, 24), B.BitnetError),
                      (lambda: B.ffn_gate_up_fused(x, packed, gamma, 32, h_dtype=B.I32), B.BitnetError)]:
        with pytest.raises(err):
            call()
    with pytest.raises(B.BitnetError) as e:
        B.linear(xq, sx, packed, gamma, N, fmt=7)
    assert e.value.status == 4 and "bitnet_linear" in str(e.value)
    want = B.linear(xq, sx, packed, gamma, N, y_dtype=B.BF16)
    y, s = torch.empty(M, N, device="cuda", dtype=torch.bfloat16), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        assert B.linear(xq=xq, sx=sx, packed=packed, gamma=gamma, N=np.int64(N), y_dtype=B.BF16, y=y) is y
    s.synchronize()
    assert torch.equal(y, want)
    graph = torch.cuda.CUDAGraph()          # captured where the current stream says, replayed on new inputs
    with torch.cuda.graph(graph):
        yg = B.linear_fused(x, packed, gamma, N, y_dtype=B.BF16)
    x.mul_(-1.0)
    graph.replay()
    assert torch.equal(yg, -want)


# SwiGLU by table: every finite bf16 gate, in rows of each width the form takes (one, two and four loads per thread, partly
# filled), the up half chosen so that every product is of one magnitude and a neighbouring table entry would show in the
# codes; more tokens than workgroups; rows with gates outside the table among the others
@pytest.mark.parametrize("F", [5120, 8192, 8200, 11008, 16384, 16392, 32768])
def test_swiglu_table_every_gate(gpu_lib, F):
    bits = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    g = (bits.astype(np.uint32) << 16).view(np.float32)
    bits = bits[np.isfinite(g) & (np.abs(g) < 2.0 ** 60) & (g > -80) & (np.abs(g) > 2.0 ** -60)]
    rng = np.random.default_rng(F)
    M = 300
    gb = rng.permutation(np.resize(bits, M * F)).reshape(M, F)
    g64 = (gb.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    silu = g64 / (1.0 + np.exp(-g64))
    up, ub = synth.to_bf16((rng.uniform(0.3, 1.0, (M, F)) / silu).astype(np.float32))
    gu = np.concatenate([(gb.astype(np.uint32) << 16).view(np.float32), up], axis=1)
    hq_ref, sh_ref, _ = oracle.swiglu_quantize(np.ascontiguousarray(gu))
    hq, sh = gpu_lib.swiglu_quantize(dev_bf16(np.concatenate([gb, ub], axis=1)).view(M, 2 * F))
    assert sh.cpu().numpy().tobytes() == sh_ref.tobytes()
    assert np.array_equal(hq.cpu().numpy(), hq_ref)


# ... and every bf16 gate there is, bit for bit: a token's scale is the |h| of its largest element, so tokens that hold one gate
# throughout, and tokens whose other elements are gated to zero, show the fp32 silu of each gate; against the arithmetic form,
# which fp32 input takes, on the same values
@pytest.mark.parametrize("alone", [True, False])
def test_swiglu_table_bits_of_every_gate(gpu_lib, alone):
    F, M = 5120, 8192
    gen = torch.Generator(device="cuda").manual_seed(5)
    for first in range(0, 65536, M):
        bits = torch.arange(first, first + M, device="cuda", dtype=torch.int32)
        gate = (bits << 16).view(torch.float32)
        finite = torch.isfinite(gate)
        g64 = gate.double()
        silu = torch.where(gate < -80, g64 / 1.65e38, g64 * torch.sigmoid(g64)).abs().clamp_min(2.0 ** -140)
        up = (1.0 / silu).clamp_max(3.38e38).clamp_min(2.0 ** -126)                     # |h| near 1 (0.01 for the least of gates)
        gu = torch.randn(M, 2 * F, device="cuda", generator=gen)
        gu[:, F:] = up[:, None].float() if alone else 0.0
        if alone:
            gu[:, :F] = gate[:, None]
        at = torch.randint(0, F, (M, 1), device="cuda", generator=gen)
        gu.scatter_(1, at, gate[:, None])
        gu.scatter_(1, at + F, up[:, None].float())
        x = gu.bfloat16()
        hq, sh = gpu_lib.swiglu_quantize(x)
        hq_want, sh_want = gpu_lib.swiglu_quantize(x.float())
        assert torch.equal(sh[finite].view(torch.int32), sh_want[finite].view(torch.int32))
        assert torch.equal(hq[finite], hq_want[finite])
        assert torch.equal(sh.isnan(), sh_want.isnan()) and torch.equal(sh.isinf(), sh_want.isinf())
        near = finite & (gate != 0)
        assert bool((sh[near] > 0.009).all())                                           # nothing hidden behind the least scale


@pytest.mark.parametrize("M,F", [(600, 5120), (257, 11008), (256, 5128), (255, 5128), (1100, 8640), (8, 8192), (7, 8192), (63, 9208), (64, 8192), (8, 9216), (7, 9216), (1, 16384), (1023, 264), (1024, 264),
                                 # 1024 threads a token or 256: rows on either side of the rule, read in chunks and element by element
                                 (64, 1024), (64, 1028), (600, 1796), (600, 1800), (64, 256), (64, 257), (300, 449), (300, 451)])
@pytest.mark.parametrize("bf16", [False, True])
def test_swiglu_many_tokens(gpu_lib, M, F, bf16):
    gu, bits = synth.activations(M, 2 * F, config=2, layer=F % 5, tensor=5, bf16=True)
    gu[:, :F:7] *= 0.0                        # zeros of both signs have an entry, these magnitudes have none
    gu[0, 1:F:9] = 1e-7
    gu[-1, 2:F:9] = -700.0
    gu[M // 2, 3:F:9] = 1e-39
    gu, bits = synth.to_bf16(gu)
    hq_ref, sh_ref, _ = oracle.swiglu_quantize(gu)
    hq, sh = gpu_lib.swiglu_quantize(dev_bf16(bits).view(M, 2 * F) if bf16 else dev(gu))
    assert sh.cpu().numpy().tobytes() == sh_ref.tobytes()
    assert np.array_equal(hq.cpu().numpy(), hq_ref)


# RMSNorm at the edges of its workgroup sizes: 256 threads up to four loads each at any count of tokens, 1024 beyond for few
@pytest.mark.parametrize("M,K", [(1, 8192), (1, 8200), (63, 8200), (64, 8200), (29, 4096), (63, 4100), (1, 4104), (1, 16392)])
@pytest.mark.parametrize("bf16", [False, True])
def test_rmsnorm_workgroup_sizes(gpu_lib, M, K, bf16):
    x, bits = synth.activations(M, K, config=2, layer=K % 7, tensor=3, bf16=True)
    g = (1.0 + 0.25 * np.random.default_rng(K).standard_normal(K)).astype(np.float32)
    xq_ref, sx_ref, _ = oracle.rmsnorm_quantize(x, g, 1e-6)
    xq, sx = gpu_lib.rmsnorm_quantize(dev_bf16(bits).view(M, K) if bf16 else dev(x), dev(g), 1e-6)
    assert sx.cpu().numpy().tobytes() == sx_ref.tobytes()
    assert np.array_equal(xq.cpu().numpy(), xq_ref)


# ... and with the gain requested ahead of the reduction (up to 256 tokens), every count of loads per thread
@pytest.mark.parametrize("M,K", [(256, 1032), (257, 1032), (256, 2056), (100, 7176), (5, 20488)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("with_gain", [False, True])
def test_rmsnorm_gain_first(gpu_lib, M, K, bf16, with_gain):
    x, bits = synth.activations(M, K, config=2, layer=K % 7, tensor=3, bf16=True)
    g = (1.0 + 0.25 * np.random.default_rng(K).standard_normal(K)).astype(np.float32) if with_gain else None
    xq_ref, sx_ref, _ = oracle.rmsnorm_quantize(x, g, 1e-6)
    xq, sx = gpu_lib.rmsnorm_quantize(dev_bf16(bits).view(M, K) if bf16 else dev(x), None if g is None else dev(g), 1e-6)
    assert sx.cpu().numpy().tobytes() == sx_ref.tobytes()
    assert np.array_equal(xq.cpu().numpy(), xq_ref)


def undecided_rows(K, want, seed):
    """Rows of K values whose 1 / sqrt(mean square) lies within 2^-45 of where two floats meet: a sum with fp64 rounding errors
    does not decide r for them."""
    rng, found, tried = np.random.default_rng(seed), [], 0
    while sum(len(f) for f in found) < want and tried < 40_000_000:
        x = rng.standard_normal((1_000_000, K)).astype(np.float32)
        y = 1.0 / np.sqrt((x.astype(np.float64) ** 2).sum(axis=1) / K + np.float64(np.float32(1e-6)))
        found.append(x[(y * (1 - 2.0 ** -45)).astype(np.float32) != (y * (1 + 2.0 ** -45)).astype(np.float32)])
        tried += len(x)
    return np.concatenate(found)


def test_rmsnorm_exact_sum_where_the_rounded_one_does_not_decide(gpu_lib):
    K, N = 16, 32
    x = undecided_rows(K, 6, 7)
    assert len(x) >= 3
    W = synth.weights(N, K)
    packed, gamma = gpu_lib.quantize_weights(dev(W))
    for rows in (x, x[:1], np.repeat(x, 100, axis=0), np.concatenate([x, np.zeros((2, K), np.float32)])):
        xq_ref, sx_ref, _ = oracle.rmsnorm_quantize(rows, None, 1e-6)
        xq, sx = gpu_lib.rmsnorm_quantize(dev(rows), None, 1e-6)
        assert sx.cpu().numpy().tobytes() == sx_ref.tobytes()
        assert np.array_equal(xq.cpu().numpy(), xq_ref)
    for m in (1, 2, 3):      # the decode launch with the norm in front, tokens decided and undecided in one call
        rows = np.concatenate([x[:m], synth.activations(3, K)])
        xq_ref, sx_ref, _ = oracle.rmsnorm_quantize(rows, None, 1e-6)
        got = gpu_lib.rmsnorm_linear_fused(dev(rows), None, 1e-6, packed, gamma, N)
        want = gpu_lib.linear(dev(xq_ref), dev(sx_ref), packed, gamma, N)
        assert torch.equal(got, want)


# a token of zeros, alone and among others: with eps = 0 its r is 1 / 0, which no rounded sum decides
@pytest.mark.parametrize("K", [16, 4096, 8208])
@pytest.mark.parametrize("eps", [0.0, 1e-6])
def test_rmsnorm_of_a_token_of_zeros(gpu_lib, K, eps):
    N = 32
    packed, gamma = gpu_lib.quantize_weights(dev(synth.weights(N, K)))
    rows = synth.activations(3, K, config=1, layer=2)
    rows[1] = 0.0
    for x in (rows, rows[1:2]):
        xq_ref, sx_ref, _ = oracle.rmsnorm_quantize(np.ascontiguousarray(x), None, eps)
        xq, sx = gpu_lib.rmsnorm_quantize(dev(x), None, eps)
        assert sx.cpu().numpy().tobytes() == sx_ref.tobytes() and np.array_equal(xq.cpu().numpy(), xq_ref)
        assert torch.equal(gpu_lib.rmsnorm_linear_fused(dev(x), None, eps, packed, gamma, N), gpu_lib.linear(xq, sx, packed, gamma, N))


# x in rows of any length and alignment through the quantizer that holds a row in registers: less than one load, whole loads and
# a rest of every size class, the longest rows it takes and the first beyond, a base one element past an aligned address
@pytest.mark.parametrize("M,K", [(3, 1), (5, 7), (4, 9), (2, 2047), (77, 2050), (9, 4099), (2, 8187), (2, 8191), (2, 16381), (2, 16391), (300, 333),
                                 # the shortest rows it takes, and those whose last elements need a ninth load
                                 (3, 63), (3, 65), (3, 127), (3, 129), (2, 16383), (2, 8189)])
@pytest.mark.parametrize("bf16", [False, True])
def test_quantize_acts_rows_of_any_length(gpu_lib, M, K, bf16):
    x, bits = synth.activations(M, K, config=2, layer=K % 7, tensor=3, bf16=True)
    xq_ref, sx_ref = oracle.quantize_acts(x)
    xd = dev_bf16(bits).view(M, K) if bf16 else dev(x)
    off = torch.empty(M * K + 1, dtype=xd.dtype, device="cuda")
    off[1:] = xd.reshape(-1)
    out = torch.full((M * K + 65,), 0x55, dtype=torch.int8, device="cuda")
    for src in (xd, off[1:].view(M, K)):
        for dst in (None, out[1:1 + M * K].view(M, K)):
            xq, sx = gpu_lib.quantize_acts(src, xq=dst)
            assert sx.cpu().numpy().tobytes() == sx_ref.tobytes()
            assert np.array_equal(xq.cpu().numpy(), xq_ref)
    assert bool((out[1 + M * K:] == 0x55).all()) and int(out[0]) == 0x55


# the gate/up launch with the norm in front on narrow layers: K split over four waves, fewer steps than waves to a partial
# eleventh, one and two tokens; and its neighbours (three tokens, eleven steps, 513 pairs)
@pytest.mark.parametrize("M,F,K", [(1, 2752, 1024), (2, 4096, 1536), (1, 16, 16), (2, 48, 528), (1, 8192, 2560), (1, 1008, 2064), (3, 1008, 1040),
                                   (1, 1008, 2576), (1, 8208, 528)])
@pytest.mark.parametrize("bf16", [False, True])
def test_gate_up_with_norm_on_narrow_layers(gpu_lib, M, F, K, bf16):
    B = gpu_lib
    x, bits = synth.activations(M, K, config=2, layer=F % 5, bf16=True)
    g = (1.0 + 0.25 * np.random.default_rng(K).standard_normal(K)).astype(np.float32)
    packed, gamma = B.quantize_weights(dev(synth.weights(2 * F, K, config=1, layer=2)))
    xd = dev_bf16(bits).view(M, K) if bf16 else dev(x)
    gu = B.linear(*B.rmsnorm_quantize(xd, dev(g), 1e-6), packed, gamma, 2 * F)      # fp32 gate and up, each step against the oracle elsewhere
    h = B.ffn_gate_up_fused(xd, packed, gamma, F, norm=True, g=dev(g), eps=1e-6)
    _, _, h_ref = oracle.swiglu_quantize(gu.cpu().numpy())
    assert np.array_equal(h.cpu().numpy().view(np.uint32), h_ref.view(np.uint32))


# the |W| sum of bf16 weights: vectors of eight whose exponents lie just within and just beyond what one fp32 sum takes exactly,
# zeros among them, denormals, all of it mixed; gamma bit for bit
@pytest.mark.parametrize("spread", [0, 11, 12, 13, 14, 40, 100])
@pytest.mark.parametrize("N,K", [(64, 264), (2048, 3072), (3, 40)])
def test_abs_sum_bf16_exponent_spread(gpu_lib, N, K, spread):
    rng = np.random.default_rng([spread, N])
    W = (rng.uniform(1.0, 2.0, (N, K)) * 2.0 ** -rng.integers(0, spread + 1, (N, K)) * rng.choice([-1.0, 1.0], (N, K))).astype(np.float32)
    W[rng.random((N, K)) < 0.05] = 0.0
    if spread == 100:
        W *= np.float32(2.0 ** -30)          # down to denormals
    W, bits = synth.to_bf16(W)
    packed, gamma = gpu_lib.quantize_weights(dev_bf16(bits).view(N, K))
    check_packed(gpu_lib, W, packed, gamma)
    s = gpu_lib.abs_sum(dev_bf16(bits).view(N, K)).cpu().numpy()
    from fractions import Fraction
    if N * K < 100_000:
        got, want = Fraction(float(s[0])) + Fraction(float(s[1])), sum(map(Fraction, np.abs(W).astype(np.float64).ravel().tolist()))
        # 8 bits, a spread of up to 40 and 15 bits of count fit a pair of doubles; a spread of 100 does not, and each of up to
        # 2^15 additions may round the low word, which is below 2^15 roundings of the high one, by 2^-53 of itself
        assert got == want if spread <= 40 else abs(got - want) <= want * Fraction(2) ** (15 + 15 - 53 - 53)


# ... and near the top of bf16's range: eight magnitudes whose fp32 sum would, or would just not, pass the largest float (eight
# times 2^125 is 2^128), alone and among smaller ones; every entry point that takes the sum
@pytest.mark.parametrize("top", [1.9 * 2.0 ** 124, 255 / 128 * 2.0 ** 124, 2.0 ** 125, 9.97e37, 255 / 128 * 2.0 ** 127])
@pytest.mark.parametrize("spread", [0, 3, 12])
@pytest.mark.parametrize("N,K", [(16, 64), (48, 1032)])
def test_abs_sum_bf16_near_the_top_of_the_range(gpu_lib, N, K, top, spread):
    rng = np.random.default_rng([spread, K])
    W = (np.float32(top) * 2.0 ** -rng.integers(0, spread + 1, (N, K)) * rng.choice([-1.0, 1.0], (N, K))).astype(np.float32)
    W, bits = synth.to_bf16(W)
    Wd = dev_bf16(bits).view(N, K)
    packed, gamma = gpu_lib.quantize_weights(Wd)
    check_packed(gpu_lib, W, packed, gamma)
    assert np.isfinite(gamma.cpu().numpy()).all()
    from fractions import Fraction
    s = gpu_lib.abs_sum(Wd).cpu().numpy()
    assert Fraction(float(s[0])) + Fraction(float(s[1])) == sum(map(Fraction, np.abs(W).astype(np.float64).ravel().tolist()))
    codes_ref, gamma_ref = oracle.quantize_weights(W)
    packed5, gamma5 = gpu_lib.quantize_weights(Wd, gpu_lib.PACK_TRIT5)
    assert gamma5.cpu().numpy().tobytes() == np.float32(gamma_ref).tobytes()
    assert np.array_equal(gpu_lib.unpack_weights(packed5, N, K, gpu_lib.PACK_TRIT5).cpu().numpy(), codes_ref)
    packed_s, gamma_s = gpu_lib.quantize_weights_segmented(Wd, [N])
    assert torch.equal(packed_s, packed) and bool((gamma_s == gamma).all())


def test_repack_of_more_chunks_than_one_launch_takes(gpu_lib):
    """5-trit -> 2-bit with a wave per chunk (16 rows x 320 columns): 2^26 chunks would be 2^32 threads.  64 GiB of codes in; what
    comes out is compared, at both ends and where one launch ends, with the repacking of those rows alone."""
    B, K, N = gpu_lib, 1, 2 ** 30 + 40
    torch.cuda.empty_cache()
    blocks = -(-N // 16)
    if torch.cuda.mem_get_info()[0] < (90 << 30):
        pytest.skip("needs 90 GiB of GPU memory")
    p5 = torch.empty(B.packed_bytes(N, K, B.PACK_TRIT5), dtype=torch.uint8, device="cuda")
    p2 = torch.empty(B.packed_bytes(N, K), dtype=torch.uint8, device="cuda")
    assert p5.numel() == blocks * 1024 and p2.numel() == blocks * 256
    gen = torch.Generator(device="cuda").manual_seed(3)
    spots = [(0, 40), (2 ** 25 - 20, 40), (2 ** 26 - 20, 20), (blocks - 7, 7)]          # row blocks: first, how many
    for at, n in spots:
        p5[at * 1024:(at + n) * 1024] = torch.randint(0, 243, (n * 1024,), dtype=torch.uint8, device="cuda", generator=gen)
        p2[at * 256:(at + n) * 256] = 0x5A
    B.repack_weights(p5, N, K, B.PACK_TRIT5, B.PACK_2BIT, out=p2)
    for at, n in spots:
        want = B.repack_weights(p5[at * 1024:(at + n) * 1024], 16 * n, K, B.PACK_TRIT5, B.PACK_2BIT)
        assert torch.equal(p2[at * 256:(at + n) * 256], want)
    del p5, p2
    torch.cuda.empty_cache()


@pytest.mark.parametrize("fmt", ["PACK_2BIT", "PACK_TRIT5"])
def test_unpack_of_more_weights_than_one_launch_has_threads(gpu_lib, fmt):
    """65552 x 65536 codes: more than 2^32 of them.  The weights are 0 and +-0.02, so their signs are the codes."""
    B, N, K = gpu_lib, 65552, 65536
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (40 << 30):
        pytest.skip("needs 40 GiB of GPU memory")
    sign = torch.randint(-1, 2, (N, K), dtype=torch.int8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
    W = sign.bfloat16().mul_(0.02)
    packed, _ = B.quantize_weights(W, getattr(B, fmt))
    del W
    codes = B.unpack_weights(packed, N, K, getattr(B, fmt), codes=torch.full((N, K), 9, dtype=torch.int8, device="cuda"))
    assert torch.equal(codes, sign)
    del sign, codes, packed
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kind", ["acts", "rmsnorm", "swiglu"])
def test_producers_on_more_tokens_than_one_launch_has_threads(gpu_lib, kind):
    """2^24 + 40 tokens, a workgroup of 256 threads each: more than 2^32 threads.  Against the same tokens in two calls."""
    B, M, K = gpu_lib, 2 ** 24 + 40, 48
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (40 << 30):
        pytest.skip("needs 40 GiB of GPU memory")
    call = {"acts": B.quantize_acts, "rmsnorm": B.rmsnorm_quantize, "swiglu": B.swiglu_quantize}[kind]
    x = torch.randn(M, K * (2 if kind == "swiglu" else 1), device="cuda", generator=torch.Generator(device="cuda").manual_seed(4)).bfloat16()
    q, s = torch.full((M, K), 5, dtype=torch.int8, device="cuda"), torch.full((M,), -1.0, device="cuda")
    call(x, **dict(zip(("hq", "sh") if kind == "swiglu" else ("xq", "sx"), (q, s))))
    half = M // 2 + 3
    for at, part in ((0, x[:half]), (half, x[half:])):
        q2, s2 = call(part)
        assert torch.equal(q[at:at + len(part)], q2) and torch.equal(s[at:at + len(part)], s2)
    del x, q, s, q2, s2
    torch.cuda.empty_cache()


def test_trit5_packing_of_more_chunks_than_one_launch_takes(gpu_lib):
    """A wave per 16 rows x 320 columns, 2^26 of them and more; every weight is +-0.02, so that any part of the matrix has its gamma."""
    B, K, N = gpu_lib, 1, 2 ** 30 + 40
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (90 << 30):
        pytest.skip("needs 90 GiB of GPU memory")
    gen = torch.Generator(device="cuda").manual_seed(3)
    W = torch.randint(0, 2, (N, K), dtype=torch.uint8, device="cuda", generator=gen).bfloat16().sub_(0.5).mul_(0.04)
    packed = torch.empty(B.packed_bytes(N, K, B.PACK_TRIT5), dtype=torch.uint8, device="cuda")
    blocks = -(-N // 16)
    spots = [(0, 40), (2 ** 25 - 20, 40), (2 ** 26 - 20, 20), (blocks - 7, 7)]          # row blocks: first, how many
    for at, n in spots:
        packed[at * 1024:(at + n) * 1024] = 0xFF
    _, gamma = B.quantize_weights(W, B.PACK_TRIT5, packed=packed)
    for at, n in spots:
        want, g = B.quantize_weights(W[16 * at:16 * (at + n)], B.PACK_TRIT5)
        assert torch.equal(g, gamma) and torch.equal(packed[at * 1024:(at + n) * 1024], want)
    del W, packed
    torch.cuda.empty_cache()
