"""The whole layer in one call (svdq_layer_forward) against the oracle, at the sizes where its kernels change or end:
token counts around the 32- and 64-token tiles, fewer groups than a block has waves, odd group counts, K split between
blocks in the quantise pass, and token counts on both sides of each change of kernel.

Codes are compared exactly.  y: the bar of the layer (workloads/harness.py) against the oracle's binary64 value: relative
Frobenius error <= 2e-3 (half a bf16 step at random is 1.1e-3) and per element 1e-2 rms or one bf16 step.
"""
import numpy as np
import pytest
import torch

from workloads import synth
from tests.helpers import dev, host_bits, rel_fro, unpack_act_e3m2_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def svdq():
    import paper_2605_27003_amd as m
    m.load_library(build_if_missing=False)
    assert torch.cuda.is_available()
    yield m
    from paper_2605_27003_amd import binding
    binding._staging.clear()                      # other tests look at the size of the shared staging buffer


SHAPES = [  # M, K, N, r, gelu
    (1, 64, 128, 16, False), (31, 192, 128, 0, False), (33, 576, 256, 32, False), (64, 1088, 128, 32, True),
    (65, 2112, 384, 16, False),                   # K split in the quantise pass, odd group count
    (1030, 1024, 640, 32, False),                 # 64 x 64 tiles (MXFP4: 32 x 64), ragged
    (4096, 64, 128, 16, False), (4097, 64, 128, 16, False),     # last of the 32 x 32 tiles and the next
    (15360, 64, 128, 0, False), (15361, 64, 128, 32, False),
    (8192, 64, 128, 16, False), (8193, 64, 128, 16, False),     # int4: last of the 64 x 64 tiles with few weights and the next
    (448, 2048, 4096, 32, False), (449, 2048, 4096, 16, False),   # and with many: canonical weights
    (160, 2112, 6144, 0, False), (161, 2112, 6144, 32, False), (170, 2112, 6272, 16, True),     # E3M2 fields: the last, the next, and more channels
    (150, 5120, 5120, 32, False), (130, 2112, 9728, 16, False),   # 64 x 64 tiles in all forms, ten and five steps a wave (MXFP4: the first)
    (16, 1408, 256, 32, False), (1000, 704, 256, 16, True),     # one launch: 16-token tiles, 32-token tiles
    (1916, 384, 4992, 32, False), (1300, 1088, 3072, 16, False), (206, 2112, 4992, 16, False),   # E3M2: one tile for every CU, K whole, in 2 and in 8
    (10240, 64, 128, 32, False), (10241, 64, 128, 16, False),   # MXFP4: last of the 32 x 64 tiles and the next
    (1025, 2112, 2048, 32, False),                # E3M2: K in halves, odd group count; MXFP4: 128 x 128 tiles
    (2049, 192, 4096, 16, True),
    (2049, 1088, 1408, 32, False),                # MXFP4: the last token in a launch of its own on the few-token kernel,
    (6401, 576, 2560, 16, True),                  # the others on 128 x 128 tiles or walked
    (2305, 3648, 640, 32, False),                 # MXFP4: six uneven slices of K, two blocks per CU in the quantise pass; E3M2: in 4
]


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble", "mxfp4"])
@pytest.mark.parametrize("M,K,N,r,gelu", SHAPES)
def test_layer_forward(svdq, oracle, container, M, K, N, r, gelu):
    mx = container == "mxfp4"
    x, _ = synth.make_x(M + K, M, K, outlier_count=3, outlier_scale=30.0)
    xa = oracle.gelu_tanh_bf16(x) if gelu else x
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(xa)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(M + K, K, N, r, cm, fmt="mxfp4" if mx else "int4")
    lin = svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1) if r else None, dev(L.L2) if r else None, dev(L.qw), dev(L.sw),
                          dev(L.bias), container=container.split()[0], resident="packed" if "packed" in container else "w4")
    rho = 0.8
    y = lin.forward(dev(x), rho, gelu=gelu)
    torch.cuda.synchronize()
    oq, os_ = (oracle.quantize_act_mxfp4 if mx else oracle.quantize_act)(xa, L.inv_lambda, rho)
    qx, sx = lin.buffers(M, y.device)[:2]
    if mx:
        gq, gs = svdq.mx_to_token_major(qx, sx, K)
        assert np.array_equal(gs.cpu().numpy(), os_)
    elif container == "nibble":                  # with many tokens too, where the GEMM takes E3M2 fields
        gq, gs = svdq.to_token_major(qx, sx)
        assert np.array_equal(gs.cpu().numpy().view(np.uint32), os_.view(np.uint32))
    else:
        codes, _ = unpack_act_e3m2_np(qx.buf.cpu().numpy(), M, K)
        assert np.array_equal(codes, synth.unpack_int4(oq))
        gq = None
    if gq is not None:
        assert np.array_equal(gq.cpu().numpy(), oq)
    oh = oracle.lowrank_down(xa, L.inv_lambda, L.L1) if r else None
    if r:                                        # the operands are whole (the bar of the quantise pass alone): gemm() on them gives the layer again
        assert rel_fro(lin.buffers(M, y.device)[2].double().cpu().numpy(), np.asarray(oh, np.float64)) <= 3e-5
    orc = (oracle.linear_mxfp4 if mx else oracle.linear)(oq, os_, L.qw, L.sw, oh, L.L2 if r else None, L.bias)
    got, want = synth.bf16_bits_to_f32(host_bits(y)).astype(np.float64), orc["y64"]
    assert rel_fro(got, want) <= 2e-3
    rms = float(np.sqrt(np.mean(want ** 2)))
    ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), 1e-30))) - 7)
    assert np.all(np.abs(got - want) <= np.maximum(1e-2 * rms, ulp))
    # the GEMM alone, from the separate quantise pass: the same kernels on one h instead of its slices
    y1 = y.clone()
    y2 = lin.gemm(*lin.quantize(dev(x), rho, gelu))
    torch.cuda.synchronize()
    assert rel_fro(synth.bf16_bits_to_f32(host_bits(y2)).astype(np.float64), synth.bf16_bits_to_f32(host_bits(y1)).astype(np.float64)) <= 2e-3


# M, K, N, r, gelu, ldx; tests/test_small_plan.py asks the plan whether they are one launch
ONE_LAUNCH = [
    (1, 64, 128, 32, False, 64), (1, 1792, 256, 16, True, 1792), (1, 3328, 128, 0, False, 3400),    # one token; fewer groups than waves, the longest K
    (2, 576, 128, 16, False, 584), (3, 1344, 384, 32, True, 1344), (5, 1600, 128, 0, False, 1600),  # odd group counts; a tile of 2, 4, 8
    (16, 1408, 256, 32, False, 1408), (17, 832, 128, 16, False, 840), (500, 576, 128, 0, True, 576),   # 16-token tiles: full, one over, ragged
    (33, 512, 128, 32, False, 512), (1000, 704, 256, 16, False, 704),             # 32-token tiles of 32 channels, ragged
    (1025, 1216, 384, 32, True, 1224), (1023, 448, 512, 0, False, 448),           # and of 64
]
# where MXFP4 goes further: the longest K of every kind, and 160 640 bytes of LDS (16 tokens)
ONE_LAUNCH_MX = [(9, 1792, 256, 32, False, 1792), (16, 1792, 256, 16, True, 1800), (8, 2304, 128, 32, False, 2304), (1, 4352, 128, 0, False, 4352),
                 (16, 3328, 128, 0, True, 3328), (40, 1664, 1024, 32, False, 1664)]


@pytest.mark.parametrize("container,M,K,N,r,gelu,ldx", [(c, *s) for s in ONE_LAUNCH for c in ("e3m2", "e3m2 packed", "nibble", "mxfp4")] +
                         [("mxfp4", *s) for s in ONE_LAUNCH_MX])
def test_layer_in_one_launch(svdq, container, M, K, N, r, gelu, ldx):
    """Few tokens and a short K: forward() is one kernel.  Codes and scales left behind are those of the quantise pass, bit for bit,
    h is its sum in another order at most (32-bit sums of K products: 1e-6), and y that of the GEMM on them (the bar of the layer)."""
    mx = container == "mxfp4"
    xs = torch.full((M, ldx), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    bits, _ = synth.make_x(M + K, M, K, outlier_count=3, outlier_scale=30.0)
    xs[:, :K] = dev(bits).view(torch.bfloat16)
    x = xs[:, :K]
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(bits)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(M + K, K, N, r, cm, fmt="mxfp4" if mx else "int4")
    lin = svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1) if r else None, dev(L.L2) if r else None, dev(L.qw), dev(L.sw),
                          dev(L.bias), container=container.split()[0], resident="packed" if "packed" in container else "w4")
    codes, scales, h, _ = lin.buffers(M, "cuda:0")
    buf = codes.buf if container.startswith("e3m2") else codes

    def held():                                   # rows M .. M + 3 of the E3M2 planes are nobody's
        if not container.startswith("e3m2"):
            return [buf.clone(), scales.view(torch.uint8).clone()]
        Mp = (M + 3) // 4 * 4
        planes, at = buf.view(K // 64, Mp * 56), [(0, 32)] + [(Mp * 32 + i * Mp * 8, 8) for i in range(3)]
        return [planes[:, o:o + M * w].clone() for o, w in at]

    buf.fill_(0xA5)
    y = lin.forward(x, 0.8, gelu=gelu).clone()
    one, h_one = held(), None if h is None else h.clone()
    two = lin.gemm(*lin.quantize(x, 0.8, gelu))
    assert all(torch.equal(a, b) for a, b in zip(one, held()))
    if r:
        assert rel_fro(h_one.double().cpu().numpy(), h.double().cpu().numpy()) <= 1e-6
    assert rel_fro(y.double().cpu().numpy(), two.double().cpu().numpy()) <= 2e-3
    assert torch.isfinite(y.float()).all()


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble", "mxfp4"])
@pytest.mark.parametrize("M,K,r", [(1, 1536, 32), (12, 1024, 16), (256, 512, 32), (256, 512, 0), (700, 512, 16), (300, 2048, 32)])
def test_layer_on_its_own_output(svdq, container, M, K, r):
    """forward(forward(x)) of a square layer: the buffer that the first call returns is the second one's x and y.  Codes and
    scales are bit for bit those of a copy of it, and y their product (the bar of the layer)."""
    mx = container == "mxfp4"
    bits, _ = synth.make_x(M + K, M, K, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(bits)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(M + K, K, K, r, cm, fmt="mxfp4" if mx else "int4")
    lin = svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1) if r else None, dev(L.L2) if r else None, dev(L.qw), dev(L.sw),
                          dev(L.bias), container=container.split()[0], resident="packed" if "packed" in container else "w4")
    x = dev(bits).view(torch.bfloat16)
    codes, scales, _, buf = lin.buffers(M, "cuda:0")
    fields = svdq.unpack_act_e3m2 if container.startswith("e3m2") else torch.clone
    once = lin.forward(x, 0.8).clone()
    want = lin.gemm(*lin.quantize(once, 0.8)).clone()
    want_codes, want_scales = fields(codes).clone(), None if scales is None else scales.clone()
    y = lin.forward(lin.forward(x, 0.8), 0.8)
    assert y.data_ptr() == buf.data_ptr()
    assert torch.equal(fields(codes), want_codes) and (scales is None or torch.equal(scales, want_scales))
    assert rel_fro(y.double().cpu().numpy(), want.double().cpu().numpy()) <= 2e-3


# M, K, N, r, slices of K in the quantise pass, two teams of waves (tests/test_e3m2_plan.py asks the plan)
SLICED = [
    (500, 5120, 5120, 32, 8, True), (513, 5120, 5120, 16, 8, True),   # two teams, eight slices; a last tile of one token
    (513, 2624, 3200, 32, 4, True),                                   # odd group count, four slices
    (2048, 2048, 2048, 16, 4, True), (2049, 2048, 2048, 16, 2, False),   # a tile on every CU, the last of two teams; one team, slices summed ahead
    (801, 1088, 2944, 32, 2, False),                                  # K < 2048: one team
]


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble"])
@pytest.mark.parametrize("M,K,N,r,slices,teams", SLICED)
def test_tiles_behind_a_sliced_quantise_pass(svdq, container, M, K, N, r, slices, teams):
    """More tokens than the few-token path takes: two teams' blocks sum the slices of h.  The h left behind is whole (the bar
    of the quantise pass alone), and the GEMM on it, the same kernel on one h, gives the same bits."""
    x, _ = synth.make_x(M + K, M, K, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(x)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(M + K, K, N, r, cm)
    lin = svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1), dev(L.L2), dev(L.qw), dev(L.sw), dev(L.bias),
                          container=container.split()[0], resident="packed" if "packed" in container else "w4")
    y = lin.forward(dev(x), 0.8).clone()
    work = lin._workspace(M, y.device, lin._descriptor(r))
    assert work.scratch.numel() == slices * M * r * 4
    qx, sx, h, _ = work.public
    want = (dev(x).view(torch.bfloat16).double() * dev(L.inv_lambda).double()) @ dev(L.L1).view(torch.bfloat16).double()
    assert rel_fro(h.double().cpu().numpy(), want.cpu().numpy()) <= 3e-5
    again = lin.gemm(qx, sx, h)
    if container != "nibble":
        assert torch.equal(again, y)
    else:                                                # its gemm() multiplies on other matrix cores
        assert rel_fro(again.double().cpu().numpy(), y.double().cpu().numpy()) <= 2e-3


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble"])
@pytest.mark.parametrize("M,K,N,r,walked", [
    (3300, 5120, 5120, 32, 3072),                       # slices of h summed ahead; the last 228 tokens by two teams
    (3300, 5120, 5120, 0, 3072),
    (1216, 2112, 13824, 32, 1024),                      # odd group count in both kernels
    (5376, 2112, 3072, 16, 5376),
])
def test_walked_layers(svdq, container, M, K, N, r, walked):
    """Layers whose first tokens take 256 x 256 tiles and whose last are left to two teams of the 128 x 128 kernel, which begins
    behind them (tests/test_e3m2_plan.py: they do).  Against that kernel with one team on the h that the layer has left:
    the same bits where tokens are walked, another order of K elsewhere (the bar of the layer)."""
    x, _ = synth.make_x(M + K, M, K, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(x)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(M + K, K, N, r, cm)
    inv = dev(L.inv_lambda)
    lin = svdq.W4A4Linear(inv, dev(L.L1) if r else None, dev(L.L2) if r else None, dev(L.qw), dev(L.sw), dev(L.bias),
                          container=container.split()[0], resident="packed" if "packed" in container else "w4")
    y = lin.forward(dev(x), 0.8)
    h = lin.buffers(M, y.device)[2] if r else None
    act = svdq.quantize_act_e3m2(dev(x), inv, 0.8, None, 0)[0]
    want = svdq.linear_w4a4_e3m2(act, svdq.pack_weight_e3m2(dev(L.qw), dev(L.sw)), N, h, dev(L.L2) if r else None, dev(L.bias),
                                 out_dtype=torch.float32).to(torch.bfloat16)
    assert torch.equal(y[:walked], want[:walked])
    if walked < M:
        assert rel_fro(y[walked:].double().cpu().numpy(), want[walked:].double().cpu().numpy()) <= 2e-3


# M, K, N, r and the entry of E3M2_MID that takes them (tests/test_e3m2_plan.py asks the plan)
MIDDLING = [
    (1500, 320, 6784, 16, 0), (1916, 384, 4992, 32, 0), (2047, 448, 5120, 0, 0),   # 256 x 192: K as long as the ring, whole channel tiles; one that stands over N
    (1300, 1088, 3072, 16, 1), (1916, 1088, 2176, 0, 1),     # 128 x 192, two teams of 9 and 8 groups
    (1025, 1600, 1280, 32, 2), (2305, 3648, 640, 32, 2),     # 128 x 96, four teams of 7, 6, 6, 6 and of 15, 14, 14, 14; a last tile of one token
    (1916, 1088, 768, 32, 3), (2100, 1216, 512, 0, 3),       # 64 x 96, eight teams, one and three of them with a group more
    (206, 2112, 4992, 16, 3),
]


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble"])
@pytest.mark.parametrize("M,K,N,r,shape", MIDDLING)
def test_layers_of_middling_tokens(svdq, container, M, K, N, r, shape):
    """One tile for every CU at most, K split between teams of waves: against the 128 x 128 kernel's binary32 output on the same
    codes (the bar of the layer); the h left behind is whole."""
    x, _ = synth.make_x(M + K, M, K, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(x)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(M + K, K, N, r, cm)
    bias = dev(L.bias) if r else None
    make = lambda c: svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1) if r else None, dev(L.L2) if r else None, dev(L.qw), dev(L.sw), bias,
                                     container=c.split()[0], resident="packed" if "packed" in c else "w4")
    lin, ref = make(container), make("e3m2 packed")
    y = lin.forward(dev(x), 0.8).clone()
    h = lin.buffers(M, y.device)[2]
    act, _, h_ref = ref.quantize(dev(x), 0.8)
    want = svdq.linear_w4a4_e3m2(act, ref.w_packed, N, h_ref, ref.L2, ref.bias, out_dtype=torch.float32).double()
    if r:
        assert rel_fro(h.double().cpu().numpy(), h_ref.double().cpu().numpy()) <= 1e-6
    d = (y.double() - want).abs()
    assert (d.norm() / want.norm()).item() <= 2e-3
    ulp = torch.exp2(torch.floor(torch.log2(want.abs().clamp_min(1e-30))) - 7)
    assert bool((d <= torch.maximum(1e-2 * want.pow(2).mean().sqrt(), ulp)).all())
    # rows of a wider tensor: the same bits, and nothing beside them
    from paper_2605_27003_amd import binding
    layer = lin._descriptor(r)
    work = lin._workspace(M, y.device, layer)
    staging = lin._staging(work, y.device)
    room = torch.full((M + 1, N + 8), 3.0, device="cuda", dtype=torch.bfloat16)
    xd = dev(x)
    assert binding.load_library().svdq_layer_forward(layer.address, xd.data_ptr(), K, 0.8, 0, M, *work.ptrs, binding._addr(staging),
                                                     room.data_ptr(), N + 8, binding._raw_stream()) == 0
    assert torch.equal(room[:M, :N], y) and (room[M] == 3.0).all() and (room[:, N:] == 3.0).all()


def test_layer_gemm_last_tokens_beyond_4_gb(svdq):
    """MXFP4, 4 GB of codes: the last tokens have a launch of their own on the few-token kernel where its 32-bit offsets
    reach them, and must not have one here.  Against the tile kernels alone (sums in another order: one bf16 step)."""
    M, K, N = 524389, 16384, 128
    g = torch.Generator(device="cuda").manual_seed(1)
    qw = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    sw = torch.randint(118, 123, (K // 32, N), generator=g, device="cuda", dtype=torch.uint8)
    lin = svdq.W4A4Linear(torch.ones(K, device="cuda"), None, None, qw, sw, None, container="mxfp4")
    qx, sx = lin.buffers(M, qw.device)[:2]
    qx.random_(0, 256, generator=g)
    sx.random_(118, 123, generator=g)
    y = lin.gemm(qx, sx, None)[-200:].float()
    want = svdq.linear_mxfp4(qx, sx, lin.w_packed, N)[-200:].float()
    assert torch.all((y - want).abs() <= want.abs() * 2.0 ** -7 + 1e-3 * want.std())


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble", "mxfp4"])
@pytest.mark.parametrize("M", [40, 15400])
def test_layer_gemm_beyond_quantise_limit(svdq, oracle, container, M):
    """The quantise pass ends at K = 16384; the GEMM takes more (the layer before may emit its operands)."""
    Kh, N = 8320, 128
    mx = container == "mxfp4"
    x, _ = synth.make_x(3, M, Kh, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(x)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(5, Kh, N, 0, cm, fmt="mxfp4" if mx else "int4")
    make = lambda qw, sw: svdq.W4A4Linear(dev(L.inv_lambda), None, None, qw, sw, dev(L.bias), container=container.split()[0],
                                          resident="packed" if "packed" in container else "w4")
    qw, sw = dev(L.qw), dev(L.sw)
    half, both = make(qw, sw), make(torch.cat([qw, qw], 1).contiguous(), torch.cat([sw, sw]).contiguous())
    qx, sx, _ = half.quantize(dev(x), 0.8)
    twice = lambda t: torch.cat([t, t]).contiguous()
    acts = (svdq.ActE3M2(twice(qx.buf), M, 2 * Kh), None) if "e3m2" in container else (twice(qx), twice(sx))
    y = both.gemm(*acts, None).float()
    once = half.gemm(qx, sx, None).float()
    want = 2.0 * once - half.bias                       # K taken twice: twice the sum, one bias
    tol = once.abs() * 2.0 ** -7 + want.abs() * 2.0 ** -7 + 1e-3 * want.std()      # a bf16 step of each output
    assert torch.all((y - want).abs() <= tol)


def test_layer_follows_its_tensors_and_copies(svdq):
    """Tensors replaced after construction are the ones used, and a copy has buffers of its own."""
    import copy
    x, _ = synth.make_x(3, 40, 512, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(x)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(5, 512, 128, 16, cm)
    lin = svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1), dev(L.L2), dev(L.qw), dev(L.sw), dev(L.bias))
    y = lin.forward(dev(x), np.float32(0.8)).clone()
    other = copy.deepcopy(lin)
    other.bias = other.bias + 64.0
    y2 = other.forward(dev(x), 0.8)
    assert y2.data_ptr() != lin.buffers(40, y.device)[3].data_ptr()
    assert torch.all((y2.float() - 64.0 - y.float()).abs() <= 0.5 + y.float().abs() * 2.0 ** -7)
    assert torch.equal(lin.forward(dev(x), 0.8), y)


@pytest.mark.parametrize("M", [40, 900])
def test_nibble_layer_keeps_its_form_and_no_staging(svdq, M):
    """The nibble container holds 4-bit activations and weights whatever its forward() multiplies: quantize()'s operands
    outlive a forward(), and what forward() expands into is given back (few tokens expand nothing)."""
    K, N = 1024, 2560
    x, _ = synth.make_x(3, M, K, outlier_count=3, outlier_scale=30.0)
    cm = np.maximum(np.abs(synth.bf16_bits_to_f32(x)).max(axis=0), 1e-3).astype(np.float32)
    L = synth.make_layer(5, K, N, 16, cm)
    lin = svdq.W4A4Linear(dev(L.inv_lambda), dev(L.L1), dev(L.L2), dev(L.qw), dev(L.sw), dev(L.bias), container="nibble")
    q = lin.quantize(dev(x), 0.8)
    codes, scales = q[0].clone(), q[1].clone()
    want = lin.gemm(*q).clone()
    before = torch.cuda.memory_allocated()
    y = lin.forward(dev(x), 0.8)
    assert torch.cuda.memory_allocated() - before <= 1024        # no more than the input's own rounding
    assert torch.equal(q[0], codes) and torch.equal(q[1], scales)
    assert rel_fro(y.double().cpu().numpy(), want.double().cpu().numpy()) <= 2e-3
    assert rel_fro(lin.gemm(*q).double().cpu().numpy(), want.double().cpu().numpy()) <= 2e-3     # h summed in another order


def _random_layer(svdq, container, K, N, r, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
    qw = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    sw = (torch.randint(118, 123, (K // 32, N), generator=g, device="cuda", dtype=torch.uint8) if container == "mxfp4"
          else rand(K // 64, N).abs() * 0.01 + 0.001)
    low = ((rand(K, r) * 0.02).bfloat16(), (rand(r, N) * 0.02).bfloat16()) if r else (None, None)
    return svdq.W4A4Linear(0.5 + rand(K).abs(), *low, qw, sw, rand(N), container=container.split()[0],
                           resident="packed" if "packed" in container else "w4")


# few tokens (one launch, 32 x 32, 64 x 64: in all forms, canonical weights only); two teams; one tile for every CU;
# tile kernels; MXFP4 with a launch for the last token
FORMS = [(40, 1088, 128, 16), (40, 2112, 640, 16), (150, 5120, 5120, 0), (420, 2112, 4096, 0), (1025, 2112, 2048, 32), (1300, 1088, 3072, 16),
         (2305, 2048, 6912, 32)]


@pytest.mark.parametrize("container", ["e3m2", "e3m2 packed", "nibble", "mxfp4"])
@pytest.mark.parametrize("M,K,N,r", FORMS)
def test_layer_forward_strides_ratios_and_non_finite_rows(svdq, container, M, K, N, r):
    """Rows of a wider tensor, clipping ratios at the ends of their range, and rows with infinities, NaN, zeros or values whose
    scales overflow: nothing reaches another row, and those rows are finite and not exactly where they are with the separate
    calls (the nibble container's multiplies nibbles, which overflows earlier: its finite rows only)."""
    lin = _random_layer(svdq, container, K, N, r)
    wide = torch.randn(M, K + 72, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda").bfloat16()
    x = wide[:, 8:K + 8]
    for rho in (1.0, 2.0 ** -20, 0.8):
        y = lin.forward(x.contiguous(), rho).clone()
        assert torch.equal(lin.forward(x, rho), y)
        if rho == 1.0:
            assert torch.isfinite(y).all()
    bad = x.clone()
    rows = [1, 5, 9, 13, M - 1]
    bad[1, 3], bad[5, K - 1], bad[9], bad[13, :64], bad[M - 1, 70] = float("inf"), float("nan"), 0, float("-inf"), 3e38
    good = torch.ones(M, dtype=torch.bool, device="cuda")
    good[rows] = False
    yb = lin.forward(bad, 0.8).clone()
    assert torch.equal(yb[good], y[good]) and torch.isfinite(yb[9]).all()
    q = lin.quantize(bad, 0.8)
    if container == "mxfp4":
        apart = svdq.linear_mxfp4(q[0], q[1], lin.weights(), N, q[2], lin.L2, lin.bias)
    elif container == "nibble":
        apart = svdq.linear_w4a4(q[0], q[1], lin.weights(), N, q[2], lin.L2, lin.bias)
    else:
        apart = svdq.linear_w4a4_e3m2(q[0], lin.weights(), N, q[2], lin.L2, lin.bias)
    if container == "nibble":
        assert torch.isfinite(yb)[torch.isfinite(apart)].all()
    else:
        assert torch.equal(torch.isfinite(yb), torch.isfinite(apart))


@pytest.mark.parametrize("M", [40, 900])
def test_nibble_layers_on_two_streams(svdq, M):
    """Layers of the nibble container are independent of each other: they share no buffer, whatever stream they run on."""
    K, N = 1024, 2560
    lins = [_random_layer(svdq, "nibble", K, N, 16, seed) for seed in (1, 2)]
    xs = [torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(s), device="cuda").bfloat16() for s in (3, 4)]
    want = [lin.forward(x, 0.8).clone() for lin, x in zip(lins, xs)]
    streams = [torch.cuda.Stream() for _ in lins]
    torch.cuda.synchronize()
    for _ in range(5):
        for lin, x, s in zip(lins, xs, streams):
            with torch.cuda.stream(s):
                lin.forward(x, 0.8)
    torch.cuda.synchronize()
    for lin, w in zip(lins, want):
        assert torch.equal(lin.buffers(M, w.device)[3], w)


def test_few_tokens_on_canonical_weights_on_two_streams(svdq):
    """Layers whose weights could be expanded in registers share no buffer either (300 tokens, 400 tiles of 64 x 64)."""
    M, K, N = 300, 5120, 5120
    lins = [_random_layer(svdq, "e3m2", K, N, 16, seed) for seed in (1, 2)]
    xs = [torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(s), device="cuda").bfloat16() for s in (3, 4)]
    want = [lin.forward(x, 0.8).clone() for lin, x in zip(lins, xs)]
    streams = [torch.cuda.Stream() for _ in lins]
    torch.cuda.synchronize()
    for _ in range(10):
        for lin, x, s in zip(lins, xs, streams):
            with torch.cuda.stream(s):
                lin.forward(x, 0.8)
    torch.cuda.synchronize()
    for lin, w in zip(lins, want):
        assert torch.equal(lin.buffers(M, w.device)[3], w)


@pytest.mark.parametrize("container", ["e3m2", "nibble"])
@pytest.mark.parametrize("M,K,N,r", [(161, 2112, 5504, 32), (300, 5120, 5120, 16), (448, 2048, 4096, 0)])
def test_layer_without_staging(svdq, container, M, K, N, r):
    """The C call takes NULL for the staging of a layer of few tokens: codes and scales of forward(), bit for bit, and the
    product on the few-token kernel (the bar of the layer)."""
    from paper_2605_27003_amd import binding
    lin = _random_layer(svdq, container, K, N, r)
    x = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").bfloat16()
    want = lin.forward(x, 0.8).clone()
    codes, scales, h, y = lin.buffers(M, "cuda:0")
    if container == "e3m2":
        codes, scales = codes.buf, None
        read = lambda: unpack_act_e3m2_np(codes.cpu().numpy(), M, K)      # rows up to M, of a buffer with whole tiles
    else:
        read = lambda: (codes.cpu().numpy(), scales.cpu().numpy())
    held = read()
    for t in (codes, y) + (() if scales is None else (scales,)):
        t.zero_()
    scratch = torch.empty(8 * M * max(r, 1) * 4, dtype=torch.uint8, device="cuda")
    layer = lin._descriptor(r)
    for part in (scratch, None):
        status = binding.load_library().svdq_layer_forward(layer.address, x.data_ptr(), K, 0.8, 0, M, codes.data_ptr(), binding._addr(scales), binding._addr(h),
                                                           binding._addr(part), None, y.data_ptr(), N, binding._raw_stream())
        assert status == 0
        assert all(np.array_equal(a, b) for a, b in zip(read(), held))
        assert rel_fro(y.double().cpu().numpy(), want.double().cpu().numpy()) <= 2e-3


@pytest.mark.parametrize("container", ["e3m2", "nibble", "mxfp4"])
@pytest.mark.parametrize("M", [40, 900])
def test_layer_forward_captured(svdq, container, M):
    """A captured forward() keeps the memory that its operands are expanded into: every replay gives the eager result, with
    eager calls of the layer and of others in between."""
    K, N = 1024, 2560
    lin, other = _random_layer(svdq, container, K, N, 16), _random_layer(svdq, container, K, N, 16, seed=2)
    x = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").bfloat16()
    xs = [x * s for s in (1.0, -0.5, 2.0, 3.0)]
    want = [lin.forward(v, 0.8).clone() for v in xs]
    held = x.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        lin.forward(held, 0.8)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = lin.forward(held, 0.8)
    for v, w in zip(xs, want):
        held.copy_(v)
        other.forward(v, 0.8)
        lin.forward(xs[0], 0.9)
        junk = torch.full((1 << 24,), 7, dtype=torch.uint8, device="cuda")
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, w)
        del junk


def test_mxfp4_forward_takes_raw_bits(svdq):
    """bf16 bits held in 16-bit integers, as the MXFP4 quantise pass takes them; the other containers refuse them."""
    x = torch.randn(40, 1024, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda").bfloat16()
    lin = _random_layer(svdq, "mxfp4", 1024, 256, 16)
    y = lin.forward(x, 0.8).clone()
    assert torch.equal(lin.forward(x.view(torch.int16), 0.8), y)
    for bad in (lambda: lin.forward(x.float(), 0.8), lambda: _random_layer(svdq, "e3m2", 1024, 256, 16).forward(x.view(torch.int16), 0.8)):
        with pytest.raises(AssertionError):
            bad()
