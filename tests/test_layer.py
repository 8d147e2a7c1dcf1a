"""The layer's host side (no GPU): what it hands to the library follows the tensors that it holds."""
import copy
import pickle

import pytest
import torch

import paper_2605_27003_amd as svdq
from paper_2605_27003_amd import binding


def test_descriptor_follows_the_layer():
    qw, sw = torch.zeros((128, 32), dtype=torch.uint8), torch.ones((1, 128))
    lin = svdq.W4A4Linear(torch.ones(64), None, None, qw, sw, torch.zeros(128))
    lin._descriptor(0)
    for other in (copy.copy(lin), copy.deepcopy(lin), pickle.loads(pickle.dumps(lin))):
        other.bias = torch.ones(128)
        other._descriptor(0)
        assert other._layer.bias == other.bias.data_ptr() and other._layer.qw == other.qw.data_ptr()
    lin.bias = None
    lin._descriptor(16)
    assert lin._layer.bias is None and lin._layer.r == 16


def _layer(K=1024, N=128, **kw):
    return svdq.W4A4Linear(torch.ones(K), None, None, torch.zeros((N, K // 2), dtype=torch.uint8), torch.ones((K // 64, N)),
                           torch.zeros(N), **kw)


def test_buffers_follow_what_their_sizes_depend_on():
    """A low-rank pair of another rank, or another form of the weights, between two calls with the same token count: h,
    the partial h's and the staging buffer are written by the kernels for the layer as it is, so they have its sizes."""
    lin, M, sizes = _layer(), 40, []
    for r in (16, 32, 0, 32):
        lin.r = r
        lin.l1_packed = torch.zeros(svdq.packed_l1_bytes(lin.K), dtype=torch.uint8) if r else None
        lin.L2 = torch.zeros((r, lin.N), dtype=torch.bfloat16) if r else None
        h = lin.buffers(M, "cpu")[2]
        assert h is None if r == 0 else h.shape == (M, r)
        sizes.append((r, lin._work.scratch))
    for r, scratch in sizes:
        need = binding.load_library().svdq_layer_scratch_bytes(binding.ctypes.byref(lin._descriptor(r)), M)
        assert (need > 0) == (r > 0) and (scratch is not None or not need) and (not need or scratch.numel() >= need)
    assert lin.buffers(M, "cpu")[3] is lin.buffers(M, torch.device("cpu"))[3]
    assert lin.buffers(M, "meta")[3].device.type == "meta" and lin.buffers(M, "cpu")[3].device.type == "cpu"
    lin = _layer(K=4096, N=2048)
    lin.w_packed = torch.zeros(svdq.packed_weight_e3m2_bytes(lin.N, lin.K), dtype=torch.uint8)
    lin.buffers(4096, "cpu")
    assert not lin._work.shared
    lin.w_packed = None
    lin.buffers(4096, "cpu")
    assert lin._work.shared
    binding._staging.clear()


def test_a_call_keeps_its_own_buffers(monkeypatch):
    """Another thread that runs the layer with another token count, or replaces a tensor, between this call's steps: the
    library gets this call's buffers and descriptor all the same."""
    lin, M, seen = _layer(), 512, []

    class Lib:
        def __getattr__(self, name):
            return getattr(real, name)

        def svdq_layer_forward(self, layer, x, ldx, rho, gelu, m, codes, *rest):
            seen.append((m, codes, binding._Layer.from_address(layer).bias))
            return 0

    real = binding.load_library()
    monkeypatch.setattr(binding, "_lib", Lib())
    monkeypatch.setattr(binding, "_raw_stream", lambda: 0)
    mine, bias = lin.buffers(M, "cpu")[0].buf, lin.bias
    other = binding.W4A4Linear(lin.inv_lambda, None, None, lin.qw, lin.sw, None)
    other.buffers(1, "cpu")
    workspace = binding.W4A4Linear._workspace

    def then_other_thread(self, *args):
        got = workspace(self, *args)
        self._work, self._layer = other._work, other._layer
        return got

    monkeypatch.setattr(binding.W4A4Linear, "_workspace", then_other_thread)
    y = lin.forward(torch.zeros((M, lin.K), dtype=torch.bfloat16), 0.8)
    assert seen == [(M, mine.data_ptr(), bias.data_ptr())] and y.shape == (M, lin.N)
    binding._staging.clear()


def test_layers_saved_by_earlier_versions():
    """The state that pickles of layers held before the whole-layer call (no format code, qw and sw with resident 4-bit
    weights only, buffers included): such a layer still runs."""
    for container in ("e3m2", "nibble", "mxfp4"):
        now = _layer()
        state = dict(container=container, N=now.N, K=now.K, r=0, inv_lambda=now.inv_lambda, l1_packed=None, L2=None,
                     w_packed=None, bias=now.bias, _bufs=tuple(torch.zeros((40, 1)) for _ in range(4)))
        if container == "e3m2":
            state.update(qw=now.qw, sw=now.sw)
        else:
            state["w_packed"] = torch.zeros(1 << 18, dtype=torch.uint8)
        old = svdq.W4A4Linear.__new__(svdq.W4A4Linear)
        copy_of = getattr(old, "__setstate__", old.__dict__.update)
        copy_of(state)
        assert old._descriptor(0).format == {"e3m2": 1, "nibble": 0, "mxfp4": 2}[container]
        assert old.buffers(40, "cpu")[3].shape == (40, now.N)
    binding._staging.clear()


def test_stream_without_torchs_private_functions(monkeypatch):
    """The current stream is found through torch's public interface where the private one has gone."""
    class Stream:
        cuda_stream = 1234

    monkeypatch.setattr(torch, "_C", object())
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    assert binding._raw_stream() == 1234


@pytest.mark.parametrize("M,K,N", [(161, 2112, 5504), (175, 4672, 5632), (320, 5120, 5120), (384, 2048, 4096), (480, 2048, 4096), (481, 2048, 4096),
                                   (384, 1984, 4096), (384, 2048, 3968)])
def test_few_tokens_on_weights_to_expand(M, K, N):
    """Up to 480 tiles of 64 x 64, N >= 4096 and K >= 2048 the weights can also be expanded in registers: the C functions take NULL for the
    staging, and W4A4Linear, whose layers may run on several streams there, takes it for each call."""
    lib, can = binding.load_library(), -(-M // 64) * (-(-N // 64)) <= 480 and N >= 4096 and K >= 2048
    for container, packed in (("e3m2", False), ("nibble", True), ("e3m2", True)):
        held = (256, None, None) if packed else (None, 256, 256)
        layer = binding._Layer(binding._FORMATS[container], N, K, 0, 256, None, None, None, *held)
        ref = binding.ctypes.byref(layer)
        assert (lib.svdq_layer_staging_bytes(ref, M) > 0) == (container == "nibble" or not packed)
        call = lambda staging: lib.svdq_layer_forward(ref, 256, K, 0.8, 0, M, 256, 256, None, None, staging, 256 << 30, N, None)
        if not torch.cuda.is_available():            # refused for their arguments, or for want of a GPU
            none = lib.svdq_layer_forward(ref, None, K, 0.8, 0, M, 256, 256, None, None, None, 256, N, None)
            assert (call(None) == none) == (not can and (container, packed) != ("e3m2", True)) and call(256) != none
            product = lib.svdq_layer_gemm(ref, 256, 256, None, M, None, 256, N, None)
            assert (product == none) == (not can and not packed)
    lin = _layer(K=K, N=N)
    lin.buffers(M, "cpu")
    assert lin._work.staging and lin._work.shared == (not can)
    binding._staging.clear()
