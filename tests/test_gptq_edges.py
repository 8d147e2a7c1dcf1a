"""GPTQ kernels at their edges: a channel count that is odd (rows of W are then not 16-byte aligned), pivots whose
quotients leave the exponent range of the fast division, and the Hessian with unaligned rows, a token count that is no
multiple of its four-token step, and both of its tile sizes."""
import numpy as np
import pytest
import torch

from workloads import synth
from tests.helpers import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def svdq():
    import paper_2605_27003_amd as m
    m.load_library(build_if_missing=False)
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("K,N,scale", [(192, 67, 1.0), (64, 1, 1.0), (256, 96, 2.0 ** -720), (128, 64, 2.0 ** 720),
                                       (320, 130, 1.0), (384, 67, 2.0 ** 720)])   # panels go in pairs: 3, 1, 4, 2, 5, 6
def test_gptq_bit_exact_at_the_edges(svdq, oracle, K, N, scale):
    """Codes and scales are those of the definition (binary64, oracle) whatever the scale of H: scaling H scales H^-1
    exactly, by a power of two, but takes the quotients by its diagonal out of the range of the fast division."""
    g = np.random.default_rng(K + N)
    z = np.round(8 * (g.standard_normal((2 * K, K)) + np.repeat(g.standard_normal((2 * K, K // 8)), 8, axis=1)))
    H = (z.T @ z) * scale
    R = (g.standard_normal((K, N)) * 0.02).astype(np.float32)
    qw, sw = svdq.gptq_quantize(dev(R), torch.from_numpy(H).cuda())
    torch.cuda.synchronize()
    oq, os_ = oracle.gptq_quantize(R, H)
    assert np.array_equal(sw.cpu().numpy().view(np.uint32), os_.view(np.uint32))
    assert np.array_equal(qw.cpu().numpy(), oq)


@pytest.mark.parametrize("K,N", [(128, 37), (192, 80)])
def test_gptq_scales_of_every_size(svdq, oracle, K, N):
    """Channels beside each other whose weights are ordinary, all zero, on the halfway points of the grid, so small or so
    large that the fast quotient by the scale does not take them, and zero in one group only: bit for bit the oracle's."""
    g = np.random.default_rng(K)
    z = np.round(8 * (g.standard_normal((2 * K, K)) + np.repeat(g.standard_normal((2 * K, K // 8)), 8, axis=1)))
    R = (g.standard_normal((K, N)) * 0.02).astype(np.float32)
    R *= np.array([1, 2.0 ** -40, 2.0 ** -58, 2.0 ** -66, 2.0 ** -120, 2.0 ** -141, 2.0 ** 54, 2.0 ** 70, 2.0 ** 120, 0, 1], np.float32)[np.arange(N) % 11]
    R[:, 10::11] = np.float32(0.25) * g.integers(-14, 15, R[:, 10::11].shape)
    R[0::64, 10::11] = 3.5
    R[64:128, 1::3] = 0
    qw, sw = svdq.gptq_quantize(dev(R), torch.from_numpy(z.T @ z).cuda())
    torch.cuda.synchronize()
    oq, os_ = oracle.gptq_quantize(R, z.T @ z)
    assert np.array_equal(sw.cpu().numpy().view(np.uint32), os_.view(np.uint32))
    assert np.array_equal(qw.cpu().numpy(), oq)


@pytest.mark.parametrize("M,K,ld", [(1, 64, 64), (37, 192, 192), (130, 256, 257), (41, 2048, 2048), (19, 2048, 2051)])
def test_hessian_edges(svdq, oracle, M, K, ld):
    """Against the oracle's binary64 product; sums of M terms in another order: M 2^-53 relative to the diagonal's size."""
    x, _ = synth.make_x(3 + M, M, ld, outlier_count=3, outlier_scale=30.0)
    il = (np.random.default_rng(K).random(K).astype(np.float32) + 0.5)
    Hg = svdq.gptq_hessian(dev(x)[:, :K], dev(il))
    torch.cuda.synchronize()
    H = oracle.gptq_hessian(np.ascontiguousarray(x[:, :K]), il)
    d = np.sqrt(np.diag(H))
    assert np.all(np.abs(Hg.cpu().numpy() - H) <= (M + 2) * 2.0 ** -52 * np.outer(d, d))


def panels_hessian(seed, panels, classes):
    """A Hessian that couples panel p (64 channels) with the panels p + i classes only: GPTQ then visits each class for
    itself, and every other update subtracts zero."""
    g = np.random.default_rng(seed)
    K = 64 * panels
    cls = (np.arange(K) // 64) % classes
    H = np.zeros((K, K))
    for c in range(classes):
        i = np.flatnonzero(cls == c)
        z = np.round(8 * (g.standard_normal((2 * len(i), len(i))) + np.repeat(g.standard_normal((2 * len(i), len(i) // 8)), 8, axis=1)))
        H[np.ix_(i, i)] = z.T @ z
    return H, cls


@pytest.mark.parametrize("panels,N,classes,channels", [
    (7, 65, 1, None), (8, 64, 1, None), (9, 258, 1, None), (12, 31, 1, None), (13, 130, 1, None),   # the last batch of four: 3, 4, 1, 4, 1
    (49, 30011, 7, 40)])                                  # more blocks of the rest than fit one round, in every stage
def test_gptq_batches_of_panels(svdq, oracle, panels, N, classes, channels):
    """Bit for bit the oracle's, whatever share of a batch of four panels the last one is, and where the batch's updates
    take several rounds of blocks.  Channels are independent, and classes of panels that H does not couple too (the damping
    term, relative to the mean of the diagonal, is added here): the large case is checked on some channels, by class."""
    H, cls = panels_hessian(panels, panels, classes)
    H[np.diag_indices_from(H)] += 0.01 * H.diagonal().mean()
    g = np.random.default_rng(N)
    R = (g.standard_normal((64 * panels, N), dtype=np.float32) * np.float32(0.02))
    qw, sw = svdq.gptq_quantize(dev(R), torch.from_numpy(H).cuda(), damp=0.0)
    torch.cuda.synchronize()
    n = np.arange(N) if channels is None else np.unique(np.concatenate([[0, N - 1], g.integers(0, N, channels)]))
    qw, sw = qw.cpu().numpy()[n], sw.cpu().numpy()[:, n]
    for c in range(classes):
        k = np.flatnonzero(cls == c)
        oq, os_ = oracle.gptq_quantize(np.ascontiguousarray(R[np.ix_(k, n)]), np.ascontiguousarray(H[np.ix_(k, k)]), damp=0.0)
        assert np.array_equal(sw[k[::64] // 64].view(np.uint32), os_.view(np.uint32))
        assert np.array_equal(qw[:, k[::2] // 2], oq)


@pytest.mark.parametrize("panels,N,classes", [(56, 70, 7), (76, 33, 19), (97, 40, 13)])
def test_gptq_batches_of_two_and_four(svdq, oracle, panels, N, classes):
    """The sizes at which a batch of the inverse is two panels and four (three in the cases above), and the visit's four too."""
    test_gptq_batches_of_panels(svdq, oracle, panels, N, classes, None)
