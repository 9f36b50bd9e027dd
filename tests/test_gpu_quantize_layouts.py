"""The one-pass quantizer writes the canonical arrays and the kernels' private layout (run with -m gpu): both against the
separate steps, bit for bit."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("N,K,G", [(8, 8, 32), (33, 136, 64), (31, 72, 128), (96, 64, 32), (100, 520, 128), (64, 1032, 32), (40, 640, 64)])
def test_quantize_equals_canonical_codes_then_prepack(N, K, G, bits):
    # one row more or less than a fragment, K of less than a piece, of an odd number of k-tiles, with a short last group and
    # with k-tile padding that reaches into a group of its own
    import paper_2602_10431_amd as qt
    W = torch.randn(N, K, generator=torch.Generator().manual_seed(N + K)).cuda() * 0.05
    W[0, : min(K, G)] = 0.0
    got = qt.qtale_quantize(W, bits, G)
    want = qt.qtale_prepack(got.codes, got.scales, got.zeros, N, K, bits, G)
    torch.cuda.synchronize()
    assert torch.equal(got.prepacked, want.prepacked)
    # without the private layout: the same canonical arrays
    codes, scales, zeros = (torch.zeros_like(t) for t in (got.codes, got.scales, got.zeros))
    p = lambda t: C.c_void_p(t.data_ptr())
    assert qt.load_library().qtale_quantize(p(W), N, K, bits, G, p(codes), p(scales), p(zeros), None, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(codes, got.codes) and torch.equal(scales, got.scales) and torch.equal(zeros, got.zeros)
