"""GPU parity of the linears at 65 to 256 rows, and at 9 to 16 rows of very wide outputs (run with -m gpu): the 128-row x
128-column K-sliced kernel in its three epilogues, and the shapes next to it that stay on the other kernels.  References and tolerances as in the other GPU tests."""
import pytest
import torch

import synth_inputs as si
from oracle import qtale_oracle as orc
from tests.helpers import check_parity, to_f64
from tests.test_gpu_layer import _check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import paper_2602_10431_amd as pkg
    pkg.load_library()
    return pkg


# One and two row chunks with 2, 3 and 4 live 32-row fragments, rows at their edges; a width that fills the chip with one
# chunk, one that does with two, one too wide, one too narrow, last column blocks of one fragment of 8 columns; K of less than
# a round of four k-tiles, of every remainder of the three-slot ring, and not a multiple of 64.
@pytest.mark.parametrize("M", [65, 96, 97, 128, 129, 150, 192, 193, 256])
@pytest.mark.parametrize("N,K,G,bits", [(20488, 136, 128, 4), (10248, 64, 32, 3), (10248, 1096, 64, 2), (33000, 72, 64, 4), (6152, 1480, 128, 4),
                                        (3080, 776, 32, 4)])
def test_linear_of_a_hundred_rows(qt, M, N, K, G, bits):
    g = torch.Generator().manual_seed(M + N + K)
    W = torch.randn(N, K, generator=g) * 0.05
    A = torch.randn(M, K, generator=g).to(torch.float16)
    out = qt.qtale_linear_w4a16(qt.qtale_quantize(W.cuda(), bits, G), A.cuda())
    torch.cuda.synchronize()
    want = to_f64(A) @ orc.dequantize(*orc.quantize_rtn(W.numpy(), bits, G), G).T
    check_parity(orc.parity_error(to_f64(out), want), "fp16", ("linear", M, N, K))


@pytest.mark.parametrize("M", [66, 97, 128, 150, 192, 200])
@pytest.mark.parametrize("I,K,G,bits", [(8200, 520, 128, 4), (16392, 72, 64, 2), (4104, 328, 32, 3)])
def test_swiglu_of_a_hundred_rows(qt, M, I, K, G, bits):
    g = torch.Generator().manual_seed(M + I + K)
    Wg, Wu = torch.randn(I, K, generator=g) * 0.05, torch.randn(I, K, generator=g) * 0.05
    A = torch.randn(M, K, generator=g).to(torch.float16)
    out = qt.qtale_swiglu_w4a16(qt.qtale_quantize(Wg.cuda(), bits, G), qt.qtale_quantize(Wu.cuda(), bits, G), A.cuda())
    torch.cuda.synchronize()
    d = [orc.dequantize(*orc.quantize_rtn(W.numpy(), bits, G), G).T for W in (Wg, Wu)]
    want = orc.silu(to_f64(A) @ d[0]) * (to_f64(A) @ d[1])
    check_parity(orc.parity_error(to_f64(out), want), "fp16", ("swiglu", M, I, K))


# Each arm of the rules: narrow and very narrow outputs whose 64-row chunks run at once (one fragment per workgroup; two, with
# K of 64 k-tiles), just past one round, and above 192 rows.
@pytest.mark.parametrize("M,N,K,G,bits", [(129, 8, 136, 128, 4), (256, 1032, 328, 32, 3), (192, 2728, 72, 64, 4), (193, 2056, 520, 64, 2),
                                          (97, 8192, 4104, 128, 4), (129, 8192, 4104, 128, 4)])
def test_narrow_linear_of_a_hundred_rows(qt, M, N, K, G, bits):
    test_linear_of_a_hundred_rows(qt, M, N, K, G, bits)


# gate/up: two workgroups per CU of 64-row chunks (up to 512, and one more), one round of wide workgroups above 192 rows with K of
# 32 k-tiles and with less, a second round with little K (64-row chunks, 64-row tiles), more than a round at 65 to 96 rows
@pytest.mark.parametrize("M,I,K,G,bits", [(256, 4096, 72, 32, 4), (256, 4104, 72, 64, 3), (200, 4104, 2056, 128, 4), (256, 8192, 2056, 64, 2),
                                          (65, 8192, 520, 128, 4), (129, 11008, 136, 128, 4), (192, 12296, 72, 64, 4), (150, 12296, 1096, 32, 4),
                                          (96, 16392, 4104, 128, 4)])
def test_swiglu_of_a_hundred_rows_in_each_arm(qt, M, I, K, G, bits):
    test_swiglu_of_a_hundred_rows(qt, M, I, K, G, bits)


# 9 to 16 rows: widths whose 16-column groups overflow one round of workgroups a little go to the kernel of 17 to 64 rows
@pytest.mark.parametrize("M,N,K", [(8, 20488, 136), (9, 20488, 136), (16, 24576, 72), (16, 24584, 72)])
def test_few_row_linear_past_one_round(qt, M, N, K):
    test_linear_of_a_hundred_rows(qt, M, N, K, 64, 4)


@pytest.mark.parametrize("M,K,G,bits", [(14, 5064, 128, 4), (15, 5064, 128, 4), (16, 5064, 128, 4), (8, 5064, 32, 4), (9, 5064, 32, 3),
                                        (13, 5064, 32, 2), (11, 3080, 32, 4), (14, 3080, 32, 3)])
def test_few_row_swiglu_past_one_round(qt, M, K, G, bits):
    test_swiglu_of_a_hundred_rows(qt, M, 12304, K, G, bits)


@pytest.mark.parametrize("M,bits", [(2, 4), (3, 4), (5, 3), (6, 3), (9, 2)])
def test_few_row_linear_past_one_round_with_small_groups(qt, M, bits):
    test_linear_of_a_hundred_rows(qt, M, 20488, 5064, 32, bits)


def test_fused_call_of_a_width_past_one_round(qt):
    # three tokens, 20480 columns of q|k|v, groups of 32: the launch that selects and normalises stays on the few-row kernel
    _check_layer(qt, si.LayerShape(5120, 160, 80, 64, 64, 4, 32, "bf16"), 3, [2, 1], "ratio", 1.0, seed=77)


# hidden 2568: 21 column blocks, two row chunks, the o- and down-proj leave K parts (27 k-tiles with a ragged last one)
SHAPE = si.LayerShape(2568, 24, 24, 64, 1672, 4, 64, "bf16")


@pytest.mark.parametrize("T,mode,val", [(150, "ratio", 1.0), (230, "threshold", 0.5), (300, "ratio", 0.5)])
def test_layer_with_k_parts_in_two_row_chunks(qt, T, mode, val):
    _check_layer(qt, SHAPE, T, [T // 2, 0, T - T // 2], mode, val, seed=T)


def test_stack_with_k_parts_equals_layer_by_layer_calls(qt):
    T, L = 140, 2
    layers = [qt.quantize_layer(si.layer_tensors(SHAPE, l, 3, unit_gains=False), 4, 64) for l in range(L)]
    cfg, ctx = qt.cfg_from_shape(SHAPE), qt.Context()
    qt.qtale_set_exec_ratio(ctx, 0.96)
    x0 = si.hidden_states(SHAPE, T, 3).cuda()
    offs, pos = (t.cuda() for t in si.ragged_sequences([100, 40]))
    xs, xl = x0.clone(), x0.clone()
    zs, zl = torch.zeros(L, T, device="cuda"), torch.zeros(L, T, device="cuda")
    qt.qtale_stack_forward(ctx, qt.Stack(cfg, layers), xs, offs, pos, scores=zs)
    for l in range(L):
        qt.qtale_layer_forward(ctx, cfg, layers[l], xl, offs, pos, scores=zl[l])
    torch.cuda.synchronize()
    assert torch.equal(xs, xl) and torch.equal(zs, zl)


# three to six row chunks; the parts' buffer of the first shape (1.6 M floats) holds two parts up to 315 rows and none beyond, the
# narrow one takes four parts at 513 rows, two at 768 and the ordinary path at 769; at 801 rows of the first shape the 128-row
# kernel saves a round for q|k|v (K of 41 k-tiles; the down-proj's 27 are too few), and with a longer down-proj for that one too,
# with one part (the o-proj has no room for one)
LONG_DOWN = si.LayerShape(2568, 24, 24, 64, 2056, 4, 64, "bf16")
NARROW = si.LayerShape(1032, 32, 8, 64, 1096, 4, 128, "fp16")


@pytest.mark.parametrize("shape,T,mode,val", [(SHAPE, 257, "ratio", 1.0), (SHAPE, 315, "ratio", 1.0), (SHAPE, 316, "ratio", 1.0),
                                              (SHAPE, 310, "threshold", 0.5), (NARROW, 513, "ratio", 1.0),
                                              (NARROW, 768, "threshold", 0.5), (NARROW, 769, "ratio", 1.0),
                                              (SHAPE, 801, "ratio", 1.0), (SHAPE, 801, "threshold", 0.5),
                                              (LONG_DOWN, 801, "ratio", 1.0), (LONG_DOWN, 801, "threshold", 0.3)])
def test_layer_with_k_parts_in_more_row_chunks(qt, shape, T, mode, val):
    _check_layer(qt, shape, T, [T // 3, 0, T - T // 3], mode, val, seed=T)


# the 128-row kernel fills one round where the 64-row kernel needs two: from the first row count above 256 to a full round of
# 256 workgroups, and 261, which go elsewhere, as do K of less than 32 k-tiles
@pytest.mark.parametrize("M,N,bits,G", [(257, 8200, 4, 128), (385, 6152, 3, 32), (1000, 4096, 2, 64), (1025, 3592, 4, 64)])
@pytest.mark.parametrize("K", [328, 2008])
def test_linear_that_fills_one_round_of_128_row_workgroups(qt, M, N, bits, G, K):
    test_linear_of_a_hundred_rows(qt, M, N, K, G, bits)


# two k-slices (two workgroups per CU): gate/up in two chunks with K of 64 k-tiles and more (odd numbers of rounds, every
# remainder of the ring, a ragged last k-tile), in three chunks with a short K (of 16 k-tiles above 320 rows), with a width whose
# full chunks run at once and one whose large tiles take a second round, and outputs whose large tiles are a few more than the CUs;
# 1 to 4 live row fragments in the last chunk.  (200 k-columns at 352 rows and 353 rows are the large tiles'.)
@pytest.mark.parametrize("M,I,K,G,bits", [(129, 8328, 4096, 128, 4), (160, 8328, 4104, 64, 3), (193, 8328, 4168, 32, 2), (256, 8328, 4352, 128, 4),
                                          (150, 8328, 4296, 32, 4), (257, 13192, 72, 64, 4), (320, 13192, 136, 128, 2), (352, 13192, 200, 32, 3),
                                          (353, 13192, 136, 64, 4), (352, 13192, 1032, 32, 3), (321, 16376, 1000, 64, 4), (257, 21896, 72, 32, 2),
                                          (352, 21896, 136, 128, 4), (385, 9352, 264, 128, 4), (420, 9352, 72, 32, 4), (448, 9352, 200, 64, 3)])
def test_swiglu_on_two_slices(qt, M, I, K, G, bits):
    test_swiglu_of_a_hundred_rows(qt, M, I, K, G, bits)


# up to 160 rows on both sides of 160 columns of workgroups, where two k-slices begin (161 rows: below it too)
@pytest.mark.parametrize("M,I,K,G,bits", [(129, 10240, 4096, 128, 4), (129, 10248, 4096, 128, 4), (160, 10240, 4104, 32, 3), (160, 10248, 4104, 32, 3),
                                          (150, 10312, 4296, 32, 4), (145, 10312, 4168, 64, 2), (161, 8328, 4104, 32, 3)])
def test_swiglu_where_two_slices_begin(qt, M, I, K, G, bits):
    test_swiglu_of_a_hundred_rows(qt, M, I, K, G, bits)


# (the second of each pair of widths is one column block too wide, the last row count has a last chunk of more than half)
@pytest.mark.parametrize("M,N,K,G,bits", [(1300, 6136, 136, 128, 4), (1300, 6152, 136, 128, 4), (1313, 6136, 72, 32, 3), (1313, 6152, 72, 32, 3),
                                          (700, 12280, 328, 64, 4), (700, 12296, 328, 64, 4), (704, 12280, 136, 32, 2), (705, 12296, 136, 32, 2)])
def test_linear_on_two_slices(qt, M, N, K, G, bits):
    test_linear_of_a_hundred_rows(qt, M, N, K, G, bits)
