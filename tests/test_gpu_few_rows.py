"""GPU parity of the few-row paths (run with -m gpu): the 16-column-fragment GEMM (at most 16 rows), the calls of at most
four tokens whose q|k|v and gate/up launches also select and normalise, and the decode attention kernel that rotates,
appends and combines its key ranges by itself.  References and tolerances are those of the other GPU tests."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import qtale_oracle as orc
from tests.helpers import cfg_dict, check_parity, oracle_layer, to_f64
from tests.test_gpu_layer import _cache_case, _check_layer, _run_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import paper_2602_10431_amd as pkg
    pkg.load_library()
    return pkg


# Output widths in each of the workgroup shapes (16-column fragments: up to 256, 512, 768, more) with a last fragment of 8
# columns; K of one k-tile, an odd number of k-tiles, and not a multiple of 64; rows at the edges of the staged 4 / 8 / 16
# and just past the kernel's range.
@pytest.mark.parametrize("M", [1, 4, 5, 8, 9, 16, 17])
@pytest.mark.parametrize("N,K,G,bits", [(8, 64, 64, 4), (40, 1096, 128, 4), (4104, 72, 32, 3), (8200, 192, 64, 2), (12296, 136, 128, 4),
                                        (4088, 320, 32, 4)])
def test_few_row_linear(qt, M, N, K, G, bits):
    g = torch.Generator().manual_seed(M + N + K)
    W = torch.randn(N, K, generator=g) * 0.05
    A = torch.randn(M, K, generator=g).to(torch.float16)
    out = qt.qtale_linear_w4a16(qt.qtale_quantize(W.cuda(), bits, G), A.cuda())
    torch.cuda.synchronize()
    want = to_f64(A) @ orc.dequantize(*orc.quantize_rtn(W.numpy(), bits, G), G).T
    check_parity(orc.parity_error(to_f64(out), want), "fp16", ("few-row linear", M, N, K))


@pytest.mark.parametrize("M", [1, 8, 16])
@pytest.mark.parametrize("I,K,G,bits", [(24, 136, 64, 4), (4104, 64, 32, 2), (8200, 72, 64, 3), (12296, 64, 64, 4)])
def test_few_row_swiglu(qt, M, I, K, G, bits):
    g = torch.Generator().manual_seed(M + I + K)
    Wg, Wu = torch.randn(I, K, generator=g) * 0.05, torch.randn(I, K, generator=g) * 0.05
    A = torch.randn(M, K, generator=g).to(torch.float16)
    out = qt.qtale_swiglu_w4a16(qt.qtale_quantize(Wg.cuda(), bits, G), qt.qtale_quantize(Wu.cuda(), bits, G), A.cuda())
    torch.cuda.synchronize()
    d = [orc.dequantize(*orc.quantize_rtn(W.numpy(), bits, G), G).T for W in (Wg, Wu)]
    want = orc.silu(to_f64(A) @ d[0]) * (to_f64(A) @ d[1])
    check_parity(orc.parity_error(to_f64(out), want), "fp16", ("few-row swiglu", M, I, K))


@pytest.mark.parametrize("T,lens,old,cap", [(1, [1], [0], 64), (1, [0, 1, 0], [9, 700, 3], 704), (3, [1, 1, 1], [300, 1, 77], 304),
                                            (4, [4], [130], 256), (4, [2, 0, 2], [63, 5, 64], 128), (5, [1] * 5, [9, 8, 7, 6, 5], 64)])
@pytest.mark.parametrize("H,ratio", [(256, 1.0), (256, 0.5), (4104, 1.0)])
def test_decode_call_of_a_few_tokens(qt, T, lens, old, cap, H, ratio):
    # up to four tokens select and normalise inside the GEMM launches, five do not; hidden 4104 takes two pieces per thread
    # and is not a multiple of the 64-wide k-tile; empty and fresh caches, several new rows per sequence, empty sequences
    if int(ratio * T + 0.5) == 0:
        pytest.skip("no token executes")
    shape = si.LayerShape(H, 4, 2, 64, 344, 4, 32, "bf16") if H == 256 else si.LayerShape(H, 2, 1, 128, 136, 3, 64, "fp16")
    _cache_case(qt, shape, lens, old, old, cap, 400 + T + H, ratio)


@pytest.mark.parametrize("router", ["linear", "mlp"])
@pytest.mark.parametrize("mode,val", [("ratio", 0.5), ("threshold", 0.5), ("threshold", 0.0), ("threshold", 1.0)])
def test_selection_inside_the_first_gemm(qt, router, mode, val):
    # four tokens without a cache, two of them tied: decision, scores and bypassed rows against the oracle
    shape = si.LayerShape(512, 4, 4, 64, 344, 4, 64, "bf16")
    tensors = si.layer_tensors(shape, 0, 5, unit_gains=False, std=0.057)
    if router == "mlp":
        tensors["router_mlp"] = si.router_mlp(shape, 0, 5, std1=0.057)
    x = si.hidden_states(shape, 4, 5)[[0, 1, 0, 3]].contiguous()
    offs, pos = si.ragged_sequences([3, 1], [0, 9])
    got, idx, _ = _run_layer(qt, shape, tensors, x, offs, pos, mode, val)
    p, _ = oracle_layer(shape, 0, 5, tensors=tensors)
    if router == "mlp":
        p.router_mlp = tuple(t.numpy() for t in tensors["router_mlp"])
    want, widx, _ = orc.layer_forward(to_f64(x), p, cfg_dict(shape), offs.numpy(), pos.numpy(), mode, val)
    assert np.array_equal(idx, widx)
    skipped = np.setdiff1d(np.arange(4), widx)
    assert torch.equal(got[skipped], x[skipped])
    if len(widx):
        check_parity(orc.parity_error(to_f64(got)[widx], want[widx]), shape.act_dtype, ("few tokens", router, mode, val), hidden=shape.hidden)


# Workgroup shapes of the launches that select and normalise (16-column fragments of q|k|v: up to 512, 768, more; pairs of
# gate and up: up to 512, 768, more), and a hidden size whose row takes two passes of the 768-thread workgroups
@pytest.mark.parametrize("H,nh,nkv,I,bits,dtype", [(256, 40, 20, 4104, 4, "bf16"), (128, 80, 40, 8200, 3, "fp16"), (256, 120, 60, 12296, 4, "fp16"),
                                                   (6152, 80, 40, 8200, 4, "bf16")])
@pytest.mark.parametrize("T,mode,val", [(1, "ratio", 1.0), (3, "threshold", 0.5), (4, "ratio", 0.5), (4, "threshold", 0.5)])
def test_fused_prologues_in_every_workgroup_shape(qt, H, nh, nkv, I, bits, dtype, T, mode, val):
    shape = si.LayerShape(H, nh, nkv, 64, I, bits, 64, dtype)
    _check_layer(qt, shape, T, [T // 2, 0, T - T // 2], mode, val, seed=600 + T, std=1.28 / H ** 0.5, starts=[0, 5, 9])


@pytest.mark.parametrize("rep", [1, 4])
@pytest.mark.parametrize("d", [64, 128])
def test_decode_calls_of_more_than_256_tokens(qt, rep, d):
    # selection and normalisation are launches of their own, and the normalising one leaves the rotary table and the cleared
    # counters; with 90 executed rows the keys are split into equally many ranges per row (no length from the device); empty,
    # very short and full caches.  Two tokens per sequence: the same with rotation and append before the attention kernel.
    shape = si.LayerShape(256, rep, 1, d, 344, 4, 32, "fp16")
    old = [int(v) for v in np.random.default_rng(rep + d).integers(0, 511, size=300)]
    old[:6] = [0, 1, 511, 2, 0, 63]
    _cache_case(qt, shape, [1] * 300, old, old, 512, 550 + rep, 1.0)
    _cache_case(qt, shape, [1] * 300, old, old, 512, 560 + rep, 0.3)
    _cache_case(qt, shape, [2] * 150, old[:150], old[:150], 513, 570 + rep, 0.4)


@pytest.mark.parametrize("rep", [1, 2, 4, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_decode_attention_rotates_and_appends(qt, rep, d):
    # many rows (keys not split) and few rows (split, combined by the last range); more new rows per sequence than one step
    # of the kernel covers
    shape = si.LayerShape(256, 2 * rep, 2, d, 128, 4, 32, "fp16")
    old = [int(v) for v in np.random.default_rng(rep + d).integers(0, 300, size=140)]
    _cache_case(qt, shape, [1] * 140, old, old, 301, 500 + rep, 1.0)
    _cache_case(qt, shape, [40, 0, 1, 3] + [0] * 8, [70, 5, 640, 0] + [1] * 8, [70, 5, 640, 0] + [1] * 8, 641, 510 + rep, 1.0)


@pytest.mark.parametrize("rep", [1, 2, 4, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_decode_attention_after_a_separate_append(qt, rep, d):
    # more than 96 new tokens beyond one per sequence: rotation and append are a launch of their own; keys not split (134
    # rows), and split into equally many ranges per row (67 rows), with an empty sequence, fresh and very short caches
    shape = si.LayerShape(256, 2 * rep, 2, d, 128, 4, 32, "fp16")
    lens = [100, 0] + [1] * 34
    old = [300, 9] + [int(v) for v in np.random.default_rng(rep * d).integers(0, 640, size=34)]
    old[5], old[6] = 0, 1
    _cache_case(qt, shape, lens, old, old, 641, 520 + rep, 1.0)
    _cache_case(qt, shape, lens, old, old, 641, 530 + rep, 0.5)


@pytest.mark.parametrize("B", [160, 161])
@pytest.mark.parametrize("rep", [1, 2])
def test_decode_attention_beside_idle_sequences(qt, B, rep):
    # one long new part and empty sequences around it, at the token count where one query head per kv head changes its route
    shape = si.LayerShape(256, 2 * rep, 2, 64, 128, 4, 32, "fp16")
    lens, old = [0] * B, [7] * B
    lens[3], old[3] = B, 100
    _cache_case(qt, shape, lens, old, old, 300, 545 + rep, 1.0)


@pytest.mark.parametrize("lens,old,cap", [([1, 1, 1], [300, 0, 77], 304), ([2, 0, 3], [63, 5, 700], 704), ([1] * 140, [90] * 140, 96)])
def test_decode_attention_of_heads_wider_than_the_hidden_size(qt, lens, old, cap):
    # the rotary table has no room in the residual's buffer: the same decode kernel, rotation and append before it
    _cache_case(qt, si.LayerShape(64, 4, 2, 128, 136, 4, 32, "bf16"), lens, old, old, cap, 540 + len(lens), 1.0)


def test_decode_rows_that_do_not_fit_the_cache(qt):
    # five new rows, room for two: the others are dropped, see what the cache holds, and the counter stops at the capacity
    shape = si.LayerShape(256, 4, 2, 64, 344, 4, 32, "fp16")
    tensors = si.layer_tensors(shape, 0, 8, unit_gains=False, std=0.08)
    x = si.hidden_states(shape, 5, 8)
    offs, pos = torch.tensor([0, 5, 5], dtype=torch.int32), torch.arange(30, 35, dtype=torch.int32)
    kc, vc = si.kv_cache(shape, 2, 32, 0, 8)

    def run(n):
        kv = qt.KVCache.from_token_major(kc.cuda(), vc.cuda(), torch.tensor([30, 4], dtype=torch.int32).cuda(), 2)
        o = torch.tensor([0, n, n], dtype=torch.int32)
        got, _, _ = _run_layer(qt, shape, tensors, x[:n], o, pos[:n], "ratio", 1.0, kv=kv)
        return got, kv

    full, kv = run(5)
    fits, kv2 = run(2)
    assert kv.kv_len.tolist() == [32, 4] and kv2.kv_len.tolist() == [32, 4]
    assert torch.equal(kv.k, kv2.k) and torch.equal(kv.v, kv2.v)
    check_parity(orc.parity_error(to_f64(full[:2]), to_f64(fits)), "fp16", "rows that fit", hidden=256)
    assert torch.isfinite(full).all()


@pytest.mark.parametrize("lens,absent", [([1, 1], {"router", "select", "norm1", "rope_append", "norm2"}), ([1] * 8, {"norm1", "rope_append"}),
                                         ([110] + [1] * 40, {"norm1"}), ([1] * 300, {"rope_append"})])
def test_profile_classes_of_fused_calls(qt, lens, absent):
    # which classes have launches of their own, as include/qtale.h describes them
    shape = si.LayerShape(256, 4, 2, 64, 344, 4, 32, "fp16")
    T, B = sum(lens), len(lens)
    lw = qt.quantize_layer(si.layer_tensors(shape, 0, 12, unit_gains=False, std=0.08), 4, 32)
    kc, vc = si.kv_cache(shape, B, 160, 0, 12)
    kv = qt.KVCache.from_token_major(kc.cuda(), vc.cuda(), torch.full((B,), 40, dtype=torch.int32).cuda(), 2)
    offs, pos = si.ragged_sequences(lens, [40] * B)
    ctx = qt.Context()
    qt.qtale_profile_enable(ctx, True)
    qt.qtale_layer_forward(ctx, qt.cfg_from_shape(shape), lw, si.hidden_states(shape, T, 12).cuda(), offs.cuda(), pos.cuda(), kv=kv)
    prof = qt.qtale_profile_read(ctx)
    assert {name for name, (_, n) in prof.items() if n == 0} == absent
    assert all(n <= 1 for _, n in prof.values())


def test_few_row_stack_is_the_same_on_every_run(qt):
    # the last range to arrive combines the key ranges: whichever that is, the bits are the same
    shape = si.LayerShape(256, 8, 2, 64, 344, 4, 32, "bf16")
    layers = [qt.quantize_layer(si.layer_tensors(shape, l, 9, unit_gains=False, std=0.08), 4, 32) for l in range(3)]
    old = [900, 333, 1200]
    caches = [si.kv_cache(shape, 3, 1216, l, 9) for l in range(3)]
    offs, pos = torch.arange(4, dtype=torch.int32).cuda(), torch.tensor(old, dtype=torch.int32).cuda()
    ctx = qt.Context()
    qt.qtale_set_exec_ratio(ctx, 1.0)
    outs = []
    for _ in range(4):
        kvs = [qt.KVCache.from_token_major(k.cuda(), v.cuda(), torch.tensor(old, dtype=torch.int32).cuda(), 2) for k, v in caches]
        x = si.hidden_states(shape, 3, 9).cuda()
        qt.qtale_stack_forward(ctx, qt.Stack(qt.cfg_from_shape(shape), layers, kvs), x, offs, pos)
        torch.cuda.synchronize()
        outs.append((x.cpu(), [kv.k.cpu() for kv in kvs]))
    for x, ks in outs[1:]:
        assert torch.equal(x, outs[0][0]) and all(torch.equal(a, b) for a, b in zip(ks, outs[0][1]))


@pytest.mark.parametrize("T", [1, 4, 5, 8])
@pytest.mark.parametrize("I,G", [(6152, 128), (6136, 32)])
def test_streamed_weights_give_the_bits_of_cached_ones(qt, T, I, G):
    # gate/up of 6 MB: non-temporal loads in a call of a single layer (just below it: ordinary ones), ordinary loads in a stack whose
    # weights fit the memory-side cache
    shape = si.LayerShape(1024, 16, 4, 64, I, 4, G, "fp16")
    _check_layer(qt, shape, T, [T - T // 2, T // 2], "ratio", 1.0, seed=60 + T)
    layer = qt.quantize_layer(si.layer_tensors(shape, 0, 60 + T, unit_gains=False), 4, G)
    cfg, ctx = qt.cfg_from_shape(shape), qt.Context()
    qt.qtale_set_exec_ratio(ctx, 1.0)
    x0 = si.hidden_states(shape, T, 60 + T).cuda()
    offs, pos = (t.cuda() for t in si.ragged_sequences([T - T // 2, T // 2]))
    xl, xs = x0.clone(), x0.clone()
    qt.qtale_layer_forward(ctx, cfg, layer, xl, offs, pos)
    qt.qtale_stack_forward(ctx, qt.Stack(cfg, [layer]), xs, offs, pos)
    torch.cuda.synchronize()
    assert torch.equal(xl, xs)
