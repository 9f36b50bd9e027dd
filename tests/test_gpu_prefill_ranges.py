"""GPU parity of prefill attention whose keys are cut into ranges (run with -m gpu): few query tiles, ranges that end inside a
query tile's causal triangle, ranges without a visible key for some queries, one range and the most there are.  References and
tolerances are those of the other GPU tests."""
import pytest

import synth_inputs as si
from tests.test_gpu_layer import _cache_case, _check_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qt():
    import paper_2602_10431_amd as pkg
    pkg.load_library()
    return pkg


@pytest.mark.parametrize("nh,nkv", [(8, 2), (3, 3)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,old", [([5], [0]), ([127], [1]), ([128], [2111]), ([129, 0, 300], [0, 9, 640]), ([200, 40], [63, 1500]),
                                      ([513], [64]), ([33] * 7, [0, 1, 63, 64, 65, 700, 1])])
def test_chunks_on_a_cache(qt, nh, nkv, d, lens, old):
    shape = si.LayerShape(256, nh, nkv, d, 688, 4, 32, "fp16")
    _cache_case(qt, shape, lens, old, old, max(a + o for a, o in zip(lens, old)) + 1, 800 + sum(lens) + d, 1.0)
    _cache_case(qt, shape, lens, old, old, max(a + o for a, o in zip(lens, old)) + 1, 810 + sum(lens) + d, 0.6)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mode,val", [("ratio", 1.0), ("threshold", 0.5)])
def test_prompts_without_a_cache(qt, d, mode, val):
    shape = si.LayerShape(256, 8, 8, d, 688, 4, 32, "fp16")
    _check_layer(qt, shape, 1100, [1000, 0, 100], mode, val, seed=820 + d, std=0.08, starts=[0, 5, 11])


@pytest.mark.parametrize("d", [64, 128])
def test_a_cache_that_fills_up(qt, d):
    # rows that do not fit are dropped: every query of the last tiles sees the same keys
    import numpy as np
    import torch
    from oracle import qtale_oracle as orc
    from tests.helpers import cfg_dict, check_parity, oracle_layer, to_f64
    from tests.test_gpu_layer import _run_layer
    shape = si.LayerShape(256, 4, 2, d, 688, 4, 32, "fp16")
    cap, old, T = 700, 500, 200
    tensors = si.layer_tensors(shape, 0, 830, unit_gains=False, std=0.08)
    x = si.hidden_states(shape, T, 830)
    offs, pos = si.ragged_sequences([T], [old])
    kc, vc = si.kv_cache(shape, 1, cap, 0, 830)
    kv = qt.KVCache.from_token_major(kc.cuda(), vc.cuda(), torch.tensor([old], dtype=torch.int32).cuda(), shape.n_kv_heads)
    got, idx, _ = _run_layer(qt, shape, tensors, x, offs, pos, "ratio", 1.0, kv=kv)
    p, _ = oracle_layer(shape, 0, 830, tensors=tensors)
    want, widx, _ = orc.layer_forward(to_f64(x), p, cfg_dict(shape), offs.numpy(), pos.numpy(), "ratio", 1.0,
                                      orc.KVCache(to_f64(kc), to_f64(vc), [old]))
    assert np.array_equal(idx, widx) and int(kv.kv_len[0]) == cap
    check_parity(orc.parity_error(to_f64(got), want), "fp16", ("full cache", d), hidden=shape.hidden)
