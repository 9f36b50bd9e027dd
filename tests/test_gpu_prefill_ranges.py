"""GPU parity of prefill attention whose keys are cut into ranges (run with -m gpu): few query tiles, ranges that end inside a
query tile's causal triangle, ranges without a visible key for some queries, one range and the most there are.  References and
tolerances are those of the other GPU tests."""
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


@pytest.mark.parametrize("nh,nkv", [(8, 2), (3, 3)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,old", [([5], [0]), ([127], [1]), ([128], [2111]), ([129, 0, 300], [0, 9, 640]), ([200, 40], [63, 1500]),
                                      ([513], [64]), ([33] * 7, [0, 1, 63, 64, 65, 700, 1])])
def test_chunks_on_a_cache(qt, nh, nkv, d, lens, old):
    shape = si.LayerShape(256, nh, nkv, d, 688, 4, 32, "fp16")
    _cache_case(qt, shape, lens, old, old, max(a + o for a, o in zip(lens, old)) + 1, 800 + sum(lens) + d, 1.0)
    _cache_case(qt, shape, lens, old, old, max(a + o for a, o in zip(lens, old)) + 1, 810 + sum(lens) + d, 0.6)


# more than 64 sequences: the work list is sorted by 256 threads, which also measure the ranges and clear their counters; more than 256
# sequences: a thread takes several.  (The ranges' sums lie in the workspace, most of it in the SwiGLU's buffer: its width has room
# for two ranges and more.)
@pytest.mark.parametrize("B,nh,nkv,most,I", [(70, 2, 1, 2000, 24576), (70, 3, 3, 1500, 32768), (260, 1, 1, 1050, 16384)])
@pytest.mark.parametrize("d", [64, 128])
def test_chunks_of_many_sequences(qt, B, nh, nkv, most, I, d):
    shape = si.LayerShape(256, nh, nkv, d, I, 4, 32, "fp16")
    lens = [0 if b % 13 == 5 else 1 + 3 * b % 11 for b in range(B)]
    lens[B // 2], lens[B - 1] = 130, 1
    old = [0 if b % 9 == 2 else (most * (b * 37 % B)) // B for b in range(B)]
    assert sum(lens) > 4 * B                                     # prefill
    _cache_case(qt, shape, lens, old, old, most + 140, 850 + B + d, 1.0)
    _cache_case(qt, shape, lens, old, old, most + 140, 860 + B + d, 0.6)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("mode,val", [("ratio", 1.0), ("threshold", 0.5)])
def test_prompts_without_a_cache(qt, d, mode, val):
    shape = si.LayerShape(256, 8, 8, d, 688, 4, 32, "fp16")
    _check_layer(qt, shape, 1100, [1000, 0, 100], mode, val, seed=820 + d, std=0.08, starts=[0, 5, 11])


def _on_a_full_cache(x, p, cfg, positions, k, v):
    """The oracle's layer for rows that no cache takes in any more: each attends to the entries k, v [cap, n_kv * d] and not to itself."""
    nh, nkv, d = cfg["n_heads"], cfg["n_kv_heads"], cfg["head_dim"]
    q = orc.rmsnorm(x, p.g1, cfg["rms_eps"]) @ p.Wq.T
    attn = np.zeros((len(x), nh * d))
    for i, pos in enumerate(positions):
        qi = orc.rope(q[i], pos, d, cfg["rope_base"])
        for h in range(nh):
            hk = h // (nh // nkv)
            s = k[:, hk * d:(hk + 1) * d] @ qi[h * d:(h + 1) * d] / np.sqrt(d)
            w = np.exp(s - s.max())
            attn[i, h * d:(h + 1) * d] = (w / w.sum()) @ v[:, hk * d:(hk + 1) * d]
    h1 = x + attn @ p.Wo.T
    n2 = orc.rmsnorm(h1, p.g2, cfg["rms_eps"])
    return h1 + (orc.silu(n2 @ p.Wg.T) * (n2 @ p.Wu.T)) @ p.Wd.T


# capacities that end inside a tile of 64 keys and at its end, keys not cut (up to 512 of them) and cut; no row, some rows and all rows fit
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cap,old,T", [(300, 250, 200), (320, 250, 200), (65, 0, 300), (300, 300, 20), (641, 600, 200), (704, 600, 200), (700, 500, 200), (1537, 1500, 140)])
def test_a_cache_that_fills_up(qt, d, cap, old, T):
    # rows that do not fit are dropped and attend to the entries that are there; the second sequence is not concerned
    shape = si.LayerShape(256, 4, 2, d, 688, 4, 32, "fp16")
    tensors = si.layer_tensors(shape, 0, 830, unit_gains=False, std=0.08)
    lens, olds = [T, 30], [old, 10]
    x = si.hidden_states(shape, T + 30, 830)
    offs, pos = si.ragged_sequences(lens, olds)
    kc, vc = si.kv_cache(shape, 2, cap, 0, 830)
    kv = qt.KVCache.from_token_major(kc.cuda(), vc.cuda(), torch.tensor(olds, dtype=torch.int32).cuda(), shape.n_kv_heads)
    got, idx, _ = _run_layer(qt, shape, tensors, x, offs, pos, "ratio", 1.0, kv=kv)
    assert np.array_equal(idx, np.arange(T + 30)) and kv.kv_len.tolist() == [min(old + T, cap), 40]
    fit = min(T, cap - old)
    kept = np.r_[0:fit, T:T + 30]
    p, _ = oracle_layer(shape, 0, 830, tensors=tensors)
    okv = orc.KVCache(to_f64(kc), to_f64(vc), olds)
    want = np.empty((T + 30, shape.hidden))
    want[kept], _, _ = orc.layer_forward(to_f64(x)[kept], p, cfg_dict(shape), np.array([0, fit, fit + 30]), pos.numpy()[kept], "ratio", 1.0, okv)
    want[fit:T] = _on_a_full_cache(to_f64(x)[fit:T], p, cfg_dict(shape), pos.numpy()[fit:T], okv.k[0, :cap], okv.v[0, :cap])
    check_parity(orc.parity_error(to_f64(got), want), "fp16", ("full cache", d, cap, old, T), hidden=shape.hidden)


@pytest.mark.parametrize("nkv,T", [(4, 9), (4, 4), (2, 4), (1, 4), (1, 9)])
@pytest.mark.parametrize("d", [64, 128])
def test_many_small_probabilities_beside_a_large_one(qt, d, nkv, T):
    # one cached key whose score is 10.4 above that of 3000 others: each of these weighs 2^-15 of it (below the smallest normal
    # fp16) and together a tenth, of numerator and denominator.  Prefill (9 rows) and decode forms (4 rows), 1, 2 and 4 query heads per kv head
    shape = si.LayerShape(256, 4, nkv, d, 688, 4, 32, "fp16")
    tensors = si.layer_tensors(shape, 0, 840, unit_gains=False, std=0.08)
    rep, n = 4 // nkv, 3000
    tensors["q"] = tensors["q"].view(nkv, rep, d, 256)[:, :1].expand(nkv, rep, d, 256).reshape(4 * d, 256).contiguous()   # equal in a group
    x = si.hidden_states(shape, 1, 840).expand(T, 256).contiguous()          # the same query in every row
    offs, pos = torch.tensor([0, T], dtype=torch.int32), torch.full((T,), 3001, dtype=torch.int32)
    p, _ = oracle_layer(shape, 0, 840, tensors=tensors)
    q = orc.rope((orc.rmsnorm(to_f64(x[:1]), p.g1, shape.rms_eps) @ p.Wq.T)[0], 3001, d, shape.rope_base).reshape(nkv, rep, d)[:, 0]
    big = q * (10.4 * np.sqrt(d) / (q * q).sum(axis=1, keepdims=True))
    kc, vc = torch.zeros(1, n + 1 + T, nkv * d, dtype=torch.float16), torch.ones(1, n + 1 + T, nkv * d, dtype=torch.float16)
    kc[0, 700], vc[0, 700] = torch.from_numpy(big.reshape(-1)).half(), -1.0
    kv = qt.KVCache.from_token_major(kc.cuda(), vc.cuda(), torch.tensor([n + 1], dtype=torch.int32).cuda(), nkv)
    got, _, _ = _run_layer(qt, shape, tensors, x, offs, pos, "ratio", 1.0, kv=kv)
    want, _, _ = orc.layer_forward(to_f64(x), p, cfg_dict(shape), offs.numpy(), pos.numpy(), "ratio", 1.0, orc.KVCache(to_f64(kc), to_f64(vc), [n + 1]))
    check_parity(orc.parity_error(to_f64(got), want), "fp16", ("small probabilities", d, nkv, T), hidden=shape.hidden)
