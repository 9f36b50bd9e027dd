"""GPU parity of decode attention with grouped queries on the matrix cores (run with -m gpu): lengths of cache and of new part
around the 16-key fragments, the 32-key steps of a wave and the 128-key steps of a workgroup, with split and unsplit keys.
References and tolerances are those of the other GPU tests."""
import pytest

import synth_inputs as si
from tests.test_gpu_layer import _cache_case

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 3, 4, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 95, 96, 97, 127, 128, 129, 159, 160, 161, 255, 256, 257, 383, 384, 385, 640]


@pytest.fixture(scope="module")
def qt():
    import paper_2602_10431_amd as pkg
    pkg.load_library()
    return pkg


@pytest.mark.parametrize("rep", [2, 4, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_cache_lengths_around_the_steps(qt, rep, d):
    shape = si.LayerShape(256, 2 * rep, 2, d, 128, 4, 32, "fp16")
    _cache_case(qt, shape, [1] * len(EDGES), EDGES, EDGES, 641, 700 + rep, 1.0)      # few rows: keys split
    old = (EDGES * 5)[:140]
    _cache_case(qt, shape, [1] * 140, old, old, 641, 710 + rep, 1.0)                 # many rows: not split


@pytest.mark.parametrize("rep", [2, 8])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [2, 16, 17, 32, 33, 34])
def test_new_parts_around_the_steps(qt, rep, d, n):
    # the last of n new rows sees n - 1 earlier ones in steps of 32, beside rows without any; a fresh cache and longer ones
    shape = si.LayerShape(256, 2 * rep, 2, d, 128, 4, 32, "fp16")
    lens = [n, 1, n, 1] + [0] * 40
    old = [0, 130, 127, 0] + [3] * 40
    _cache_case(qt, shape, lens, old, old, 192, 720 + n, 1.0)


@pytest.mark.parametrize("rep", [1, 2, 4])
@pytest.mark.parametrize("d", [64, 128])
def test_sequences_of_one_and_of_several_rows_in_one_call(qt, rep, d):
    # the cached keys of the former are read once per call, those of the latter again for each row: two ways to load them
    shape = si.LayerShape(256, 2 * rep, 2, d, 128, 4, 32, "fp16")
    lens, old = [1, 3, 1, 4, 0, 2, 1, 1], [130, 257, 640, 64, 9, 511, 0, 300]
    _cache_case(qt, shape, lens, old, old, 645, 740 + rep, 1.0)                      # few rows: keys split
    lens, old = [1, 3] * 35, (EDGES * 3)[:70]
    _cache_case(qt, shape, lens, old, old, 645, 750 + rep, 1.0)                      # more than 128 rows: not split
