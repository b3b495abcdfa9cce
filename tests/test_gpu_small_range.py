"""Small ranges whose configurations are dealt over the workgroups in turn
(searches without a dump): the same calls with a dump, which go in order and
which the oracle pins elsewhere, give the same counts, top-k indices and
canonical J, bit for bit, for odd sizes and offsets, option counts of one and
large k, and where equal J lie in one run of neighbours."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2609_02109_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_02109_amd import mf as mfmod
    return mfmod


@pytest.mark.parametrize("K,H,k,lo,n", [
    ((7,), 32, 3, 0, None),                    # a tile with empty columns
    ((1, 33), 32, 16, 0, None),                # one tile and one configuration
    ((1, 5, 1, 13, 1), 64, 8, 3, 61),          # option counts of one, a sub-range
    ((9, 11, 7, 13), 32, 64, 0, None),         # k = 64 over 18 workgroups
    ((9, 11, 7, 13), 32, 1, 17, 8191),
    ((11, 13, 9, 11, 5), 64, 16, 12345, 50021),
    ((200, 251, 17), 32, 16, 1, 853399),       # more tiles than waves
])
@pytest.mark.parametrize("flat", [False, True])
def test_dealt_ranges(mf, K, H, k, lo, n, flat):
    inst = synth.make_instance(list(K), 12, 6, H, H, seed=len(K) + k, vram_quantile=0.8)
    if flat:   # the last model's options all alike: runs of equal J
        f = np.array(inst.features, copy=True)
        f[len(f) - K[-1]:] = f[len(f) - K[-1]]
        inst = replace(inst, features=f)
    p = mf.Problem(inst)
    hi = inst.space_size if n is None else lo + n
    a = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi)
    b = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi, dump=True)
    p.close()
    assert a["n_eval"] == b["n_eval"] == hi - lo
    assert a["n_vram"] == b["n_vram"] and a["n_feas"] == b["n_feas"]
    np.testing.assert_array_equal(a["top_idx"], b["top_idx"])
    assert a["top_J"].tobytes() == b["top_J"].tobytes()


@pytest.mark.parametrize("K", [(16,) * 4, (8,) * 5, (32,) * 3, (8,) * 6, (16,) * 5, (5, 5, 5, 5, 4), (20,) * 3, (10,) * 3])
@pytest.mark.parametrize("k", [16, 64])
def test_dealt_ranges_of_equal_counts(mf, K, k):
    """Where every option count is the same power of two, and one model weighs
    little, the best configurations lie at regular distances.  The dealing has
    to spread them all the same: no workgroup may hold so many of them that the
    search needs its fallback pass."""
    inst = synth.make_instance(list(K), 8, 4, 32, 32, seed=1, vram_quantile=0.75)
    p = mf.Problem(inst)
    for light in (None, *range(len(K) - 1)):
        om = np.ones(len(K), np.float32)
        if light is not None:
            om[light] = 0.02
        a = p.search(inst.sla, om, k=k)
        b = p.search(inst.sla, om, k=k, dump=True)
        assert a["n_topk_collect"] == 0, light
        assert a["n_vram"] == b["n_vram"] and a["n_feas"] == b["n_feas"]
        np.testing.assert_array_equal(a["top_idx"], b["top_idx"])
        assert a["top_J"].tobytes() == b["top_J"].tobytes()
    p.close()
