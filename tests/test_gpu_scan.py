"""The scan of ranges past the small-range limit (two tiles per wave, steps
taken from the workgroup's counter, indices decoded by reciprocals) against
the same range searched piece by piece through the small-range kernel: counts
and the merged top-k, bit for bit, at odd offsets and sizes, one to sixteen
models, option counts of one and of 250, and every aggregate width; and the
prediction list at the edges of a step against the dump."""
import numpy as np
import pytest

from paper_2609_02109_amd import synth

pytestmark = pytest.mark.gpu

SMALL = 1 << 20   # the largest small range


@pytest.fixture(scope="module")
def mf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_02109_amd import mf as mfmod
    return mfmod


@pytest.mark.parametrize("K,A,H,k,lo,n", [
    ((250, 250, 17), 2, 32, 1, 3, SMALL + 1),            # one past the limit, wide digits
    ((1, 200, 251, 1, 30), 4, 32, 16, 77, SMALL + 63),
    ((11, 13, 9, 11, 15, 7), 6, 64, 16, 123457, SMALL + 65),
    ((11, 13, 9, 11, 15, 7), 8, 64, 64, 0, None),        # the whole space, k = 64
    ((6, 6, 6, 6, 6, 6, 6, 6), 8, 32, 5, 600011, SMALL + 12289),
    ((2,) * 9 + (4,) * 7, 6, 32, 7, 5000011, SMALL + 129),   # 16 models
    ((3,) * 12 + (2,) * 2, 4, 32, 3, 1000003, SMALL + 191),
])
def test_scan_against_pieces(mf, K, A, H, k, lo, n):
    inst = synth.make_instance(list(K), 12, A, H, H, seed=len(K) + k, vram_quantile=0.8)
    hi = inst.space_size if n is None else lo + n
    p = mf.Problem(inst)
    a = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi)
    parts = [p.search(inst.sla, inst.omega, k=k, lo=x, hi=min(x + SMALL, hi)) for x in range(lo, hi, SMALL)]
    p.close()
    assert a["n_eval"] == hi - lo
    assert a["n_vram"] == sum(r["n_vram"] for r in parts)
    assert a["n_feas"] == sum(r["n_feas"] for r in parts)
    idx = np.concatenate([r["top_idx"] for r in parts])
    J = np.concatenate([r["top_J"] for r in parts])
    order = np.lexsort((idx, -J))[:len(a["top_idx"])]
    assert len(a["top_idx"]) == min(k, len(idx))
    np.testing.assert_array_equal(a["top_idx"], idx[order])
    assert a["top_J"].tobytes() == J[order].tobytes()


# up to a tile of 32 per wave (65,536 on 256 CUs) by the small ranges' kernel,
# past that by the scan
@pytest.mark.parametrize("n", [1, 31, 32, 63, 64, 65, 511, 513, 8191, 8193, 65535, 65536, 65537, 70001])
@pytest.mark.parametrize("K,A,H,act", [([9, 1, 11, 7], 6, 64, "identity"), ([2] * 9 + [1, 3], 4, 32, "sigmoid"),
                                       ([250, 3], 2, 64, "sigmoid")])
def test_list_edges(mf, n, K, A, H, act):
    """A configuration's predictions do not depend on its place in the list,
    nor on which kernel made them."""
    inst = synth.make_instance(K, 12, A, H, H, seed=3, vram_quantile=0.8, act=act)
    p = mf.Problem(inst)
    dump = p.search(inst.sla, inst.omega, k=1, dump=True)["pred"].cpu().numpy()
    idx = np.random.default_rng(n).integers(0, inst.space_size, n)
    got = p.eval_fast(idx).cpu().numpy()
    p.close()
    assert got.tobytes() == dump[idx].tobytes()
