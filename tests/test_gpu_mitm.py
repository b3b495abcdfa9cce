"""The separable searches by meet in the middle (fixed-state and static,
without a dump) against the general scan of the same library (the same call
with a dump, which the oracle pins elsewhere) and, where a space is too large
for a dump, against an enumeration in whole numbers: counts, top-k indices and
canonical J bit for bit, over the splits, ranges and values where they could
differ.  n_scans tells which path answered.  The inversion of the rounded VRAM
additions is checked on the CPU against the additions themselves."""
import math
import os
import subprocess
from dataclasses import replace

import numpy as np
import pytest

from paper_2609_02109_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_02109_amd import mf as mfmod
    return mfmod


INVERSE_TEST = r"""
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <random>
#include "mf_vram.h"
static float bits(uint32_t b) { float f; memcpy(&f, &b, 4); return f; }
int main()
{
    std::mt19937_64 r(1);
    long bad = 0;
    for (long t = 0; t < 20000000; t++) {
        float thr, v;
        const int kind = t % 5;
        if (kind == 0) {                       // any finite bit patterns
            do thr = bits((uint32_t)r()); while (!std::isfinite(thr));
            do v = bits((uint32_t)r()); while (!std::isfinite(v));
        } else if (kind == 1) {                // VRAM-like
            thr = (float)(r() % 4000000) * 0x1p-14f;
            v = (float)(r() % 700000) * 0x1p-14f;
        } else if (kind == 2) {                // off the grid, mixed sign
            thr = 300.f * (float)((double)r() * 0x1p-64 - 0.3);
            v = 40.f * (float)((double)r() * 0x1p-64 - 0.5);
        } else if (kind == 3) {                // cancelling, within a few units of each other
            v = 100.f * (float)((double)r() * 0x1p-64);
            thr = v;
            for (int i = (int)(r() % 5); i > 0; i--) thr = nextafterf(thr, (r() & 1) ? INFINITY : -INFINITY);
        } else {                               // extremes
            const float e[] = {FLT_MAX, -FLT_MAX, FLT_MIN, -FLT_MIN, 0x1p-149f, -0x1p-149f, 0.f, -0.f, 1.f, 0x1p100f, -INFINITY};
            thr = e[r() % 11];
            v = e[r() % 10];
        }
        const float x = mfi::vram_inverse(thr, v);
        bool ok = true;
        volatile float s;
        if (x > -INFINITY) { s = x + v; ok = ok && s <= thr; }
        if (x < FLT_MAX) { const float y = nextafterf(x, INFINITY); s = y + v; ok = ok && !(s <= thr); }
        if (!ok && ++bad < 10) printf("thr %a v %a x %a\n", thr, v, x);
    }
    printf("bad %ld\n", bad);
    return bad != 0;
}
"""


def test_vram_inverse_cpu(tmp_path):
    src, exe = tmp_path / "inv.cpp", tmp_path / "inv"
    src.write_text(INVERSE_TEST)
    inc = os.path.join(ROOT, "paper_2609_02109_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", f"-I{inc}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def same(a, b):
    assert a["n_eval"] == b["n_eval"] and a["n_vram"] == b["n_vram"] and a["n_feas"] == b["n_feas"]
    np.testing.assert_array_equal(a["top_idx"], b["top_idx"])
    assert a["top_J"].tobytes() == b["top_J"].tobytes()


def instance(n_options, seed=0, edit=None, **kw):
    kw.setdefault("vram_quantile", 0.6)
    inst = synth.make_instance(n_options, 8, 4, 32, 32, seed=seed, quantise=False, sla_range=(0.2, 1.0), **kw)
    if edit is not None:
        edit(inst)
    return inst


def negative_vram(inst):
    inst.features[:, synth.COL_VRAM] -= 15.0


def huge_vram(inst):   # sums that overflow to infinity (the surrogates do not see the column)
    inst.features[::3, synth.COL_VRAM] = 3e38
    for i in range(inst.n_models):
        inst.model_weights(i)[0][:, synth.COL_VRAM] = 0.0


def tied(inst):        # every configuration's J equal
    for i in range(inst.n_models):
        W1, b1, W2, b2, W3, b3 = inst.model_weights(i)
        W3[1, :] = 0.0


# one model; the largest option count; single options; suffixes of exactly
# 64, 4,096 and just past; more than eight models.  All of one workgroup (up
# to 4,096 prefixes); larger grids are below
SHAPES = [([5], None), ([255], None), ([3, 1, 1, 5], None), ([2] * 6, None), ([2] * 12, None), ([2] * 13, None),
          ([63, 65], None), ([255, 20], None), ([7, 11, 5, 9], negative_vram), ([9, 8, 7, 6], huge_vram),
          ([9, 10, 8], tied), ([13, 16, 16, 17], None), ([4] * 9, None), ([24, 24, 24, 24], None), ([130, 131], None)]


@pytest.mark.gpu
@pytest.mark.parametrize("n_options,edit", SHAPES, ids=[f"{'x'.join(map(str, s))}{'-' + e.__name__ if e else ''}" for s, e in SHAPES])
@pytest.mark.parametrize("eq3", [False, True])
def test_mitm_matches_general_scan(mf, n_options, edit, eq3):
    inst = instance(n_options, edit=edit, vram_cap=90.0 if edit is huge_vram else None)
    n = inst.space_size
    ob = synth.make_objective(inst, 3, tau_range=(-0.4, 0.3)) if eq3 else None
    st = synth.make_state(instance(n_options), 5)
    p = mf.Problem(inst, variants=ob)
    for lo, hi in {(0, n), (n // 3, n), (1, max(n - 1, 1)), (n // 2, min(n // 2 + 3, n)), (0, max(2 * n // 3, 1))}:
        for k in (1, 33, 64):
            print(f"[mitm] {n_options} eq3={eq3} [{lo},{hi}) k={k}", flush=True)
            a = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi, objective=ob, state=st)
            b = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi, objective=ob, state=st, dump=True)
            same(a, b)
            assert b["n_scans"] == 1
            assert a["n_scans"] == 0 or edit is tied
    p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("omega", [np.array([1, -2, 0, 0.5, 1], np.float32), np.full(5, 1e30, np.float32)])
def test_mitm_cap_equal_to_a_sum_and_weights(mf, omega):
    # an inclusive cap that some configurations' rounded sums equal, weights of
    # either sign and of a size whose slack is large against J's differences
    inst = instance([12, 7, 9, 9, 5], seed=2)
    d = [3, 2, 5, 7, 1]
    v = np.float32(0)
    for i in range(5):
        v = np.float32(v + inst.features[inst.option_offsets[i] + d[i], synth.COL_VRAM])
    st = synth.make_state(inst, 1)
    for cap in (v, np.nextafter(v, np.float32(0))):
        p = mf.Problem(replace(inst, vram_cap=float(cap)))
        a = p.search(inst.sla, omega, k=16, state=st)
        same(a, p.search(inst.sla, omega, k=16, state=st, dump=True))
        p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n_options", [[12, 12, 9, 9, 9], [5, 4, 3], [6, 7, 8, 9, 10, 5]])
@pytest.mark.parametrize("steps", [1, 2, 17])
def test_mitm_static_matches_general_scan(mf, n_options, steps):
    inst = synth.make_instance(n_options, 8, 4, 64, 32, seed=4, vram_quantile=0.7, act="sigmoid", quantise=False)
    ob = synth.make_objective(inst, 4)
    sc = synth.make_scenarios(inst, 1, steps, seed=4)
    n = inst.space_size
    p = mf.Problem(inst, variants=ob)
    for lo, hi in ((0, n), (5, n - 2), (n // 2 + 1, n // 2 + 4)):
        for k in (1, 40):
            print(f"[mitm static] {n_options} T={steps} [{lo},{hi}) k={k}", flush=True)
            args = (sc.states[0], sc.sla[0], sc.omega[0])
            a = p.search_static(*args, k=k, lo=lo, hi=hi, objective=ob)
            b = p.search_static(*args, k=k, lo=lo, hi=hi, objective=ob, dump=True)
            same(a, b)
            assert a["n_scans"] == 0 and b["n_scans"] == 1
    p.close()


# ---- searches of more than 4,096 prefixes, by many workgroups

def separable(n_options, good=None, cap=None, seed=0):
    """An instance whose predictions are columns of the option row (latency
    column 6: 0 for the options of `good`, 1 for the others, bound 0.5;
    throughput column 7), every value on the 2^-14 grid: sums are exact in any
    order, so the whole space can be enumerated in integers."""
    inst = synth.make_instance(n_options, 8, 4, 32, 32, seed=seed, vram_quantile=0.6)
    if cap is not None:
        inst = replace(inst, vram_cap=cap)
    f = inst.features
    f[:, 6] = 0.0 if good is None else 1.0
    f[:, 7] += 1.0
    for i, off in enumerate(inst.option_offsets):
        if good is not None:
            f[off + np.asarray(good[i]), 6] = 0.0
        W1, b1, W2, b2, W3, b3 = inst.model_weights(i)
        for a in (W1, b1, W2, b2, W3, b3):
            a[:] = 0.0
        W1[0, 6] = W1[1, 7] = W2[0, 0] = W2[1, 1] = W3[0, 0] = W3[1, 1] = 1.0
    return replace(inst, sla=np.full(inst.n_models, 0.5, np.float32))


def enumerate_separable(inst, omega, lo, hi, k):
    """Counts and top-k of a separable instance (whole-number weights) over
    [lo, hi) by integer sums over every configuration, in torch."""
    import torch
    K = [int(x) for x in inst.n_options]
    j0, S = len(K), 1
    while j0 > 0 and S * K[j0 - 1] <= 1 << 24:
        j0 -= 1
        S *= K[j0]

    def sums(models):
        v = torch.zeros(1, dtype=torch.int64, device="cuda")
        J, ok = v.clone(), torch.ones(1, dtype=torch.bool, device="cuda")
        for i in models:
            r = inst.features[inst.option_offsets[i]:inst.option_offsets[i] + K[i]].astype(np.float64)
            col = lambda c, w: torch.as_tensor(np.rint(r[:, c] * w * 2 ** 14).astype(np.int64), device="cuda")
            v = (v[:, None] + col(synth.COL_VRAM, 1.0)).flatten()
            J = (J[:, None] + col(7, float(omega[i]))).flatten()
            ok = (ok[:, None] & (col(6, 1.0) == 0)).flatten()
        return v, J, ok

    cap = int(np.floor(float(inst.vram_cap) * 2 ** 14))
    (pv, pJ, pok), (sv, sJ, sok) = sums(range(j0)), sums(range(j0, len(K)))
    u = torch.arange(S, device="cuda")
    n_vram = n_feas = 0
    best = torch.empty(0, dtype=torch.int64, device="cuda")   # J 2^34 - index: one integer orders by (J, -index)
    for p in range(lo // S, (hi - 1) // S + 1):
        vram = (sv + pv[p] <= cap) & (u >= lo - p * S) & (u < hi - p * S)
        feas = vram & sok & pok[p]
        n_vram += int(vram.sum())
        n_feas += int(feas.sum())
        key = torch.where(feas, ((sJ + pJ[p]) << 34) - (u + p * S), torch.iinfo(torch.int64).min)
        best = torch.cat([best, key])
        best = torch.topk(best, min(k, len(best)))[0]
    best = best[best > torch.iinfo(torch.int64).min].cpu().numpy()
    J = -(-best >> 34)                                        # rounded up: the index was subtracted
    return dict(n_eval=hi - lo, n_vram=n_vram, n_feas=n_feas, top_idx=((J << 34) - best).astype(np.uint64),
                top_J=J.astype(np.float64) * 2.0 ** -14)


def prefixes(n_options):
    """Prefixes of the split (models before the suffix kept in LDS)."""
    space, S, left = math.prod(n_options), 1, math.prod(n_options)
    for j in range(len(n_options) - 1, -1, -1):
        S *= n_options[j]
        if S > 4096:
            break
        left = space // S
        if left <= 1024 or (left <= 1 << 18 and (j == 0 or S * n_options[j - 1] > 1024)):
            break
    return left


@pytest.mark.gpu
def test_mitm_few_feasible_prefixes_of_many(mf):
    # 2^20 prefixes, four to a lane, of which 64 are feasible, laid out so that
    # some lanes hold three or four of them and their waves few others
    good = [[0, 4, 8, 12], [0], [0, 8, 1, 10], [0, 12, 8, 4], [0], [0], [0], [0]]
    inst = separable([16] * 8, good, cap=1e4)
    p = mf.Problem(inst)
    a = p.search(inst.sla, inst.omega, k=64, state=synth.make_state(inst, 1))
    p.close()
    assert a["n_feas"] == 64 and len(a["top_idx"]) == 64
    same(a, enumerate_separable(inst, inst.omega, 0, inst.space_size, 64))


# 8 to 46 workgroups, a ragged last one, more than eight models
@pytest.mark.gpu
@pytest.mark.parametrize("n_options", [[20] * 5, [9] * 7, [11, 13, 17, 5, 9, 23], [6] * 9], ids=lambda k: "x".join(map(str, k)))
@pytest.mark.parametrize("eq3", [False, True])
def test_mitm_many_workgroups(mf, n_options, eq3):
    assert prefixes(n_options) > 4096
    inst = instance(n_options, seed=3)
    n = inst.space_size
    ob = synth.make_objective(inst, 3, tau_range=(-0.4, 0.3)) if eq3 else None
    st = synth.make_state(inst, 5)
    p = mf.Problem(inst, variants=ob)
    for lo, hi in ((0, n), (n // 7 + 5, n - n // 9 - 1)):
        for k in (1, 33, 64):
            print(f"[mitm grid] {n_options} eq3={eq3} [{lo},{hi}) k={k}", flush=True)
            a = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi, objective=ob, state=st)
            same(a, p.search(inst.sla, inst.omega, k=k, lo=lo, hi=hi, objective=ob, state=st, dump=True))
            assert a["n_scans"] == 0
    p.close()


# one and two prefixes to a lane (331,776), four (2^20), 32 (8.4 million, and a
# range that takes two launches); the last with a clustered half of the options
@pytest.mark.gpu
@pytest.mark.parametrize("n_options,launches,half", [([24] * 6, 1, False), ([16] * 8, 1, False),
                                                     ([33, 32, 32, 255, 17], 2, False), ([16] * 8, 1, True)],
                         ids=lambda x: "x".join(map(str, x)) if isinstance(x, list) else str(x))
@pytest.mark.parametrize("ragged", [False, True])
def test_mitm_spaces_of_many_prefixes(mf, n_options, launches, half, ragged):
    per = prefixes(n_options)
    assert per > 1 << 18 and (per + (1 << 23) - 1) >> 23 == launches
    good = [range(k // 2) for k in n_options] if half else None
    inst = separable(n_options, good, seed=2)
    n = inst.space_size
    lo, hi = (n // 200 + 7, n - n // 300 - 5) if ragged else (0, n)
    p = mf.Problem(inst)
    for omega in (np.ones(len(n_options)), np.arange(len(n_options)) - 1.0):   # the second: -1, 0, 1, 2, ...
        omega = omega.astype(np.float32)
        want = enumerate_separable(inst, omega, lo, hi, 64)
        for k in (1, 33, 64):
            print(f"[mitm space] {n_options} [{lo},{hi}) omega={omega} k={k}", flush=True)
            a = p.search(inst.sla, omega, k=k, lo=lo, hi=hi, state=synth.make_state(inst, 1))
            same(a, dict(want, top_idx=want["top_idx"][:k], top_J=want["top_J"][:k]))
            assert a["n_scans"] == 0
    p.close()


# the largest suffix table (4,096) beside option rows of several steps that LDS
# does not hold as well (read from memory), and beside so many options that a
# shorter suffix is taken
@pytest.mark.gpu
def test_mitm_static_rows_beside_the_largest_table(mf):
    inst = separable([16] * 8, seed=4)
    T = 16
    omega = np.arange(T * 8, dtype=np.float32).reshape(T, 8) % 5 - 1
    want = enumerate_separable(inst, omega.sum(0), 0, inst.space_size, 64)
    p = mf.Problem(inst)
    a = p.search_static(np.stack([synth.make_state(inst, t) for t in range(T)]), np.tile(inst.sla, (T, 1)), omega, k=64)
    p.close()
    assert a["n_scans"] == 0 and a["n_vram"] == want["n_vram"] and a["n_feas"] == want["n_feas"]
    np.testing.assert_array_equal(a["top_idx"], want["top_idx"])
    assert a["top_J"].tobytes() == want["top_J"].tobytes()


@pytest.mark.gpu
@pytest.mark.parametrize("eq3", [False, True])
def test_mitm_many_option_rows(mf, eq3):
    # the range holds one option of the first four models: these meet every
    # constraint, and the cap is the mean sum of the others
    K = [255] * 5 + [64, 64]
    inst = instance(K, seed=6)
    f, off = inst.features, inst.option_offsets
    f[:off[4], synth.COL_VRAM] = 2.0
    cap = 8.0 + sum(float(f[off[i]:off[i] + K[i], synth.COL_VRAM].mean()) for i in (4, 5, 6))
    inst = replace(inst, vram_cap=cap, sla=np.array([np.inf] * 4 + [0.6] * 3, np.float32))
    lo = inst.space_size // 3 + 11
    st = synth.make_state(inst, 6)
    ob = synth.make_objective(inst, 6, tau_range=(-0.4, 0.3)) if eq3 else None
    if eq3:
        ob.tau[:4] = -np.inf
        ob.prev_variant[:4] = -1
    p = mf.Problem(inst, variants=ob)
    for n in (9000, 400_000):
        for k in (1, 64):
            a = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=lo + n, objective=ob, state=st)
            b = p.search(inst.sla, inst.omega, k=k, lo=lo, hi=lo + n, objective=ob, state=st, dump=True)
            same(a, b)
            assert a["n_scans"] == 0 and b["n_scans"] == 1 and a["n_feas"] > 0 and a["n_vram"] < n
    p.close()


# prefixes that tie, in a search of one workgroup: the first `zero` models weigh
# nothing and (flat) take the same VRAM.  Up to 1,024 of them are looked into;
# more, or a tie that goes through the suffixes too, is the scan's
@pytest.mark.gpu
@pytest.mark.parametrize("n_options,zero,flat,scans", [
    ([12, 12, 9, 9, 9], 2, False, 0), ([12, 12, 9, 9, 9], 2, True, 0), ([32, 32, 8, 8, 8], 2, True, 0),
    ([33, 32, 8, 8, 8], 2, True, 1), ([65, 60, 60], 1, True, 0), ([9, 10, 8], 3, False, 0),
    ([12, 12, 9, 9, 9], 5, False, 1)])
def test_mitm_prefixes_that_tie(mf, n_options, zero, flat, scans):
    inst = instance(n_options, seed=5)
    if flat:
        inst.features[:sum(n_options[:zero]), synth.COL_VRAM] = 2.0
        inst = replace(inst, vram_cap=inst.vram_cap - 2.0 * zero)
    inst = replace(inst, sla=np.full(inst.n_models, np.inf, np.float32))
    omega = (np.arange(len(n_options)) >= zero).astype(np.float32)
    st = synth.make_state(inst, 5)
    n = inst.space_size
    p = mf.Problem(inst)
    for lo, hi in ((0, n), (n // 50 + 1, n - n // 60)):
        for k in (1, 33, 64):
            print(f"[mitm tie] {n_options} zero={zero} flat={flat} [{lo},{hi}) k={k}", flush=True)
            a = p.search(inst.sla, omega, k=k, lo=lo, hi=hi, state=st)
            b = p.search(inst.sla, omega, k=k, lo=lo, hi=hi, state=st, dump=True)
            same(a, b)
            assert b["n_feas"] > 64
            if (lo, hi) == (0, n):
                assert a["n_scans"] == scans
    p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [1, 7])
def test_static_scan_without_mask(mf, orc, steps):
    # 1,280 prefixes that tie (the first two models weigh nothing): more than
    # the meet in the middle takes, so the scan answers, without a mask
    inst = synth.make_instance([40, 32, 7, 6, 5], 8, 4, 64, 32, seed=4, vram_quantile=0.7, act="sigmoid", quantise=False)
    inst.features[:72, synth.COL_VRAM] = 2.0
    sc = synth.make_scenarios(inst, 1, steps, seed=4)
    om = sc.omega[0].copy()
    om[:, :2] = 0.0
    g = mf.Problem(inst).search_static(sc.states[0], sc.sla[0], om, k=9)
    r = orc.static_search(inst, None, sc.states[0], sc.sla[0], om, k=9)
    assert g["n_scans"] == 1
    assert g["n_vram"] == r["n_vram"] and g["n_feas"] == r["n_feas"]
    np.testing.assert_array_equal(g["top_idx"], r["top_idx"])
    assert g["top_J"].tobytes() == r["top_J"].tobytes()
