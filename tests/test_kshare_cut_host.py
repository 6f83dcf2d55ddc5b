"""Cut tiles of the kernels whose waves share K, on the CPU: what a family promises whatever the cut."""
import ctypes as C
import os
import random
import subprocess
import sys
import time

import pytest

from paper_2512_09196_amd import tf

WHOLE = {b"kshare_32x32x64_k4_s2": 65536, b"kshare_32x64x64_k8_s1": 98304, b"kshare_64x64x64_k8_s1": 131072}


def test_families_with_cut_tiles():
    rng = random.Random(2)
    seen, rows_over_64 = set(), False
    for _ in range(300):
        M, N, K, nk = rng.choice([rng.randint(1, 64), rng.randint(65, 900)]), 8 * rng.randint(1, 900), 8 * rng.randint(8, 900), rng.randint(0, 1)
        with tf.Problem(M, N, K, trans_b=nk) as p:
            fam = p.variants()
        for v in [v for v in fam if v.name.startswith(b"kshare_")]:
            kernel = b"_".join(v.name.split(b"_")[:4])
            cut = v.lds_bytes % 1024 == 64
            seen.add((kernel, cut, v.split_k > 1))
            if cut:                              # one round, no slices, no workspace, within a CU
                assert v.split_k == 1 and v.workspace_bytes == 0 and 0 < v.grid <= 256 and v.lds_bytes <= 160 * 1024
                assert tf.kernel_substr(v).endswith("true")
            else:                                # whole tiles, as they are without cuts
                assert v.lds_bytes == WHOLE[kernel] and v.bm >= 32
                assert v.split_k > 1 or v.grid == -(-M // v.bm) * -(-N // v.bn)
                assert tf.kernel_substr(v).endswith("false")
        rows16 = [i for i, v in enumerate(fam) if v.name.startswith(b"kshare_16x")]
        lined = [i for i, v in enumerate(fam) if v.direct_to_lds == 3] if M > 64 else []
        last = len(fam) - len(lined)
        assert rows16 == list(range(last - len(rows16), last)) and lined == list(range(last, len(fam)))     # behind all others, but for rows in whole lines
        small = any(v.kind == tf.TF_KIND_MFMA_LDS_ANY for v in fam)
        assert M <= 64 or not rows16 or small
        rows_over_64 |= M > 64 and bool(rows16)
        assert all((fam[i].kind == tf.TF_KIND_MFMA_LDS_ANY) == small for i in rows16)
    assert {(k, c, s) for k, c, s in seen if k in WHOLE} >= {(k, False, True) for k in WHOLE} | {(k, True, False) for k in list(WHOLE)[1:]}
    assert (b"kshare_32x32x64_k4_s2", True, False) not in seen and rows_over_64


def test_rows_of_16_go_by_size_and_not_by_what_else_the_family_has():
    """A K of whole tiles and its neighbours, whose families end in instances that stage rows in whole lines (us in tiles of 32 rows /
    of 16: 141 x 184 x 11760 with B as [N][K] 15.2 / 10.7, 87 x 336 x 7704 21.2 / 15.3)."""
    hw, lined = tf.hw_nominal(), 0
    for M, N, Ks, nk in ((79, 256, (11448, 11456, 11464), 1), (79, 320, (10272, 10280), 0), (141, 184, (11760,), 1), (87, 336, (7680, 7704), 0)):
        for K in Ks:
            with tf.Problem(M, N, K, trans_b=nk) as p:
                fam = p.variants()
            pick = fam[tf.proposal(p.desc, hw, fam, [v.id == 0 for v in fam], 0, tf.TF_BN_UNKNOWN)]
            assert pick.bm == 16 and pick.kind == tf.TF_KIND_MFMA_LDS_ANY, (M, N, K)
            lined += any(v.direct_to_lds == 3 for v in fam)
    assert lined >= 5
    rng = random.Random(5)
    for _ in range(100):
        M, N, K, nk = rng.randint(65, 400), 8 * rng.randint(8, 60), 64 * rng.randint(32, 128), rng.randint(0, 1)
        offers = []
        for k in (K - 8, K, K + 8):
            with tf.Problem(M, N, k, trans_b=nk) as p:
                fam = p.variants()
            if any(v.kind == tf.TF_KIND_MFMA_LDS_ANY for v in fam):
                offers.append({v.name for v in fam if v.bm == 16 and v.name.startswith(b"kshare_")})
        assert all(o == offers[0] for o in offers), (M, N, K, nk)


@pytest.mark.parametrize("M,N,K,name", [(3, 48, 8000, b"kshare_16x32x64_k8_s1_sk1_or_any"), (349, 8, 11136, b"kshare_16x32x64_k8_s1_sk1_or_any"),
                                        (2, 32, 11120, b"kshare_16x32x64_k8_s1_sk1_or_any"), (3, 104, 5824, b"kshare_16x32x64_k8_s1_sk1_or_any"),
                                        (1, 24, 304, b"kshare_32x32x64_k4_s2_sk1_or_any"), (92, 72, 296, b"kshare_32x32x64_k4_s2_sk1_or_any")])
def test_few_tiles_and_a_long_sum_go_to_the_shorter_chain(M, N, K, name):
    """The model has the two level; by their order in the family they went to tiles of 32 x 32 and four waves, which lost up to 7 % there with the
    instruction they run since (us, then / since / eight waves: 2 x 32 x 11120 13.7 / 14.6 / 8.8, 3 x 104 x 5824 8.2 / 8.9 / 6.0)."""
    hw = tf.hw_nominal()
    with tf.Problem(M, N, K) as p:
        fam = p.variants()
        assert fam[tf.proposal(p.desc, hw, fam, [v.id == 0 for v in fam], 0, tf.TF_BN_UNKNOWN)].name == name


def test_a_descriptor_with_empty_fields_is_priced():
    """A caller's descriptor may leave out what the model divides by (in a process of its own, which a division by zero would end)."""
    code = """
import math
from paper_2512_09196_amd import tf
hw = tf.hw_nominal()
for M, N, K in ((16, 4096, 4096), (256, 256, 256)):
    with tf.Problem(M, N, K) as p:
        for at in [v.id for v in p.variants() if v.name.startswith(b"kshare_")]:
            for fields in (["waves_k"], ["stages"], ["bm"], ["bn"], ["split_k"], ["lds_bytes"], ["bm", "bn", "waves_k", "stages", "split_k", "lds_bytes"]):
                v = p.variants()[at]
                for f in fields:
                    setattr(v, f, 0)
                if v.waves_k > 1 or v.kind == tf.TF_KIND_MFMA_KSHARE:
                    assert math.isfinite(tf.predict_us(p.desc, hw, v)) and 1 <= tf.resident_wgs(hw, v) <= 8 and tf.grid_fill(hw, v) > 0, fields
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)


def test_pricing_a_cut_costs_little_more_than_pricing_whole_tiles():
    """A proposal prices every variant. Pricing all 64 cuts of a 64 x 64 tile in full took 12 times what a kernel without cuts does;
    with those left out that cannot be the fastest, 3.6. (The fastest of many runs of each, taken in turn.)"""
    hw, f = tf.hw_nominal(), tf.lib().tf_predict_us
    with tf.Problem(128, 256, 11528, trans_b=1) as p:
        whole, cut = ([v for v in p.variants() if v.name.startswith(name)][0] for name in (b"kshare_32x32x64_k4_s2_bnk_sk1", b"kshare_64x64x64_k8_s1_bnk_sk1"))
        least = {id(v): float("inf") for v in (whole, cut)}
        for _ in range(40):
            for v in (whole, cut):
                args = C.byref(p.desc), C.byref(hw), C.byref(v)
                start = time.perf_counter()
                for _ in range(100):
                    f(*args)
                least[id(v)] = min(least[id(v)], time.perf_counter() - start)
    assert least[id(cut)] < 7 * least[id(whole)]


class Shape(C.Structure):
    """tf::KshareShape"""
    _fields_ = [("groups_a", C.c_int), ("groups_b", C.c_int), ("stages", C.c_int), ("tiles_m", C.c_long), ("tiles_n", C.c_long), ("lds_bytes", C.c_int),
                ("us", C.c_double), ("whole_us", C.c_double), ("is_cut", C.c_bool)]


KERNELS = [(32, 32, 4, 0), (32, 64, 8, 0), (64, 64, 8, 0), (32, 32, 4, 1), (32, 64, 8, 1), (64, 64, 8, 1), (16, 32, 8, 0), (16, 32, 16, 0), (16, 32, 8, 1), (16, 32, 16, 1)]


def takes(kernel, groups_a, groups_b, stages):
    f = tf.lib()["_ZN2tf12kshare_takesEiiii"]           # bool tf::kshare_takes(int, int, int, int), what a launch asks before it starts anything
    f.argtypes, f.restype = [C.c_int] * 4, C.c_bool
    return f(kernel, groups_a, groups_b, stages)


def test_a_cut_without_a_main_loop_is_told_from_the_others():
    """A kernel has a main loop for two K tiles in a ring up to 40 KB in flight in a work-group's rings; another launch would store the bias alone."""
    for i, (bm, bn, waves, nk) in enumerate(KERNELS):
        for ga in range(0, 11):
            for gb in range(0, 11):
                whole = bm >= 32 and (8 * ga, 8 * gb) == (bm, bn)
                cut = not whole and (bm, bn) != (32, 32) and 1 <= ga <= bm // 8 and (1 <= gb <= bn // 8 if nk else gb == bn // 8)
                two = bm <= 32 and waves * (ga + gb) <= 40
                for stages in range(0, 4):
                    want = stages == (2 if bn == 32 else 1) if whole else cut and (stages == 1 or stages == 2 and two)
                    assert takes(i, ga, gb, stages) == want, (bm, bn, waves, nk, ga, gb, stages)


def test_the_model_cuts_to_no_other():
    rng, hw, seen = random.Random(4), tf.hw_nominal(), set()
    f = tf.lib()["_ZN2tf12kshare_shapeEPK15tf_problem_descPK5tf_hwPK15tf_variant_desc"]
    f.argtypes, f.restype = [C.POINTER(tf.ProblemDesc), C.POINTER(tf.Hw), C.POINTER(tf.VariantDesc)], Shape
    for _ in range(400):
        M, N, K, nk = rng.choice([rng.randint(1, 64), rng.randint(65, 900)]), 8 * rng.randint(1, 900), 8 * rng.randint(8, 900), rng.randint(0, 1)
        with tf.Problem(M, N, K, trans_b=nk) as p:
            for v in [v for v in p.variants() if v.name.startswith(b"kshare_")]:
                s = f(C.byref(p.desc), C.byref(hw), C.byref(v))
                assert takes(KERNELS.index((v.bm, v.bn, v.waves_k, nk)), s.groups_a, s.groups_b, s.stages), (M, N, K, nk, v.name)
                assert s.lds_bytes == v.lds_bytes and (v.split_k > 1 or s.tiles_m * s.tiles_n == v.grid)
                seen.add((s.is_cut, s.stages))
    assert seen == {(False, 1), (False, 2), (True, 1), (True, 2)}
