"""The kernels whose waves share K in the variant loop, on the CPU: the diagnosis of a profile steers the next proposal where
one of them is the base, and can lead to one of them."""
import pytest

from paper_2512_09196_amd import tf

HW = tf.hw_nominal()


def follows(bn, base, v):
    """What a proposal made under a diagnosis may look like, against the variant it starts from."""
    fill, area = tf.grid_fill, lambda x: x.bm * x.bn
    return {tf.TF_BN_UNDERFILLED: fill(HW, v) > fill(HW, base),
            tf.TF_BN_HBM: v.stages > base.stages or v.split_k > base.split_k or v.grid > base.grid,
            tf.TF_BN_MFMA: area(v) >= area(base) and fill(HW, v) >= fill(HW, base) - 1e-9,
            tf.TF_BN_LDS_CONFLICT: bool(v.direct_to_lds) != bool(base.direct_to_lds) or v.bn != base.bn,
            tf.TF_BN_OCCUPANCY: area(v) < area(base) or (area(v) == area(base) and v.lds_bytes < base.lds_bytes),
            tf.TF_BN_LATENCY: v.stages > base.stages or v.bk > base.bk or area(v) > area(base)}[bn]


# a sliced pick, one without slices, a small problem's (listed under two kinds), B as [N][K]
@pytest.mark.parametrize("M,N,K,b_as_nk", [(512, 512, 8192, 0), (1024, 264, 5000, 0), (256, 256, 256, 0), (64, 264, 320, 0), (5, 11008, 4096, 1)])
def test_the_hint_steers_from_a_kernel_whose_waves_share_k(M, N, K, b_as_nk):
    with tf.Problem(M, N, K, trans_b=b_as_nk) as p:
        fam = p.variants()
        tried = [v.id == 0 for v in fam]
        pick = tf.proposal(p.desc, HW, fam, tried, 0, tf.TF_BN_UNKNOWN)
        assert fam[pick].name.startswith(b"kshare_")
        tried[pick] = True
        nxt = {bn: tf.proposal(p.desc, HW, fam, tried, pick, bn) for bn in range(tf.TF_BN_UNDERFILLED, tf.TF_BN_LATENCY + 1)}
        able = [v for v in fam if not tried[v.id] and v.kind in (tf.TF_KIND_MFMA_LDS, tf.TF_KIND_MFMA_LDS_ANY, tf.TF_KIND_MFMA_KSHARE)]
        for bn, i in nxt.items():
            assert follows(bn, fam[pick], fam[i]) or not any(follows(bn, fam[pick], v) for v in able), (bn, fam[i].name)


def test_the_hint_leads_to_a_kernel_whose_waves_share_k():
    """A few large tiles leave most of the chip idle: more and smaller units of work are these kernels' when they are predicted
    to be the fastest of that kind."""
    with tf.Problem(283, 448, 8512) as p:
        fam = p.variants()
        base = next(v for v in fam if v.kind == tf.TF_KIND_MFMA_LDS and (v.bm, v.bn, v.split_k) == (128, 128, 1))
        pred = [float(1000 + v.id) for v in fam]
        tried = [v.id in (0, base.id) for v in fam]
        want = next(v for v in fam if v.kind == tf.TF_KIND_MFMA_KSHARE and follows(tf.TF_BN_UNDERFILLED, base, v))
        other = next(v for v in fam if not tried[v.id] and not follows(tf.TF_BN_UNDERFILLED, base, v))
        pred[want.id], pred[other.id] = 2.0, 1.0
        assert tf.proposal_from(HW, fam, pred, tried, base.id, tf.TF_BN_UNDERFILLED) == want.id


# us, operands of three calls in turn: the best of the other kernels and these kernels' best where a wrong scale between the
# two predictions took, or would take, the slower of them
MEASURED = [((917, 640, 320, 0), {"lds_64x64x64_w2x2_s3_direct_sk1": 3.93, "kshare_64x64x64_k8_s1_sk1": 4.73}),
            ((1883, 320, 384, 0), {"lds_64x64x128_w2x2_s3_direct_sk1": 4.23, "kshare_64x64x64_k8_s1_sk1": 4.95}),
            ((1385, 384, 320, 1), {"lds_64x64x64_w2x2_s3_direct_bnk_sk1": 4.32, "kshare_64x64x64_k8_s1_bnk_sk1": 4.96}),
            ((2073, 448, 448, 1), {"lds_64x64x64_w2x2_s3_direct_bnk_sk1": 4.80, "kshare_64x64x64_k8_s1_bnk_sk1": 5.55}),
            ((67, 7552, 256, 0), {"lds_64x64x128_w2x2_s3_direct_sk1": 3.96, "kshare_64x64x64_k8_s1_sk1": 4.58}),
            ((1103, 640, 448, 0), {"lds_64x64x64_w2x2_s3_direct_sk1": 4.92, "kshare_64x64x64_k8_s1_sk1": 5.46}),
            ((277, 2368, 1792, 0), {"lds_64x64x128_w2x2_s3_direct_sk1x": 8.76, "kshare_64x64x64_k8_s1_sk1": 9.68}),
            ((25, 7808, 6208, 0), {"lds_32x128x64_w1x4_s3_direct_rr_sk4r": 21.8, "kshare_32x32x64_k4_s2_sk1": 24.9}),
            ((16, 8192, 8192, 0), {"lds_32x128x64_w1x4_s3_direct_rr_sk4l": 26.5, "kshare_32x64x64_k8_s1_sk2f": 31.8, "kshare_32x32x64_k4_s2_sk1": 38.1}),
            ((512, 512, 8192, 0), {"kshare_64x64x64_k8_s1_sk4f": 14.6, "lds_64x64x64_w2x2_s3_direct_sk8r": 17.9}),
            ((283, 448, 8512, 0), {"kshare_32x64x64_k8_s1_sk4f": 11.4, "lds_64x64x64_w2x2_s3_direct_sk8r": 13.6}),
            ((333, 640, 8128, 0), {"kshare_32x64x64_k8_s1_sk2f": 15.8, "lds_128x128x64_w2x4_s3_direct_sk16r": 20.6})]


@pytest.mark.parametrize("shape,us", MEASURED, ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else "")
def test_the_static_pick_is_the_faster_kind(shape, us):
    M, N, K, b_as_nk = shape
    with tf.Problem(M, N, K, trans_b=b_as_nk) as p:
        fam = p.variants()
        pick = fam[tf.proposal(p.desc, HW, fam, [v.id == 0 for v in fam], 0, tf.TF_BN_UNKNOWN)].name.decode()
        assert set(us) <= {v.name.decode() for v in fam}
        assert us.get(pick) == min(us.values()), pick
