"""The tile kernels whose variants follow all others of a family: what the other variants need stays as it is without them."""
import pytest

from paper_2512_09196_amd import tf


# (256 x 256 tiles in four slices: 512 bytes below the built-in buffer's size, fewer than the counters of 64 x 128 tiles)
def test_a_variant_that_fills_the_built_in_buffer_fits():
    with tf.Problem(670, 3136, 1536, trans_b=1) as p:
        v = [v for v in p.variants() if v.name == b"lds_256x256x64_w2x4_s2_direct_bnk_sk4r"][0]
    assert v.workspace_bytes == 33619456 <= tf.lib().tf_static_scratch_bytes()


@pytest.mark.parametrize("M,N,K,trans_b", [(670, 3136, 1536, 1), (812, 744, 9152, 1), (3219, 936, 880, 0), (1024, 1024, 16384, 0), (2048, 2048, 2048, 0), (1643, 2272, 2568, 1), (100, 4096, 4096, 0)])
def test_the_counter_area_is_that_of_the_other_variants(M, N, K, trans_b):
    tiles = lambda v: v.grid // v.split_k
    with tf.Problem(M, N, K, trans_b=trans_b) as p:
        sliced = [v for v in p.variants() if v.split_k > 1 and v.kind in (tf.TF_KIND_MFMA_LDS, tf.TF_KIND_MFMA_STREAM, tf.TF_KIND_MFMA_KSHARE)]
        streamk = [v for v in p.variants() if v.stream_k]
    area = lambda n: -(-n * 8 // 256) * 256
    others = [area(tiles(v)) for v in sliced if (v.bm, v.bn) != (64, 128) and v.kind != tf.TF_KIND_MFMA_KSHARE]
    others += [area(-(-M // v.bm) * -(-N // v.bn)) for v in streamk + [v for v in sliced if v.kind == tf.TF_KIND_MFMA_KSHARE]]
    assert others and {v.workspace_bytes - v.split_k * M * N * 4 for v in sliced} == {max(others) + 256}


def launch(v):
    return v.split_k, v.fused_reduce, v.xcd_swizzle, v.grid, v.workspace_bytes, v.trans_b


@pytest.mark.parametrize("M,N,K,trans_b,bms", [(1160, 3080, 1864, 0, {128}), (1160, 3080, 1864, 1, {128}), (551, 2880, 1128, 0, {64, 128}), (1172, 928, 2120, 1, {64, 128}),
                                               (128, 256, 11528, 1, {64, 128}), (1000, 2000, 520, 0, set()), (3219, 936, 880, 0, {128})])
def test_rows_in_whole_lines_are_offered_beside_the_other_instances(M, N, K, trans_b, bms):
    """Every launch in whole lines has its counterpart with three buffers, and follows all other variants; the static model puts
    it ahead of that one, but for a [K][N] B and fewer than 16 K tiles a slice, where the two were measured level."""
    with tf.Problem(M, N, K, trans_b=trans_b) as p:
        vs = p.variants()
        us = [tf.predict_us(p.desc, tf.hw_nominal(), v) for v in vs]
    lined = [v for v in vs if v.direct_to_lds == 3]
    assert {v.bm for v in lined} == bms and [v.id for v in lined] == list(range(len(vs) - len(lined), len(vs)))
    for v in lined:
        other = [u for u in vs if (u.kind, u.direct_to_lds, u.bm, u.bn, u.stages) == (v.kind, 2, v.bm, v.bn, 3) and launch(u) == launch(v)]
        level = not trans_b and -(-(-(-K // 64)) // v.split_k) < 16
        assert len(other) == 1 and (us[v.id] == us[other[0].id] if level else us[v.id] < us[other[0].id])


def test_the_model_takes_no_other_ragged_instance_for_one_in_whole_lines():
    """The descriptor says which they are: one more buffer alone makes no difference to a problem that three keep fed."""
    with tf.Problem(1160, 3080, 1864) as p:
        v = [v for v in p.variants() if v.name == b"lds_128x128x64_w2x4_s3_direct_sk1"][0]
        us = []
        for v.stages in (3, 4, 5):
            us.append(tf.predict_us(p.desc, tf.hw_nominal(), v))
    assert us[0] == us[1] == us[2]


# (us, the pick in whole lines / the one expected: 12.6 / 10.0, 11.0 / 9.1, 12.9 / 10.8, 12.9 / 11.0, 13.0 / 12.3)
@pytest.mark.parametrize("M,N,K,trans_b,name", [(396, 3000, 944, 1, b"lds_64x128x64_w2x4_s3_direct_bnk_sk1"), (114, 10032, 824, 1, b"lds_64x128x64_w2x4_s3_direct_bnk_sk1"),
                                                (1107, 1616, 872, 1, b"lds_64x128x64_w2x4_s3_direct_bnk_sk1"), (504, 3680, 936, 1, b"lds_64x128x64_w2x4_s3_direct_bnk_sk1"),
                                                (3219, 936, 880, 0, b"lds_128x128x64_w2x4_s3_direct_sk1")])
def test_static_picks_at_few_k_tiles_keep_off_whole_lines(M, N, K, trans_b, name):
    hw = tf.hw_nominal()
    with tf.Problem(M, N, K, trans_b=trans_b, epi=tf.TF_EPI_BIAS) as p:
        vs = p.variants()
        assert vs[tf.proposal(p.desc, hw, vs, [v.id == 0 for v in vs], 0, tf.TF_BN_UNKNOWN)].name == name


def test_whole_lines_are_no_other_staging_path_to_a_hint():
    """A bank-conflict diagnosis asks for another staging path or tile: the same tile in whole lines is neither, for the library
    and for the oracle."""
    from oracle import loop_oracle as orc
    fields = ("kind", "bm", "bn", "bk", "stages", "split_k", "direct_to_lds", "lds_bytes", "grid")
    hw = tf.hw_nominal()
    with tf.Problem(1160, 3080, 1864) as p:
        vs = p.variants()
        base, lined = ([v for v in vs if v.name == name][0] for name in (b"lds_128x128x64_w2x4_s3_direct_sk1", b"lds_128x128x64_w2x4_s4_direct_sk1"))
        assert (base.direct_to_lds, lined.direct_to_lds) == (2, 3)
        other = [v for v in vs if v.kind == base.kind and v.bn != base.bn and tf.predict_us(p.desc, hw, v) > tf.predict_us(p.desc, hw, lined)][0]
        tried = [v.id not in (lined.id, other.id) for v in vs]
        assert tf.proposal(p.desc, hw, vs, tried, base.id, tf.TF_BN_LDS_CONFLICT) == other.id
    as_dict = lambda v: {f: getattr(v, f) for f in fields}
    fill = [tf.grid_fill(hw, v) for v in (base, lined)]
    assert not orc.moves_in_direction(orc.LDS_CONFLICT, as_dict(base), as_dict(lined), *fill)
