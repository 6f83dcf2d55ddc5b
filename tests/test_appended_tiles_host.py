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
