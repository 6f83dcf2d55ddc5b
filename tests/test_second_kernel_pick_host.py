"""The static pick's move to slices behind a second kernel: from slices only, within the room that static runs have, and never further."""
import random

import pytest

from paper_2512_09196_amd import tf

HW = tf.hw_nominal()


def pick_and_first(p):
    fam = p.variants()
    pick = fam[tf.proposal(p.desc, HW, fam, [v.id == 0 for v in fam], 0, tf.TF_BN_UNKNOWN)]
    first = min(fam[1:], key=lambda v: tf.predict_us(p.desc, HW, v))
    return pick, first, any(v.kind == tf.TF_KIND_MFMA_LDS_ANY for v in fam)


def test_what_moves_and_what_stays():
    rng = random.Random(9)
    moved = 0
    for _ in range(900):
        M, N, K = rng.choice([rng.randint(1, 32), rng.randint(33, 1100)]), 8 * rng.choice([rng.randint(32, 200), rng.randint(32, 700)]), 8 * rng.randint(256, 2048)
        with tf.Problem(M, N, K, epi=rng.choice([tf.TF_EPI_BIAS_GELU_ERF, tf.TF_EPI_NONE_F32]), trans_b=rng.randint(0, 1)) as p:
            pick, first, small = pick_and_first(p)
        if small or pick.id == first.id:
            assert not small or pick.workspace_bytes == 0
            continue
        moved += 1
        assert first.split_k > 1 and pick.kind == tf.TF_KIND_MFMA_LDS and pick.split_k > 1 and pick.fused_reduce == 0
        assert 0 < pick.workspace_bytes <= max(first.workspace_bytes, tf.lib().tf_static_scratch_bytes())
    assert moved >= 5


@pytest.mark.parametrize("shape,b_as_nk", [((170, 648, 14936), 0), ((322, 504, 7528), 1), ((72, 1576, 7032), 0)])
def test_measured_moves(shape, b_as_nk):
    with tf.Problem(*shape, trans_b=b_as_nk) as p:
        pick, first, _ = pick_and_first(p)
    assert first.name.startswith(b"kshare_") and pick.kind == tf.TF_KIND_MFMA_LDS and pick.split_k > 1 and pick.fused_reduce == 0
