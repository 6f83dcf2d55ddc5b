"""Kernels whose waves share K, in tiles cut to the problem: the numbers of rows and columns that a cut can end on, one and two
K tiles in a wave's ring, a ragged last K tile, against the oracle and, bit for bit, against whole tiles of the same waves."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


def is_cut(v):
    return v.name.startswith(b"kshare_") and v.lds_bytes % 1024 == 64


# one row; eights of rows that the last tile has none, one or seven of; columns shared out unevenly; K of one round of the waves and of
# many, with 8 and 56 left over; rows of 64 (a cut of 64 x 64 tiles) and more
@pytest.mark.parametrize("M,N,K,b_as_nk,pad", [(1, 2048, 1024, 1, 0), (8, 1032, 4104, 1, 8), (9, 520, 4152, 1, 0), (16, 2064, 2048, 1, 0), (17, 1104, 2056, 0, 8),
                                               (31, 2576, 1416, 1, 0), (40, 328, 4104, 0, 0), (64, 336, 3000, 1, 16), (83, 536, 4616, 1, 0),
                                               (130, 640, 2120, 0, 0), (368, 1400, 1096, 1, 0),
                                               (71, 328, 4608, 1, 0), (190, 264, 2048, 0, 8), (79, 264, 4616, 1, 0), (150, 328, 2056, 0, 8)])       # (small problems of more than 64 rows)
def test_cut_tiles(M, N, K, b_as_nk, pad):
    A, B, bias = wl.make_custom(M, N, K, seed=7 * M + N + K)
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    _, z, s = orc.gemm_bias_gelu(A, B, bias)
    dA, dB, dbias = gu.to_dev(gu.strided(A, K + pad)), gu.to_dev(gu.strided(Bd, Bd.shape[1] + pad)), gu.to_dev(bias)
    out = gu.OutBuf(M, N, ldy=N + pad, f32=True)
    with tf.Problem(M, N, K, lda=K + pad, ldb=Bd.shape[1] + pad, ldy=N + pad, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        cut = [v for v in prob.variants() if is_cut(v)]
        assert cut and all(v.split_k == 1 and v.grid <= 256 for v in cut)
        same = {}
        for v in cut:
            print("case", (M, N, K, b_as_nk, pad), "variant", v.name.decode(), v.grid, v.lds_bytes, flush=True)
            got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
            assert intact, "%s wrote outside Y" % v.name.decode()
            assert np.all(np.abs(got - z) <= gu.preact_bound(z, s, K)), v.name.decode()
            # a sum goes by the waves that share K, whatever the tile: equal to the last bit
            assert np.array_equal(same.setdefault(v.waves_k, got), got), v.name.decode()


def test_infinities_stay_in_their_row_and_column():
    """What a cut tile reads of rows it did not fetch, and the K that the overlapped last K tile zeroes."""
    M, N, K = 20, 1112, 1032                 # the last tile is fetched from 968 on and counts from 1024 on
    A, B, bias = wl.make_custom(M, N, K, seed=3)
    A, Bd = A.copy(), np.ascontiguousarray(B.T).copy()
    A[19, 1000], Bd[N - 1, 1001], Bd[3, 5] = 0x7F80, 0x7F80, 0x7F80
    with tf.Problem(M, N, K, epi=tf.TF_EPI_NONE_F32, trans_b=1) as prob:
        dA, dB, dbias = gu.to_dev(A), gu.to_dev(Bd), gu.to_dev(bias)
        out = gu.OutBuf(M, N, f32=True)
        cut = [v for v in prob.variants() if is_cut(v)]
        assert cut
        for v in cut:
            print("variant", v.name.decode(), flush=True)
            got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
            finite = np.isfinite(got)
            assert intact and not finite[19].any() and not finite[:, [3, N - 1]].any()
            assert np.delete(np.delete(finite, 19, 0), [3, N - 1], 1).all(), v.name.decode()
