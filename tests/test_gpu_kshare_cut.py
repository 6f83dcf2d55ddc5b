"""Kernels whose waves share K, in tiles cut to the problem: the numbers of rows and columns that a cut can end on, one and two
K tiles in a wave's ring, a ragged last K tile, against the oracle and, where eight waves share K, bit for bit against whole tiles
of the same waves (sixteen have no whole tiles: the oracle's bound is all that holds them)."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


def is_cut(v):
    return v.name.startswith(b"kshare_") and v.lds_bytes % 1024 == 64


def whole_tiles(M, N, K, A, B, bias, b_as_nk):
    """The product by every kernel of whole tiles whose eight waves share K: its rows and columns over and over, until the tiles
    are more than the CUs and so are not cut."""
    N2 = max(N, 1032)
    M2 = max(M, 64 * -(-257 // -(-N2 // 64)))
    A2, B2, bias2 = A[np.arange(M2) % M], np.ascontiguousarray(B[:, np.arange(N2) % N]), bias[np.arange(N2) % N]
    if b_as_nk:
        B2 = np.ascontiguousarray(B2.T)
    out = gu.OutBuf(M2, N2, f32=True)
    with tf.Problem(M2, N2, K, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        dA, dB, dbias = gu.to_dev(A2), gu.to_dev(B2), gu.to_dev(bias2)
        for v in [v for v in prob.variants() if v.name.startswith(b"kshare_") and v.waves_k == 8 and v.split_k == 1 and not is_cut(v)]:
            print("whole", (M2, N2, K, b_as_nk), "variant", v.name.decode(), v.grid, flush=True)
            got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
            assert intact
            yield got[:M, :N]


# one row; eights of rows that the last tile has none, one or seven of; columns shared out unevenly; K of one round of the waves and of
# many, with 8 and 56 left over; rows of 64 (a cut of 64 x 64 tiles) and more
@pytest.mark.parametrize("M,N,K,b_as_nk,pad", [(1, 2048, 1024, 1, 0), (8, 1032, 4104, 1, 8), (9, 520, 4152, 1, 0), (16, 2064, 2048, 1, 0), (17, 1104, 2056, 0, 8),
                                               (31, 2576, 1416, 1, 0), (40, 328, 4104, 0, 0), (64, 336, 3000, 1, 16), (83, 536, 4616, 1, 0),
                                               (130, 640, 2120, 0, 0), (368, 1400, 1096, 1, 0),
                                               (71, 328, 4608, 1, 0), (190, 264, 2048, 0, 8), (79, 264, 4616, 1, 0), (150, 328, 2056, 0, 8), (3, 8, 2064, 0, 8), (47, 24, 1096, 0, 0), (25, 8, 1032, 1, 0)])       # (small problems of more than 64 rows)
def test_cut_tiles(M, N, K, b_as_nk, pad):
    A, B, bias = wl.make_custom(M, N, K, seed=7 * M + N + K)
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    _, z, s = orc.gemm_bias_gelu(A, B, bias)
    dA, dB, dbias = gu.to_dev(gu.strided(A, K + pad)), gu.to_dev(gu.strided(Bd, Bd.shape[1] + pad)), gu.to_dev(bias)
    out = gu.OutBuf(M, N, ldy=N + pad, f32=True)
    with tf.Problem(M, N, K, lda=K + pad, ldb=Bd.shape[1] + pad, ldy=N + pad, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        cut = [v for v in prob.variants() if is_cut(v)]
        assert cut and all(v.split_k == 1 and v.grid <= 256 for v in cut)
        whole = list(whole_tiles(M, N, K, A, B, bias, b_as_nk))
        assert whole and all(np.array_equal(w, whole[0]) for w in whole)
        same = {8: whole[0]}
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
