"""The kernel of one wave per tile: rows, columns and k past the operands' ends (repeated there, not stored, zeroed), K of less than a
group of 64, of one and of several, B in both layouts, against the oracle."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


def one_wave(prob):
    return next(v.id for v in prob.variants() if v.name == b"mfma32_direct_1wave")


@pytest.mark.parametrize("b_as_nk", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 35, 7), (31, 33, 16), (32, 64, 17), (65, 31, 48), (40, 99, 63), (5, 70, 64), (33, 65, 65), (64, 33, 203)])
def test_edges(M, N, K, b_as_nk):
    A, B, bias = wl.make_custom(M, N, K, seed=5 * M + N + K)
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    y, z, s = orc.gemm_bias_gelu(A, B, bias)
    lda, ldb = K + 3, Bd.shape[1] + 5                      # (NaN between the rows)
    dA, dB, dbias = gu.to_dev(gu.strided(A, lda)), gu.to_dev(gu.strided(Bd, ldb)), gu.to_dev(bias)
    for epi, want, bound in ((tf.TF_EPI_NONE_F32, z, gu.preact_bound(z, s, K)), (tf.TF_EPI_BIAS_GELU_ERF, y, gu.strict_bound(y, z, s, K))):
        out = gu.OutBuf(M, N, ldy=N + 1, f32=epi == tf.TF_EPI_NONE_F32)
        with tf.Problem(M, N, K, lda=lda, ldb=ldb, ldy=N + 1, epi=epi, trans_b=b_as_nk) as prob:
            got, intact, _ = gu.run_variant(prob, one_wave(prob), dA, dB, dbias, out)
        assert intact and np.all(np.abs(got - want) <= bound)


@pytest.mark.parametrize("b_as_nk", [0, 1])
def test_infinities_stay_in_their_row_and_column(b_as_nk):
    M, N, K = 35, 40, 61                                   # the last row, column and k are the ones repeated
    A, B, bias = wl.make_custom(M, N, K, seed=4)
    A, B = A.copy(), B.copy()
    A[M - 1, K - 1], B[K - 1, 3], B[K - 1, N - 1] = 0x7F80, 0x7F80, 0x7F80
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    out = gu.OutBuf(M, N, f32=True)
    with tf.Problem(M, N, K, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        got, intact, _ = gu.run_variant(prob, one_wave(prob), gu.to_dev(A), gu.to_dev(Bd), gu.to_dev(bias), out)
    finite = np.isfinite(got)
    assert intact and not finite[M - 1].any() and not finite[:, [3, N - 1]].any()
    assert np.delete(finite[:M - 1], [3, N - 1], 1).all()
