"""Tile kernels that stage rows in whole 128-byte lines: every start of a row inside its line (pointers and pitches of any
whole number of 16-byte pieces), K slices that end in front of a line, as many K tiles as buffers and around, rows and columns
that end inside a tile. What lies in the same lines as the operands but outside them is NaN. Against the oracle."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


def lined(v):
    return v.kind == tf.TF_KIND_MFMA_LDS and v.direct_to_lds == 3


def rows_from(bits, ld, skip):
    """Rows `ld` apart that begin `skip` elements behind a 256-byte address, NaN all around: (buffer, address)."""
    rows, cols = bits.shape
    flat = np.full(skip + rows * ld + 64, 0x7FC1, np.uint16)
    flat[skip:skip + rows * ld].reshape(rows, ld)[:, :cols] = bits
    t = gu.to_dev(flat)
    return t, t.data_ptr() + 2 * skip


@pytest.mark.parametrize("b_as_nk", (0, 1))
# 64 x 128 tiles from 16 K tiles a slice on, 128 x 128 ones from 12 (slices of 13, 13, 13, 12 with K 3208; of 17 and 16 with K 2056)
@pytest.mark.parametrize("M,N,K", [(136, 264, 776), (129, 136, 1032), (200, 128, 2056), (257, 392, 3208), (64, 120, 1096)])
@pytest.mark.parametrize("pad,skip", [(0, 0), (8, 8), (32, 56), (40, 16), (56, 40), (48, 24)])
def test_line_rows(M, N, K, b_as_nk, pad, skip):
    A, B, bias = wl.make_custom(M, N, K, seed=11 + M + K)
    z, s = orc.gemm_bias_gelu(A, B, bias)[1:]
    bound = gu.preact_bound(z, s, K)
    lda = K + pad
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    ldb = Bd.shape[1] + (pad if b_as_nk else 0)
    bufA, pA = rows_from(A, lda, skip)
    bufB, pB = rows_from(Bd, ldb, skip if b_as_nk else 0)
    dbias = gu.to_dev(bias)
    out = gu.OutBuf(M, N, f32=True)
    with tf.Problem(M, N, K, lda=lda, ldb=ldb, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        ran = [v for v in prob.variants() if lined(v)]
        for v in ran:
            print("case", (M, N, K, b_as_nk, pad, skip), v.name.decode(), flush=True)
            out.reset()
            prob.run(v.id, pA, pB, dbias, out.ptr)
            got, intact, _ = out.host()
            assert intact and np.all(np.abs(got - z) <= bound), v.name.decode()
    # (rows of whole half lines keep the kernels of three buffers)
    aligned = lda % 32 == 0 and (not b_as_nk or ldb % 32 == 0)
    assert bool(ran) != aligned
