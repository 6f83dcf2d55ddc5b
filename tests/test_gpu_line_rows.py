"""Tile kernels that stage rows in whole 128-byte lines: every start of a row inside its line (pointers and pitches of any
whole number of 16-byte pieces) with every length of the ragged K tile, K slices that end in front of a line, a last slice of
fewer K tiles than buffers, as many and one more, rows and columns that end inside a tile. What lies in the same lines as the
operands but outside them is NaN. Against the oracle."""
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


def check(M, N, K, b_as_nk, lda, ldb, skip):
    """Runs every variant that stages whole lines on rows of these pitches; returns them."""
    A, B, bias = wl.make_custom(M, N, K, seed=11 + M + K)
    z, s = orc.gemm_bias_gelu(A, B, bias)[1:]
    bound = gu.preact_bound(z, s, K)
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    bufA, pA = rows_from(A, lda, skip)
    bufB, pB = rows_from(Bd, ldb, skip if b_as_nk else 0)
    dbias = gu.to_dev(bias)
    out = gu.OutBuf(M, N, f32=True)
    with tf.Problem(M, N, K, lda=lda, ldb=ldb, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        ran = [v for v in prob.variants() if lined(v)]
        for v in ran:
            print("case", (M, N, K, b_as_nk, lda, ldb, skip), v.name.decode(), flush=True)
            out.reset()
            prob.run(v.id, pA, pB, dbias, out.ptr)
            got, intact, _ = out.host()
            assert intact and np.all(np.abs(got - z) <= bound), v.name.decode()
    return ran


def whole_sums(M, N, K):
    """Rows of the tiles offered without K slices: 128 x 128 from 12 K tiles on, 64 x 128 from 16, none above twice the output."""
    tiles = -(-K // 64)
    return {bm for bm, least in ((128, 12), (64, 16)) if tiles >= least and bm < 2 * M and 128 < 2 * N}


@pytest.mark.parametrize("b_as_nk", (0, 1))
# 64 x 128 tiles from 16 K tiles a slice on, 128 x 128 ones from 12 (slices of 13, 13, 13, 12 with K 3208; of 17 and 16 with K 2056)
@pytest.mark.parametrize("M,N,K", [(136, 264, 776), (129, 136, 1032), (200, 128, 2056), (257, 392, 3208), (64, 120, 1096)])
@pytest.mark.parametrize("pad,skip", [(0, 0), (8, 8), (32, 56), (40, 16), (56, 40), (48, 24)])
def test_line_rows(M, N, K, b_as_nk, pad, skip):
    lda, ldb = K + pad, K + pad if b_as_nk else N
    ran = check(M, N, K, b_as_nk, lda, ldb, skip)
    # (rows of whole half lines keep to the kernels of three buffers)
    aligned = lda % 32 == 0 and (not b_as_nk or ldb % 32 == 0)
    assert {v.bm for v in ran if v.split_k == 1} == (set() if aligned else whole_sums(M, N, K))


# 17 K tiles, the last of 8 to 56 values of K; rows of A and of an [N][K] B `pitch` pieces of 16 bytes further into a line each
# (0 and 4, whole lines and halves, only for one of the two)
@pytest.mark.parametrize("b_as_nk", (0, 1))
@pytest.mark.parametrize("K", (1032, 1040, 1048, 1064, 1072, 1080))
@pytest.mark.parametrize("pitch,pitch_b,skip", [(1, 2, 0), (2, 5, 8), (3, 6, 16), (5, 1, 40), (6, 7, 56), (7, 3, 24), (0, 3, 48), (4, 6, 8), (3, 0, 32)])
def test_every_pitch_and_every_ragged_tile(K, b_as_nk, pitch, pitch_b, skip):
    M, N = 136, 200
    to_pitch = lambda p: K + (8 * p - K) % 64
    ran = check(M, N, K, b_as_nk, to_pitch(pitch), to_pitch(pitch_b) if b_as_nk else N, skip)
    offered = pitch % 4 != 0 or (b_as_nk and pitch_b % 4 != 0)
    assert {v.bm for v in ran if v.split_k == 1} == ({64, 128} if offered else set())


# sixteen slices, all of 16 K tiles but the last: 1 to 5 of them behind four buffers, the ragged one among them
@pytest.mark.parametrize("b_as_nk", (0, 1))
@pytest.mark.parametrize("last,ragged,pad,skip", [(1, 8, 0, 0), (1, 56, 32, 24), (2, 16, 0, 8), (3, 24, 16, 40), (3, 40, 0, 56), (4, 48, 8, 16), (5, 56, 0, 32)])
def test_short_last_slice(last, ragged, pad, skip, b_as_nk):
    M, N, K = 70, 136, 64 * (15 * 16 + last - 1) + ragged
    ran = check(M, N, K, b_as_nk, K + pad, K + pad if b_as_nk else N, skip)
    tiles = -(-K // 64)
    slices = {(v.bm, v.split_k, tiles - -(-tiles // v.split_k) * (v.split_k - 1)) for v in ran}
    assert {(64, 16, last), (128, 16, last)} <= slices
