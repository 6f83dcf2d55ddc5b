"""Kernels whose waves share K: edges of the tiles, of the K tile and of the share of a wave and of a slice, both layouts
of B, against the oracle; infinities in the K that the overlapped last K tile fetches twice; slices without an order
between two problems, and replayed from a graph."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu

EPIS = (tf.TF_EPI_BIAS_GELU_ERF, tf.TF_EPI_NONE_F32, tf.TF_EPI_BIAS, tf.TF_EPI_BIAS_GELU_TANH)


def kshare(prob):
    return [v for v in prob.variants() if v.name.startswith(b"kshare_")]


def make(M, N, K, b_as_nk, seed):
    A, B, bias = wl.make_custom(M, N, K, seed=seed)
    return A, B, bias, np.ascontiguousarray(B.T) if b_as_nk else B


# one K tile; less than one per wave; a ragged last tile of 8 and of 56; more tiles than a round of the waves; slices
@pytest.mark.parametrize("b_as_nk", (0, 1))
@pytest.mark.parametrize("M,N,K,pad", [(1, 8, 64, 0), (31, 24, 72, 8), (32, 32, 120, 0), (33, 40, 512, 16), (64, 64, 584, 0),
                                       (65, 72, 1088, 8), (97, 136, 2048, 0), (129, 264, 2056, 0), (40, 512, 8192, 0)])
def test_edges(M, N, K, pad, b_as_nk):
    A, B, bias, Bd = make(M, N, K, b_as_nk, 31 + M + N + K)
    y, z, s = orc.gemm_bias_gelu(A, B, bias)
    want = {tf.TF_EPI_BIAS_GELU_ERF: y, tf.TF_EPI_NONE_F32: z, tf.TF_EPI_BIAS: z,
            tf.TF_EPI_BIAS_GELU_TANH: orc.gelu_tanh(z.ravel()).reshape(z.shape)}
    dA, dB, dbias = gu.to_dev(gu.strided(A, K + pad)), gu.to_dev(gu.strided(Bd, Bd.shape[1] + pad)), gu.to_dev(bias)
    slices = set()
    for epi in EPIS:
        f32 = epi == tf.TF_EPI_NONE_F32
        out = gu.OutBuf(M, N, ldy=N + pad, f32=f32)
        with tf.Problem(M, N, K, lda=K + pad, ldb=Bd.shape[1] + pad, ldy=N + pad, epi=epi, trans_b=b_as_nk) as prob:
            vs = kshare(prob)
            assert vs
            for v in vs:
                slices.add(v.split_k)
                print("case", (M, N, K, pad, b_as_nk), "epi", epi, "variant", v.name.decode(), flush=True)
                for _ in range(2):           # the counters of the slices are ready for a second launch
                    got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
                    assert intact, "%s wrote outside Y" % v.name.decode()
                    err = np.abs(got - want[epi])
                    bound = gu.preact_bound(z, s, K) if f32 else gu.strict_bound(want[epi], z, s, K)
                    assert np.all(err <= bound), "%s: worst excess %g" % (v.name.decode(), (err - bound).max())
    assert K < 8192 or slices == {1, 4, 8, 16}


@pytest.mark.parametrize("b_as_nk", (0, 1))
def test_infinities_where_the_last_k_tile_overlaps(b_as_nk):
    """An infinity in one operand meets zeros of the other nowhere but in its own row or column."""
    M, N, K = 40, 48, 1032                   # the last tile is fetched from 968 on and counts from 1024 on
    A, B, bias, Bd = make(M, N, K, b_as_nk, 5)
    A, Bd = A.copy(), Bd.copy()
    A[3, 1000] = 0x7F80
    if b_as_nk: Bd[7, 1001] = 0x7F80
    else: Bd[1001, 7] = 0x7F80
    with tf.Problem(M, N, K, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        dA, dB, dbias = gu.to_dev(A), gu.to_dev(Bd), gu.to_dev(bias)
        out = gu.OutBuf(M, N, f32=True)
        for v in kshare(prob):
            print("variant", v.name.decode(), flush=True)
            got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
            finite = np.isfinite(got)
            assert intact and not finite[3].any() and not finite[:, 7].any()
            assert np.delete(np.delete(finite, 3, 0), 7, 1).all(), v.name.decode()


def test_slices_are_deterministic_on_two_streams_and_in_a_graph():
    torch = gu.torch_mod()
    M, N, K = 48, 320, 6144
    A, B, bias, Bd = make(M, N, K, 0, 9)
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(Bd), gu.to_dev(bias)
    with tf.Problem(M, N, K) as p0, tf.Problem(M, N, K) as p1:
        for v in [v for v in kshare(p0) if v.split_k > 1]:
            print("variant", v.name.decode(), flush=True)
            want = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
            p0.run(v.id, dA, dB, dbias, want)
            p1.run(v.id, dA, dB, dbias, want)
            streams = [torch.cuda.Stream(), torch.cuda.Stream()]
            Ys = [[torch.zeros_like(want) for _ in range(10)] for _ in streams]
            torch.cuda.synchronize()
            for r in range(10):
                for p, st, ys in zip((p0, p1), streams, Ys):
                    p.run(v.id, dA, dB, dbias, ys[r], stream=st)
            torch.cuda.synchronize()
            assert all(torch.equal(t, want) for ys in Ys for t in ys), v.name.decode()
            Y = torch.zeros_like(want)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.stream(streams[0]):
                with torch.cuda.graph(g, stream=streams[0]):
                    for _ in range(3):
                        p0.run(v.id, dA, dB, dbias, Y, stream=streams[0])
            for _ in range(3):
                Y.zero_()
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(Y, want), v.name.decode()
                p0.run(v.id, dA, dB, dbias, Ys[0][0])
                torch.cuda.synchronize()
