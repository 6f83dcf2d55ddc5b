"""The kernel that sums the K slices of a two-kernel launch: every number of slices, quads that fill no whole work-group, one
workspace for launch after launch, against the oracle and, bit for bit, against the reduction inside the GEMM kernel."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,epi,slices", [(1, 8, 1024, tf.TF_EPI_NONE_F32, {2}), (7, 72, 8192, tf.TF_EPI_BIAS_GELU_ERF, {2, 4, 8, 16, 32}),
                                              (32, 1032, 4096, tf.TF_EPI_NONE_F32, {2, 4, 8, 16}), (65, 136, 4096, tf.TF_EPI_BIAS, {2, 4, 8, 16}),
                                              (130, 264, 4160, tf.TF_EPI_NONE_F32, {2, 4, 8}),
                                              (640, 1048, 2048, tf.TF_EPI_NONE_F32, {2, 4, 8}), (625, 1000, 2048, tf.TF_EPI_BIAS, {2, 4, 8})])   # (eight: 21 MB, not past the L2s; 20 MB)
def test_reducing_kernel(M, N, K, epi, slices):
    A, B, bias = wl.make_custom(M, N, K, seed=M + N)
    _, z, s = orc.gemm_bias_gelu(A, B, bias)
    y = orc.gemm_bias_gelu(A, B, bias)[0]
    f32 = epi == tf.TF_EPI_NONE_F32
    want = y if epi == tf.TF_EPI_BIAS_GELU_ERF else z
    bound = gu.preact_bound(z, s, K) if f32 else gu.strict_bound(want, z, s, K)
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
    out = gu.OutBuf(M, N, ldy=N + 8, f32=f32)
    counts = set()
    with tf.Problem(M, N, K, ldy=N + 8, epi=epi) as prob:
        vs = prob.variants()
        key = lambda v: (v.kind, v.bm, v.bn, v.bk, v.waves_m, v.waves_n, v.waves_k, v.stages, v.direct_to_lds, v.a_bypass_lds, v.split_k, v.xcd_swizzle)
        fused = {key(v): v for v in vs if v.split_k > 1 and v.fused_reduce == 1}
        for v in [v for v in vs if v.split_k > 1 and v.fused_reduce == 0]:
            print("case", (M, N, K, epi), "variant", v.name.decode(), flush=True)
            counts.add(v.split_k)
            first = None
            for _ in range(3):                   # the library's own workspace, written again while the last launch's lines are about
                got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
                assert intact, "%s wrote outside Y" % v.name.decode()
                assert np.all(np.abs(got - want) <= bound), v.name.decode()
                first = got if first is None else first
                assert np.array_equal(got, first)
            if key(v) in fused:
                other, _, _ = gu.run_variant(prob, fused[key(v)].id, dA, dB, dbias, out)
                assert np.array_equal(other, first), v.name.decode()
    assert counts >= slices
