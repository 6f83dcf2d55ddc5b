"""The variant loop and the profiler on operands that start at any element: what they report is the launch that those
operands get."""
import numpy as np
import pytest

from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu

# a small problem with several kernels that fall back, with B in either layout, and 256^3
SHAPES = [(64, 264, 320, 0), (40, 520, 200, 1), (256, 256, 256, 0)]
FIGURES = ("vgprs", "lds_bytes", "spill_bytes", "grid", "waves_per_simd", "grid_fill")


def odd_operands(M, N, K, nk):
    torch = gu.torch_mod()
    A, B, bias = wl.make_custom(M, N, K, seed=4)
    odd = lambda bits: gu.to_dev(np.concatenate([[np.uint16(0)], bits.ravel()]))[1:]
    return odd(A), odd(np.ascontiguousarray(B.T) if nk else B), odd(bias), torch.zeros(M * N + 1, dtype=torch.int16, device="cuda")[1:]


def falls_back_to(prob, v):
    """The variant that runs in place of v at these addresses: the any-address kernel predicted to be the quickest, or the
    one-wave kernel."""
    if v.kind != tf.TF_KIND_MFMA_LDS_ANY:
        return v.id
    vs = [u for u in prob.variants() if u.kind in (tf.TF_KIND_MFMA_ANY, tf.TF_KIND_MFMA_DIRECT)]
    return min(vs, key=lambda u: tf.predict_us(prob.desc, tf.hw_query(0), u)).id


@pytest.mark.parametrize("shape", SHAPES)
def test_reports_describe_the_kernel_that_ran(shape):
    ops = odd_operands(*shape)
    M, N, K, nk = shape
    with tf.Problem(M, N, K, trans_b=nk) as prob:
        vs = prob.variants()
        figures = lambda r: [getattr(r, f) for f in FIGURES]
        at_odd = {}
        for v in [v for v in vs if v.kind in (tf.TF_KIND_MFMA_LDS_ANY, tf.TF_KIND_MFMA_ANY, tf.TF_KIND_MFMA_DIRECT)]:
            print("profile", shape, v.name.decode(), flush=True)
            at_odd[v.id] = figures(prob.profile(v.id, *ops, warmup=1, iters=1, launches_per_iter=2))
        for i, f in at_odd.items():
            assert f == at_odd[falls_back_to(prob, vs[i])], vs[i].name
        best, rep, log = prob.tune(*ops)
        for r in log[1:]:
            print("round", shape, vs[r.variant_id].name.decode(), r.status, "%.2f us" % r.t_med_us, flush=True)
            if r.status == tf.TF_OK:
                assert figures(r) == at_odd[r.variant_id], vs[r.variant_id].name


@pytest.mark.parametrize("shape", SHAPES + [(512, 512, 2048, 0)])
def test_the_loop_spends_its_rounds_on_different_launches(shape):
    """No variant that refuses the operands, no launch twice: the any-address kernels, then the one-wave kernel, whatever the
    number of variants that fall back to them (none, for the last shape, which is no small problem)."""
    ops = odd_operands(*shape)
    M, N, K, nk = shape
    with tf.Problem(M, N, K, trans_b=nk) as prob:
        vs = prob.variants()
        best, rep, log = prob.tune(*ops)
        ran = []
        for r in log:
            print("round", shape, vs[r.variant_id].name.decode(), r.status, "%.2f us" % r.t_med_us, flush=True)
            assert r.status == tf.TF_OK
            ran.append(falls_back_to(prob, vs[r.variant_id]))
        assert len(set(ran)) == len(ran)
        assert set(ran) == {v.id for v in vs if v.kind in (tf.TF_KIND_NAIVE, tf.TF_KIND_MFMA_ANY, tf.TF_KIND_MFMA_DIRECT)}
        assert best != 0
