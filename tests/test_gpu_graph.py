"""tf_variant_run under HIP graph capture: after one eager call (which allocates the workspace and sets the
kernel attributes) a launch records nothing but kernels, so it can be captured and replayed."""
import numpy as np
import pytest

from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu
from oracle import gemm_oracle as orc

pytestmark = pytest.mark.gpu


def pick(prob, pred):
    vs = [v for v in prob.variants() if pred(v)]
    assert vs
    return vs[0]


@pytest.mark.parametrize("which", ["plain", "split_two_kernel", "split_in_kernel", "split_l2_local", "stream", "b_as_nk_staged",
                                   "b_as_nk_transposing_pass"])
def test_captured_launches_replay_to_the_eager_result(which):
    torch = gu.torch_mod()
    M, N, K = (16, 512, 4096) if which == "stream" else (256, 256, 2048)
    A, B, bias = wl.make_custom(M, N, K, seed=7)
    nk = which.startswith("b_as_nk")
    if nk:
        B = np.ascontiguousarray(B.T)
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
    Y_eager = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    Y_graph = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    with tf.Problem(M, N, K, trans_b=1 if nk else 0) as prob:
        v = pick(prob, {
            "plain": lambda v: v.kind == tf.TF_KIND_MFMA_LDS and v.split_k == 1,
            "split_two_kernel": lambda v: v.kind == tf.TF_KIND_MFMA_LDS and v.split_k > 1 and v.fused_reduce == 0,
            "split_in_kernel": lambda v: v.kind == tf.TF_KIND_MFMA_LDS and v.split_k > 1 and v.fused_reduce == 1,
            "split_l2_local": lambda v: v.kind == tf.TF_KIND_MFMA_LDS and v.split_k > 1 and v.fused_reduce == 2,
            "stream": lambda v: v.kind == tf.TF_KIND_MFMA_STREAM and v.split_k > 1,
            "b_as_nk_staged": lambda v: v.kind == tf.TF_KIND_MFMA_LDS and v.trans_b == 1,
            "b_as_nk_transposing_pass": lambda v: b"_pretransB_" in v.name,
        }[which])
        print(which, v.name.decode(), flush=True)
        prob.run(v.id, dA, dB, dbias, Y_eager)                  # eager: first use allocates and sets attributes
        torch.cuda.synchronize()
        want = Y_eager.view(torch.int16).cpu().numpy().copy()
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(s):
            prob.run(v.id, dA, dB, dbias, Y_graph, stream=s)     # same workspace, now known to the problem
            torch.cuda.synchronize()
            Y_graph.zero_()
            with torch.cuda.graph(g, stream=s):
                for _ in range(3):
                    prob.run(v.id, dA, dB, dbias, Y_graph, stream=s)
        for rep in range(4):
            Y_graph.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            got = Y_graph.view(torch.int16).cpu().numpy()
            assert np.array_equal(got, want), "replay %d differs from the eager result" % rep
            # eager work of the same problem between the replays (it shares the workspace and its counters)
            prob.run(v.id, dA, dB, dbias, Y_eager)
            torch.cuda.synchronize()
            assert np.array_equal(Y_eager.view(torch.int16).cpu().numpy(), want)


# tiles of both B layouts, K slices refused in favour of one launch, too few columns for the any-address kernel, a ragged
# K on tiles staged through registers, no tile at all
SMALL = [(256, 256, 256, 0), (5, 1032, 4096, 1), (27, 64, 4224, 1), (65, 16, 4256, 0), (35, 8, 144, 0), (2, 16, 160, 0), (24, 504, 2824, 1)]


@pytest.mark.parametrize("shape", SMALL)
def test_static_pick_of_a_small_problem_at_any_address_on_two_streams_and_captured_first(shape):
    torch = gu.torch_mod()
    M, N, K, nk = shape
    cases = []
    for seed in (1, 2):
        A, B, bias = wl.make_custom(M, N, K, seed=seed)
        y, z, s = orc.gemm_bias_gelu(A, B, bias)
        Bd = np.ascontiguousarray(B.T) if nk else B
        odd = lambda bits: gu.to_dev(np.concatenate([[np.uint16(0x7FC1)], bits.ravel(), [np.uint16(0x7FC1)]]))[1:-1]
        cases.append((y, gu.strict_bound(y, z, s, K), [gu.to_dev(A), gu.to_dev(Bd), gu.to_dev(bias)], [odd(A), odd(Bd), odd(bias)]))
    value = lambda t: wl.bf16_bits_to_f32(t.cpu().numpy().view(np.uint16)).astype(np.float64).reshape(M, N)
    new = lambda: torch.full((M * N + 2,), gu.CANARY_BF16, dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()

    with tf.Problem(M, N, K, trans_b=nk) as prob:
        vs = prob.variants()
        pick = tf.proposal(prob.desc, tf.hw_query(0), vs, [v.id == 0 for v in vs], 0, tf.TF_BN_UNKNOWN)
        assert pick > 0 and vs[pick].workspace_bytes == 0
        # the pick and the tile kernel that falls back, at aligned addresses and one element off
        for i in {pick} | {v.id for v in vs if v.kind == tf.TF_KIND_MFMA_LDS_ANY}:
            for at in (0, 1):
                print("case", shape, vs[i].name.decode(), "element offset", at, flush=True)
                Y = new()
                prob.run(i, *cases[0][2 + at], Y[at:])
                torch.cuda.synchronize()
                out = Y[at:at + M * N]
                assert np.all(np.abs(value(out) - cases[0][0]) <= cases[0][1]), vs[i].name.decode()
                assert (Y[:at] == gu.CANARY_BF16).all() and (Y[at + M * N:] == gu.CANARY_BF16).all()
        # two streams, one problem, no order between them
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        Ys = [[torch.zeros(M * N, dtype=torch.int16, device="cuda") for _ in range(8)] for _ in streams]
        torch.cuda.synchronize()
        for r in range(8):
            for c, st in enumerate(streams):
                prob.run(pick, *cases[c][2], Ys[c][r], stream=st)
        torch.cuda.synchronize()
        for c in range(2):
            assert np.all(np.abs(value(Ys[c][0]) - cases[c][0]) <= cases[c][1])
            assert all(torch.equal(Ys[c][0], t) for t in Ys[c])

    with tf.Problem(M, N, K, trans_b=nk) as prob:
        Y = torch.zeros(M * N, dtype=torch.int16, device="cuda")
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            prob.run(pick, *cases[0][2], Y)
        for _ in range(3):
            Y.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y, Ys[0][0])
            prob.run(pick, *cases[1][2], Ys[1][0])
            torch.cuda.synchronize()


def test_loop_on_a_small_problem_at_odd_addresses_finds_a_kernel():
    torch = gu.torch_mod()
    M, N, K = 64, 264, 320
    A, B, bias = wl.make_custom(M, N, K, seed=4)
    odd = lambda bits: gu.to_dev(np.concatenate([[np.uint16(0)], bits.ravel()]))[1:]
    Y = torch.zeros(M * N + 1, dtype=torch.int16, device="cuda")
    with tf.Problem(M, N, K) as prob:
        best, rep, log = prob.tune(odd(A), odd(B), odd(bias), Y[1:])
        assert best != 0 and rep.t_med_us < log[0].t_med_us
