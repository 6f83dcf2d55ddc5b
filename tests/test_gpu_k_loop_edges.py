"""The directly staged K loops where their tail begins and ends: fewer K tiles than buffers, exactly as many, one and two more;
the rotated K order, which wraps round inside that tail for some XCD; K tiles dealt to slices in turn, with a slice that has
one tile less than its neighbour; a ragged last K tile behind each of them. Every variant offered, against the oracle."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu


def check(M, N, K, b_as_nk, select):
    """Runs the selected variants; returns them."""
    A, B, bias = wl.make_custom(M, N, K, seed=7 + M + K)
    Bd = np.ascontiguousarray(B.T) if b_as_nk else B
    y, z, s = orc.gemm_bias_gelu(A, B, bias)
    bound = gu.preact_bound(z, s, K)
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(Bd), gu.to_dev(bias)
    out = gu.OutBuf(M, N, f32=True)
    with tf.Problem(M, N, K, epi=tf.TF_EPI_NONE_F32, trans_b=b_as_nk) as prob:
        ran = [v for v in prob.variants() if v.kind == tf.TF_KIND_MFMA_LDS and v.direct_to_lds and v.trans_b == b_as_nk and select(v)]
        for v in ran:
            print("case", (M, N, K, b_as_nk), v.name.decode(), flush=True)
            got, intact, _ = gu.run_variant(prob, v.id, dA, dB, dbias, out)
            assert intact and np.all(np.abs(got - z) <= bound), v.name.decode()
    return ran


# 1 to 10 K tiles of 64 (rings hold 2 to 8), 1 to 5 of 128, 2 to 20 of 32; then with eight values of K more
@pytest.mark.parametrize("b_as_nk", (0, 1))
@pytest.mark.parametrize("extra", (0, 8))
def test_few_k_tiles(b_as_nk, extra):
    depths, tiles = set(), set()
    for K in range(64, 704, 64):
        # (a ragged K below 256 is staged directly for large outputs only)
        if extra and K < 256:
            continue
        for v in check(136, 264, K + extra, b_as_nk, lambda v: v.split_k == 1 and not v.k_rotate):
            depths.add(v.stages)
            tiles.add((v.stages, -(-(K + extra) // v.bk)))
    assert {2, 3, 4} <= depths
    assert extra or all((d, n) in tiles for d in depths for n in range(1, d + 2))


# (an eighth of K per XCD: the wrap falls on every place of the last ring)
@pytest.mark.parametrize("b_as_nk", (0, 1))
@pytest.mark.parametrize("K", (512, 576, 640, 704, 768, 1024))
def test_rotated_order(K, b_as_nk):
    assert check(264, 392, K, b_as_nk, lambda v: v.k_rotate)


@pytest.mark.parametrize("b_as_nk", (0, 1))
@pytest.mark.parametrize("K", (1024, 1088, 1152, 1216, 2112, 1032, 1096))
def test_dealt_k_tiles(K, b_as_nk):
    ran = check(24, 264, K, b_as_nk, lambda v: v.split_k >= 4 and not v.xcd_swizzle)
    assert ran or b_as_nk


def test_workspace_status_of_the_librarys_buffer():
    """Asked for before any variant has used counters there (only a transposing pass has used the buffer, which it does not
    clear), and after one has."""
    torch = gu.torch_mod()
    M, N, K = 256, 512, 2048
    A, B, bias = wl.make_custom(M, N, K, seed=3)
    ops = gu.to_dev(A), gu.to_dev(np.ascontiguousarray(B.T)), gu.to_dev(bias), torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    with tf.Problem(M, N, K, trans_b=1) as prob:
        vs = prob.variants()
        prob.workspace_status()
        for v in ([v for v in vs if b"pretransB" in v.name][0], [v for v in vs if v.split_k > 1 and v.fused_reduce][0]):
            prob.run(v.id, *ops)
            prob.workspace_status()
