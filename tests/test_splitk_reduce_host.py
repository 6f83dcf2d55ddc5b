"""The second kernel of sliced products: its instances for each number of slices, the ones families list, and which slices pass the L2s by."""
import ctypes as C
import random

from paper_2512_09196_amd import tf


def takes(slices):
    f = tf.lib()["_ZN2tf19splitk_reduce_takesEi"]       # bool tf::splitk_reduce_takes(int), what a launch asks before it starts anything
    f.argtypes, f.restype = [C.c_int], C.c_bool
    return f(slices)


def test_a_number_of_slices_without_a_kernel_is_told_from_the_others():
    """(Any other number went to the kernel of 32 slices, which reads that many from a workspace that holds fewer.)"""
    assert [s for s in range(-1, 130) if takes(s)] == [2, 4, 8, 16, 32]


def test_families_list_no_other_number():
    rng, listed = random.Random(6), set()
    for M, N, K in [(1, 128, 8192)] + [(rng.randint(1, 900), 8 * rng.randint(1, 300), 8 * rng.randint(32, 2048)) for _ in range(150)]:
        with tf.Problem(M, N, K, trans_b=rng.randint(0, 1) if M > 1 else 0) as p:
            listed |= {v.split_k for v in p.variants() if v.split_k > 1 and not v.fused_reduce}
    assert listed == {2, 4, 8, 16, 32} and all(map(takes, listed))


def test_which_partial_tiles_pass_the_l2s_by():
    """Rows of whole 128-byte lines, and others up to 20 MB. (All did: 928 x 2072 x 11776 with B as [N][K] in eight slices 80.3 us, through the L2s 72.6.)"""
    f = tf.lib()["_ZN2tf14splitk_past_l2Eiii"]          # bool tf::splitk_past_l2(int M, int N, int slices), which a launch goes by
    f.argtypes, f.restype = [C.c_int] * 3, C.c_bool
    assert all(f(*s) for s in [(1024, 1024, 8), (2048, 2048, 8), (928, 2080, 8), (512, 760, 8), (1, 8, 2), (625, 1000, 8), (65, 136, 16)])
    assert not any(f(*s) for s in [(928, 2072, 8), (838, 2040, 4), (804, 2184, 4), (626, 1000, 8), (60000, 30008, 2)])
