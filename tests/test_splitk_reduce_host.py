"""The second kernel of sliced products has an instance for each number of slices: the ones there are, and the ones families list."""
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
