"""Cut tiles of the kernels whose waves share K, on the CPU: what a family promises whatever the cut."""
import random

from paper_2512_09196_amd import tf

WHOLE = {b"kshare_32x32x64_k4_s2": 65536, b"kshare_32x64x64_k8_s1": 98304, b"kshare_64x64x64_k8_s1": 131072}


def test_families_with_cut_tiles():
    rng = random.Random(2)
    seen, rows_over_64 = set(), False
    for _ in range(300):
        M, N, K, nk = rng.choice([rng.randint(1, 64), rng.randint(65, 900)]), 8 * rng.randint(1, 900), 8 * rng.randint(8, 900), rng.randint(0, 1)
        with tf.Problem(M, N, K, trans_b=nk) as p:
            fam = p.variants()
        for v in [v for v in fam if v.name.startswith(b"kshare_")]:
            kernel = b"_".join(v.name.split(b"_")[:4])
            cut = v.lds_bytes % 1024 == 64
            seen.add((kernel, cut, v.split_k > 1))
            if cut:                              # one round, no slices, no workspace, within a CU
                assert v.split_k == 1 and v.workspace_bytes == 0 and 0 < v.grid <= 256 and v.lds_bytes <= 160 * 1024
                assert tf.kernel_substr(v).endswith("true")
            else:                                # whole tiles, as they are without cuts
                assert v.lds_bytes == WHOLE[kernel] and v.bm >= 32
                assert v.split_k > 1 or v.grid == -(-M // v.bm) * -(-N // v.bn)
                assert tf.kernel_substr(v).endswith("false")
        rows16 = [i for i, v in enumerate(fam) if v.name.startswith(b"kshare_16x")]
        assert rows16 == list(range(len(fam) - len(rows16), len(fam)))     # behind all others
        small = any(v.kind == tf.TF_KIND_MFMA_LDS_ANY for v in fam)
        assert M <= 64 or not rows16 or small
        rows_over_64 |= M > 64 and bool(rows16)
        assert all((fam[i].kind == tf.TF_KIND_MFMA_LDS_ANY) == small for i in rows16)
    assert {(k, c, s) for k, c, s in seen if k in WHOLE} >= {(k, False, True) for k in WHOLE} | {(k, True, False) for k in list(WHOLE)[1:]}
    assert (b"kshare_32x32x64_k4_s2", True, False) not in seen and rows_over_64
