"""Parity at the full sizes of the five workloads, in the launch configuration the benchmark
times: every element of the output against the whole oracle, and the GPU-driven variant loop."""
import numpy as np
import pytest

from oracle import gemm_oracle as orc
from paper_2512_09196_amd import tf
from paper_2512_09196_amd import workloads as wl

import gpu_util as gu

pytestmark = pytest.mark.gpu

_cache = {}


def inputs(name):
    if name not in _cache:
        _cache.clear()                      # one full-size workload in host memory at a time
        _cache[name] = wl.make_inputs(wl.WORKLOADS[name])
    return _cache[name]


def sample_positions(M, N, n_random=1500, seed=0):
    rng = np.random.default_rng(seed)
    edges_m = sorted({m for m in (0, 1, 31, 32, 127, 128, 255, 256, M // 2, M - 2, M - 1) if 0 <= m < M})
    edges_n = sorted({n for n in (0, 7, 8, 63, 64, 127, 128, 255, 256, N // 2, N - 9, N - 8, N - 1) if 0 <= n < N})
    rows = [m for m in edges_m for _ in edges_n] + list(rng.integers(0, M, n_random))
    cols = [n for _ in edges_m for n in edges_n] + list(rng.integers(0, N, n_random))
    return np.array(rows, np.int32), np.array(cols, np.int32)


def tile_shape(v):
    return (v.kind, v.bm, v.bn, v.bk, v.waves_m, v.waves_n, v.waves_k, v.stages, v.direct_to_lds, v.a_bypass_lds, v.bn_tail,
            v.stream_k)


@pytest.mark.parametrize("name,b_as_nk", [("C2", False), ("C3", False), ("C4", False), ("C5", False), ("C2", True), ("C4", True)])
def test_full_size_every_element_against_the_whole_oracle(name, b_as_nk):
    """Every element of the output at the full size of the workload, in the launch configuration the benchmark
    times, against the whole oracle (run unchanged on disjoint row blocks from the host's cores): the strict
    a-priori bound for the bf16 epilogue, the summation bound for the fp32 pre-activation. C2, C4, C5: every
    variant; C3 (45 M outputs, a launch of the baseline kernel takes 0.1 s): the kernel the loop selects, one
    variant per compiled tile kernel, and the baseline. b_as_nk: the same numbers with B handed over as [N][K], against
    the oracle written for that layout (every variant: the kernels that stage B as it lies, the transposing pass ahead
    of an ordinary kernel, the unstaged kernels)."""
    torch = gu.torch_mod()
    w = wl.WORKLOADS[name]
    A, B, bias = inputs(name)
    if b_as_nk:
        B = np.ascontiguousarray(B.T)
    y, z, s = gu.oracle_parallel(A, B, bias, trans_b=b_as_nk)
    print(name, "oracle done", flush=True)
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
    # the bounds, evaluated once in float64 on the device (test arithmetic, not the library's)
    ty, tz, ts = (torch.from_numpy(x).cuda() for x in (y, z, s))
    g = gu.gamma(w.K + 1)
    strict = 2.0 ** -8 * ty.abs() + 1.13 * 2.0 * g * ts + 1e-6 * (1.0 + tz.abs())
    official = 1e-2 * (1.0 + ty.abs())
    preact = 2.0 * g * ts + 2.0 ** -23 * tz.abs() + 1e-30
    del ts
    checked = 0
    for epi, f32 in ((tf.TF_EPI_BIAS_GELU_ERF, False), (tf.TF_EPI_NONE_F32, True)):
        Y = torch.empty((w.M, w.N), dtype=torch.float32 if f32 else torch.bfloat16, device="cuda")
        with tf.Problem(w.M, w.N, w.K, epi=epi, trans_b=1 if b_as_nk else 0) as prob:
            vs = prob.variants()
            if b_as_nk:
                assert any(v.trans_b for v in vs) and any(b"_pretransB_" in v.name for v in vs)
            if name == "C3":
                best, rep, log = prob.tune(dA, dB, dbias, Y)
                todo, seen = [vs[best]], {tile_shape(vs[best])}
                for v in vs:
                    if v.kind == tf.TF_KIND_MFMA_DIRECT or (v.kind == tf.TF_KIND_NAIVE and f32) or tile_shape(v) in seen:
                        continue
                    seen.add(tile_shape(v))
                    todo.append(v)
            else:
                # the slow unstaged kernels only once per workload (bf16 epilogue), every tile kernel always
                todo = [v for v in vs if v.kind in (tf.TF_KIND_MFMA_LDS, tf.TF_KIND_MFMA_STREAM) or not f32]
            assert len(todo) >= 3
            for v in todo:
                print(name, "epi", epi, v.name.decode(), flush=True)
                Y.fill_(float("nan"))
                prob.run(v.id, dA, dB, dbias, Y)
                torch.cuda.synchronize()
                got = Y.double()
                assert not torch.isnan(got).any().item(), v.name.decode() + " left NaN / unwritten elements"
                if f32:
                    bad = ((got - tz).abs() > preact).sum().item()
                    assert bad == 0, "%s: %d pre-activations outside the summation bound" % (v.name.decode(), bad)
                else:
                    err = (got - ty).abs()
                    assert (err > official).sum().item() == 0, v.name.decode()
                    bad = (err > strict).sum().item()
                    assert bad == 0, "%s: %d elements outside the strict bound" % (v.name.decode(), bad)
                    del err
                del got
                checked += 1
            prob.workspace_status()
        del Y
    assert checked >= 6


def test_tune_attaches_the_profilers_counters_to_its_rounds():
    """The loop on C3 with a profiler pass handed in (tests/golden/rocprofv3_pmc_sq_loop_C3.csv: one dispatch each of
    the baseline kernel and of four tile kernels): the reports of the rounds whose kernel the file holds carry its
    counters when the hint is taken, the others do not."""
    import os
    torch = gu.torch_mod()
    w = wl.WORKLOADS["C3"]
    A, B, bias = inputs("C3")
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
    Y = torch.empty((w.M, w.N), dtype=torch.bfloat16, device="cuda")
    fixture = os.path.join(os.path.dirname(__file__), "golden", "rocprofv3_pmc_sq_loop_C3.csv")
    held = ("tf_gemm_naive_kernel", "tf_gemm_mixed_kernel<tf::LdsCfg<256, 256, 64, 2, 4, 2,", "tf_gemm_lds_kernel<tf::LdsCfg<256, 256, 32, 2, 4, 4,",
            "tf_gemm_lds_kernel<tf::LdsCfg<256, 128, 64, 4, 2, 3,", "tf_gemm_lds_kernel<tf::LdsCfg<256, 256, 64, 2, 4, 2,")
    with tf.Problem(w.M, w.N, w.K) as prob:
        vs = prob.variants()
        prob.set_counter_files([fixture])
        best, rep, log = prob.tune(dA, dB, dbias, Y)
        assert log[0].variant_id == 0 and log[0].have_counters == 1 and log[0].mfma_busy_pct == 0.0
        seen = 0
        for r in log[1:]:
            name = tf.kernel_substr(vs[r.variant_id])
            in_file = any(name.startswith(h) for h in held)
            print(vs[r.variant_id].name.decode(), "counters" if r.have_counters else "-", "%.1f" % r.mfma_busy_pct, flush=True)
            assert r.have_counters == (1 if in_file else 0)
            if in_file:
                seen += 1
                assert 40.0 < r.mfma_busy_pct < 75.0 and r.achieved_occupancy_pct > 15.0
                assert r.bottleneck in (tf.TF_BN_LATENCY, tf.TF_BN_OCCUPANCY)     # pipes 50-65 % busy: not "MFMA-bound"
        assert seen >= 1          # the first proposal on this shape is a large-tile kernel
        prob.set_counter_files([])
        best2, rep2, log2 = prob.tune(dA, dB, dbias, Y)
        assert all(r.have_counters == 0 for r in log2)


def test_tune_on_gpu_c1_and_c2():
    torch = gu.torch_mod()
    for name in ("C1", "C2"):
        w = wl.WORKLOADS[name]
        A, B, bias = inputs(name)
        dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
        Y = torch.empty((w.M, w.N), dtype=torch.bfloat16, device="cuda")
        rows, cols = sample_positions(w.M, w.N, n_random=300, seed=1)
        y, z, s = orc.gemm_bias_gelu_at(A, B, bias, rows, cols)
        r_t, c_t = torch.from_numpy(rows.astype(np.int64)).cuda(), torch.from_numpy(cols.astype(np.int64)).cuda()
        checked = []

        def gate(vid):
            got = Y.float()[r_t, c_t].double().cpu().numpy()
            checked.append(vid)
            return bool(np.all(np.abs(got - y) <= gu.strict_bound(y, z, s, w.K)))

        with tf.Problem(w.M, w.N, w.K) as prob:
            for parity in (None, gate):
                best, rep, log = prob.tune(dA, dB, dbias, Y, parity=parity)
                print(name, "tune ->", prob.variants()[best].name.decode(), "%.2f us" % rep.t_med_us,
                      "rounds", len(log) - 1, flush=True)
                assert log[0].variant_id == 0 and 1 <= len(log) - 1 <= 8
                assert len({r.variant_id for r in log}) == len(log)
                assert best != 0, "no variant beat the naive kernel"
                assert rep.parity_ok == 1 and rep.status == 0
                assert log[0].t_med_us / rep.t_med_us >= 1.05
                # the log's result by the Arbiter's rule: within 1.02 (later_accept_gain) of the fastest candidate whose
                # times are steady; one whose spread is above robust_spread is left however fast its median
                th = tf.theta_default()
                assert best == gu.arbitrated(log, th).variant_id and rep.t_med_us == gu.arbitrated(log, th).t_med_us
                steady = [r.t_med_us for r in log if r.status == 0 and r.parity_ok and (r.t_med_us - r.t_min_us) / r.t_med_us <= th.robust_spread]
                assert rep.t_med_us <= min(steady) * th.later_accept_gain
                # Y holds the selected kernel's output
                got = Y.float()[r_t, c_t].double().cpu().numpy()
                assert np.all(np.abs(got - y) <= gu.strict_bound(y, z, s, w.K))
            assert checked and checked[0] == 0


def test_profile_report_fields():
    torch = gu.torch_mod()
    w = wl.WORKLOADS["C2"]
    A, B, bias = inputs("C2")
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
    Y = torch.empty((w.M, w.N), dtype=torch.bfloat16, device="cuda")
    hw = tf.hw_query(0)
    assert hw.cus == 256 and hw.wave_size == 64 and hw.lds_bytes_per_cu == 160 * 1024
    with tf.Problem(w.M, w.N, w.K) as prob:
        v = [v for v in prob.variants() if v.kind == tf.TF_KIND_MFMA_LDS and v.bm == 128 and v.bn == 128][0]
        r = prob.profile(v.id, dA, dB, dbias, Y, warmup=3, iters=5)
        assert r.status == 0 and r.warmup == 3 and r.iters == 5 and r.launches_per_iter >= 1
        assert 0 < r.t_min_us <= r.t_med_us <= r.t_max_us and r.t_min_us <= r.t_mean_us <= r.t_max_us
        assert r.tflops == pytest.approx(w.flops / r.t_med_us * 1e-6, rel=1e-9)
        assert r.gbytes_per_s == pytest.approx(w.algorithmic_bytes / r.t_med_us * 1e-3, rel=1e-9)
        assert r.pct_mfma_peak == pytest.approx(100 * r.tflops / hw.bf16_tflops_peak, rel=1e-9)
        assert r.arithmetic_intensity == pytest.approx(w.flops / w.algorithmic_bytes, rel=1e-9)
        assert r.grid == v.grid and 1 <= r.waves_per_simd <= 8 and r.vgprs > 0 and r.lds_bytes >= v.lds_bytes
        assert 0 < r.grid_fill <= 1.0 and r.spill_bytes == 0
        assert r.tflops > 100.0       # an MFMA kernel on this shape is far above any VALU rate


def test_measured_peaks_are_plausible():
    mfma, hbm = tf.hw_measure(0)
    print("measured: %.0f TFLOP/s bf16 MFMA, %.0f GB/s HBM read" % (mfma, hbm), flush=True)
    # below the published peaks, and not absurdly so
    assert 800.0 < mfma < 2516.6 and 3000.0 < hbm < 8000.0


def test_no_kernel_reserves_much_scratch_memory():
    # register spills outside the hot loop still make every wave reserve scratch memory, which slows
    # each launch: the tile kernels must stay (almost) spill free
    torch = gu.torch_mod()
    M, N, K = 1024, 1024, 512
    A, B, bias = wl.make_custom(M, N, K, seed=3)
    dA, dB, dbias = gu.to_dev(A), gu.to_dev(B), gu.to_dev(bias)
    Y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    seen = {}
    with tf.Problem(M, N, K) as prob:
        for v in prob.variants():
            key = (v.kind, v.bm, v.bn, v.waves_m, v.waves_n, v.waves_k, v.stages, v.direct_to_lds, v.a_bypass_lds)
            if v.kind not in (tf.TF_KIND_MFMA_LDS, tf.TF_KIND_MFMA_STREAM) or key in seen or v.split_k > 1:
                continue
            r = prob.profile(v.id, dA, dB, dbias, Y, warmup=0, iters=1, launches_per_iter=1)
            seen[key] = r.spill_bytes
            assert r.spill_bytes == 0, "%s reserves %d bytes of scratch per lane" % (v.name.decode(), r.spill_bytes)
    assert len(seen) >= 15
