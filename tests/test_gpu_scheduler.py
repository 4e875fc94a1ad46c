"""GPU tests of the two-stream priority scheduler: every request completes, the
best-effort job keeps making progress and its results stay correct under preemption."""
import numpy as np
import pytest

import tally_inputs as TI

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2410_07381_amd.binding as B
    assert torch.cuda.is_available()
    hi, be = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = B.Context(hi, be)
    yield B, ctx, torch
    ctx.close()


@pytest.mark.parametrize("policy", [0, 1, 2])
@pytest.mark.parametrize("be_form", ["ptb", "ptb_chunk", "sliced"])
def test_colocated_run_completes_and_stays_correct(env, policy, be_form):
    B, ctx, torch = env
    from gpu_util import host
    n = 1 << 24                                   # 4096 reduce blocks
    x = torch.rand(n, device="cuda")
    partial = torch.zeros(n // 4096, device="cuda")
    sx = torch.ones(1 << 16, device="cuda")
    sy = torch.zeros(1 << 16, device="cuda")
    torch.cuda.synchronize()
    be_k = B.reduce_sum(x, partial)
    hi_k = B.saxpy(sx, sy, 1.0)                   # y += x each request
    cfg = {"ptb": (B.CFG_PTB, 512, 1), "ptb_chunk": (B.CFG_PTB, 512, 4),
           "sliced": (B.CFG_SLICED, 512, 1)}[be_form]
    if policy != 0:
        cfg = (B.CFG_NATIVE, 1, 1)
    arrivals = TI.poisson_arrivals_us(5000.0, 200, config_index=2)
    # the first launch of a kernel in a process loads its code (tens of milliseconds, as long
    # as the whole window below): run every form once before the run that is checked
    warm = ctx.sched_run([hi_k], arrivals[:3], [(be_k, cfg)], policy=policy, tail_us=100.0)
    assert len(warm["latency_us"]) == 3
    sy.zero_()
    torch.cuda.synchronize()
    out = ctx.sched_run([hi_k], arrivals, [(be_k, cfg)], policy=policy, tail_us=200.0)
    lat = out["latency_us"]
    assert len(lat) == 200 and (lat > 0).all() and lat.max() < 5e4
    assert out["be_kernels_done"] > 10, (out["be_kernels_done"], out["n_preempts"], out["window_us"],
                                         np.percentile(lat, [50, 99]).tolist(),
                                         out["preempt_latency_us"][:8].tolist(), warm["be_kernels_done"])
    assert out["window_us"] >= arrivals[-1]
    torch.cuda.synchronize()
    assert (host(sy) == 200.0).all()              # every request ran exactly once
    from gpu_util import oracle_block_sums, assert_close_rel
    _, want = oracle_block_sums(host(x))
    assert_close_rel(host(partial), want, 2e-6)
    if policy == 0:
        assert (out["preempt_latency_us"] >= 0).all()


def test_solo_runs(env):
    B, ctx, torch = env
    sx = torch.ones(1 << 16, device="cuda")
    sy = torch.zeros(1 << 16, device="cuda")
    x = torch.rand(1 << 22, device="cuda")
    partial = torch.zeros(1 << 10, device="cuda")
    torch.cuda.synchronize()
    hi = ctx.sched_run([B.saxpy(sx, sy, 1.0)], TI.periodic_arrivals_us(200.0, 50), [])
    assert (hi["latency_us"] > 0).all() and hi["be_kernels_done"] == 0
    be = ctx.sched_run([], [], [(B.reduce_sum(x, partial), (B.CFG_PTB, 256, 1))], tail_us=5000.0)
    assert be["be_kernels_done"] > 5 and be["window_us"] >= 5000.0


def test_several_best_effort_clients_all_progress_and_stay_correct(env):
    """Three best-effort clients (persistent workers, sliced, persistent workers with a
    chunked fetch), each on its own stream pair, against a hi-pri SAXPY: every client
    completes kernels, every request runs once, every output is right."""
    B, ctx, torch = env
    from gpu_util import host
    x0 = torch.rand(1 << 24, device="cuda")
    p0 = torch.zeros(1 << 12, device="cuda")
    x1 = torch.rand(1 << 23, device="cuda")
    p1 = torch.zeros(1 << 11, device="cuda")
    r2 = torch.randn((4096, 1024), device="cuda")
    o2 = torch.zeros_like(r2)
    sx = torch.ones(1 << 16, device="cuda")
    sy = torch.zeros(1 << 16, device="cuda")
    torch.cuda.synchronize()
    items = [(B.reduce_sum(x0, p0), (B.CFG_PTB, 512, 1)),
             (B.reduce_sum(x1, p1), (B.CFG_SLICED, 256, 1)),
             (B.softmax_f32(r2, o2), (B.CFG_PTB, 256, 4))]
    arrivals = TI.poisson_arrivals_us(4000.0, 300, config_index=2)
    out = ctx.sched_run([B.saxpy(sx, sy, 1.0)], arrivals, items, policy=0, tail_us=500.0,
                        be_clients=[1, 1, 1])
    per = out["be_client_kernels_done"]
    assert (per > 3).all(), per
    assert out["be_kernels_done"] == per.sum()
    assert (out["latency_us"] > 0).all() and out["latency_us"].max() < 5e4
    torch.cuda.synchronize()
    assert (host(sy) == 300.0).all()
    from gpu_util import oracle_block_sums, oracle_softmax_rows, assert_close_rel
    for x, p in ((x0, p0), (x1, p1)):
        _, want = oracle_block_sums(host(x))
        assert_close_rel(host(p), want, 2e-6)
    assert_close_rel(host(o2), oracle_softmax_rows(host(r2)), 1e-5, 1e-7)
    # a client may own several items (its step); two clients, 2 + 1 items
    out = ctx.sched_run([B.saxpy(sx, sy, 1.0)], arrivals[:100], items, policy=0, be_clients=[2, 1])
    assert (out["be_client_kernels_done"] > 1).all()


def test_high_priority_kernels_fit_beside_a_paused_gemm_tile(env):
    """The pause inside a GEMM tile only helps high-priority kernels that fit beside the
    paused workgroup (512 registers per lane and the LDS of a compute unit are shared): the
    kernels of the inference-like layer and of the decode step are written to fit."""
    B, ctx, torch = env
    lds_cu = B.device_info()["lds_bytes_per_cu"]
    for be in (B.K_GEMM_BF16, B.K_GEMM_BF16_N128):
        bl, bw, br = ctx.kernel_footprint(be, 0)
        assert bw == 4 and br <= 384
        for hi in (B.K_GEMM_BF16_SMALL, B.K_SOFTMAX_F32, B.K_LAYERNORM_F32, B.K_GEMV_BF16,
                   B.K_ATTN_DECODE_BF16, B.K_SAXPY):
            hl, hw, hr = ctx.kernel_footprint(hi, 1)
            assert br + ((hw + 3) // 4) * hr <= 512, (be, hi, br, hr)
            assert bl + hl <= lds_cu, (be, hi, bl, hl)
            assert bw + hw <= 32
    with pytest.raises(B.TallyError):
        ctx.kernel_footprint(B.K_ATTN_DECODE_BF16, 0)      # no persistent-worker form


def test_measured_matrix_pipe_ceiling_is_plausible(env):
    """Register-only MFMA loop on every compute unit: below the 2.5 PFLOP/s sheet figure
    (the clock is power-managed) and far above anything a mis-sized launch would give."""
    B, ctx, torch = env
    tf = ctx.mfma_ceiling_tflops(5)
    assert 800.0 < tf < 2600.0, tf
    with pytest.raises(B.TallyError):
        ctx.mfma_ceiling_tflops(0)


def test_scheduler_rejects_bad_input(env):
    B, ctx, torch = env
    import ctypes as C
    run = B.SchedRun()
    run.n_arrivals = 3                               # arrivals without kernels
    assert B.lib().tally_sched_run(ctx.h, C.byref(run)) == B.ERR_INVALID_ARG
    run = B.SchedRun()
    run.policy = 7
    assert B.lib().tally_sched_run(ctx.h, C.byref(run)) == B.ERR_INVALID_ARG
    # client item counts that do not add up to the number of items
    x = torch.rand(1 << 20, device="cuda")
    partial = torch.zeros(1 << 8, device="cuda")
    torch.cuda.synchronize()
    k = B.reduce_sum(x, partial)
    for counts in ([2], [1, 1], [0, 1], [1] * 9):
        with pytest.raises(B.TallyError):
            ctx.sched_run([], [], [(k, (B.CFG_PTB, 256, 1))], tail_us=100.0, be_clients=counts)


def test_profile_picks_a_config_under_the_threshold(env):
    B, ctx, torch = env
    x = torch.rand(1 << 26, device="cuda")
    partial = torch.zeros(1 << 14, device="cuda")
    torch.cuda.synchronize()
    k = B.reduce_sum(x, partial)
    assert ctx.lookup_config(k) is None
    cands = [(B.CFG_PTB, 256, 1), (B.CFG_PTB, 1024, 4), (B.CFG_SLICED, 4096, 1),
             (B.CFG_SLICED, 64, 1), (B.CFG_SLICED, 4096, 2)]       # the last: two slices in flight
    from oracle import profiler as OP
    meas, chosen = ctx.profile(k, cands, runs=3, threshold_ms=0.0316)
    assert all(m["latency_ms"] > 0 and m["turnaround_ms"] > 0 for m in meas)
    for m in meas:                                   # Eq. 1 / one-slice time
        if m["kind"] == B.CFG_PTB:
            want = m["latency_ms"] * m["param"] * m["chunk"] / k.total_blocks
        else:
            slices = -(-k.total_blocks // m["param"])
            want = OP.sliced_turnaround_ms(m["latency_ms"] / slices, m["chunk"], n_slices=slices)
        assert abs(m["turnaround_ms"] - want) <= 1e-5 * want + 1e-9
    # the library's choice equals the oracle's selection rule on the same measurements
    o = OP.select_config([{"kind": "ptb" if m["kind"] == 0 else "sliced", "param": m["param"],
                           "latency_ms": m["latency_ms"], "turnaround_ms": m["turnaround_ms"]}
                          for m in meas], 0.0316)
    assert (meas[chosen]["param"], meas[chosen]["kind"]) == (o["param"], 0 if o["kind"] == "ptb" else 1)
    got = ctx.lookup_config(k)
    assert got is not None and got["param"] == meas[chosen]["param"]


@pytest.mark.parametrize("m,n,stages", [(512, 512, 8), (1024, 1024, 4), (1024, 2048, 2)])
def test_turnaround_of_parts_of_blocks(env, m, n, stages):
    """256 workers on 4, 16 and 32 blocks take a part each, all at once: a part lasts as long as the
    kernel (Eq. 1 would say 64, 16 and 8 times as long), and a worker pauses after a round of
    `stages` of 64 k between two looks (at least the 4 steps of 32 k asked for) and the round in
    which the answer is on its way."""
    B, ctx, torch = env
    k = 4096
    A = torch.zeros(1, m, k, dtype=torch.bfloat16, device="cuda")
    Bt = torch.zeros(1, n, k, dtype=torch.bfloat16, device="cuda")
    C = torch.zeros(1, m, n, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, C)
    try:
        meas, _ = ctx.profile(kern, [(B.CFG_PTB, 256, 1)], runs=2)
        assert meas[0]["turnaround_ms"] == pytest.approx(meas[0]["latency_ms"] * 2 * stages / 64, rel=1e-5)
        ctx.set_yield_bound_us(0)
        meas, _ = ctx.profile(kern, [(B.CFG_PTB, 256, 1)], runs=2)
        assert meas[0]["turnaround_ms"] == pytest.approx(meas[0]["latency_ms"], rel=1e-5)
    finally:
        ctx.set_yield_bound_us(1000)
        ctx.profile_reset()


def test_workers_pause_inside_long_blocks_while_preempted(env):
    """A 256x256 tile over K = 32768 lasts about a millisecond.  A pausing preemption request
    raised mid-tile suspends the workers until the pause is ended; the kernel then finishes,
    every block exactly once, with the right numbers."""
    import time
    B, ctx, torch = env
    from gpu_util import host, assert_bf16_close
    from oracle import kernels as OK
    m = n = 1024
    k = 32768
    g = TI.gemm_inputs(m, n, k, scale=1.0 / 128.0, config_index=1)
    A = torch.from_numpy(g["A"].view(np.int16)).cuda()
    Bt = torch.from_numpy(g["Bt"].view(np.int16)).cuda()
    Cd = torch.zeros((1, m, n), dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, Cd)
    assert kern.total_blocks == 16

    def run(pause_s, bound_us):
        ctx.set_yield_bound_us(bound_us)
        t0 = time.perf_counter()
        job = ctx.launch_ptb(kern, 16, coverage=True)
        time.sleep(0.0002)
        if pause_s:
            job.preempt(pause=True)
            time.sleep(pause_s)
            job.end_pause()                      # paused workers go on and finish their tile
        st = job.wait()
        dt = time.perf_counter() - t0
        if pause_s:
            # the preemption itself stood: one tile per worker ran, then every worker left
            assert st == B.JOB_STOPPED or job.progress()[0] == 16
        if st == B.JOB_STOPPED:
            job.resume()
            assert job.wait() == B.JOB_COMPLETE
        rec = job.coverage()
        job.free()
        assert (rec["count"] == 1).all()
        return dt

    run(0.0, 1000)                               # warm-up
    base = run(0.0, 1000)
    paused = run(0.004, 100000)                  # bound 100 ms > the 4 ms pause
    unpaused = run(0.004, 0)                     # pause disabled: request has no effect mid-tile
    ctx.set_yield_bound_us(1000)
    assert paused - base > 0.6 * 0.004, (base, paused)
    assert base < 0.004, base                    # otherwise the test proves nothing
    assert unpaused >= 0.004                     # (the host itself slept that long)
    torch.cuda.synchronize()
    got = host(Cd)
    for bx, by in ((0, 0), (3, 2)):
        a = dict(g, C=np.zeros((1, m, n), np.uint16))
        OK.exec_block("gemm_bf16", (bx, by, 0), (4, 4, 1), a)
        r, c = slice(by * 256, by * 256 + 256), slice(bx * 256, bx * 256 + 256)
        assert_bf16_close(got[0, r, c], a["C"][0, r, c])


@pytest.mark.parametrize("m,n,k,n128", [
    (256, 512, 1 << 18, False), (512, 1024, 1 << 17, False), (768, 1024, 1 << 17, False), (1024, 2048, 1 << 16, False),
    (2048, 2048, 1 << 16, False), (512, 1024, 1 << 17, True), (768, 1024, (1 << 17) + 32, True), (1024, 2048, 1 << 16, True),
    (2048, 2048, (1 << 16) + 96, True)])
def test_workers_on_parts_of_blocks_pause_as_well(env, m, n, k, n128):
    """Fewer blocks than workers over a long K, handed out in parts of 32x32, and of 32x64, 64x64, 128x64
    and 128x128 (for blocks of 256 columns and of 128): a pausing request raised mid-part suspends the
    workers until the pause is ended; the numbers are those of an undisturbed run."""
    import time
    B, ctx, torch = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    A = torch.randn(1, m, k, device="cuda", generator=gen).to(torch.bfloat16)
    Bt = torch.randn(1, n, k, device="cuda", generator=gen).to(torch.bfloat16)
    C = torch.empty(1, m, n, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C, n128=n128)

    def run(pause_s):
        C.fill_(float("nan"))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        job = ctx.launch_ptb(kern, 256, coverage=True)
        t1 = t0 + 0.0001
        while time.perf_counter() < t1:
            pass
        if pause_s:
            job.preempt(pause=True)
            time.sleep(pause_s)
            job.pump()
            assert job.progress()[2] == B.JOB_RUNNING
            job.end_pause()
        st = job.wait()
        dt = time.perf_counter() - t0
        assert st == B.JOB_COMPLETE
        assert (job.coverage()["count"] == 1).all()
        job.free()
        torch.cuda.synchronize()
        return dt, C.view(torch.int16).clone()

    ctx.set_yield_bound_us(100000)
    try:
        run(0.0)
        base, want = run(0.0)
        assert 0.0003 < base < 0.004, base           # long enough to be met mid-part, shorter than the pause
        paused, got = run(0.004)
    finally:
        ctx.set_yield_bound_us(1000)
    assert paused > 0.004 and torch.equal(got, want)


@pytest.mark.parametrize("n128,k,every,chunk", [(False, (1 << 16) + 32, 1, 1), (True, (1 << 16) + 32, 4, 4),
                                                (False, 1 << 16, 64, 4)])
def test_large_tiles_pause_on_the_answer_of_an_earlier_stage(env, n128, k, every, chunk):
    """Tiles of 256 rows ask for the pause word among their operands' loads and act on the answer a
    stage later: with looks every stage, every second and every 32nd, a last stage that is half
    full, and blocks that follow another one of the same fetch.  A pause met mid-tile holds the workers
    until it is ended, and the numbers are those of the original form."""
    import time
    B, ctx, torch = env
    m, n = 512, 1024
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k + every)
    A = torch.randn(1, m, k, device="cuda", generator=gen).to(torch.bfloat16)
    Bt = torch.randn(1, n, k, device="cuda", generator=gen).to(torch.bfloat16)
    C = torch.empty(1, m, n, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C, n128=n128)
    torch.cuda.synchronize()
    ctx.launch_native(kern)
    torch.cuda.synchronize()
    want = C.view(torch.int16).clone()
    ctx.set_yield_bound_us(100000)
    ctx.set_yield_every(every)
    try:
        for pause_s in (0.0, 0.004):
            C.fill_(float("nan"))
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            job = ctx.launch_ptb(kern, kern.total_blocks // chunk, chunk=chunk, coverage=True)
            while time.perf_counter() < t0 + 0.0003:
                pass
            if pause_s:
                job.preempt(pause=True)
                time.sleep(pause_s)
                job.pump()
                assert job.progress()[2] == B.JOB_RUNNING
                job.end_pause()
            assert job.wait() == B.JOB_COMPLETE      # (every block had been fetched)
            assert (job.coverage()["count"] == 1).all()
            job.free()
            assert torch.equal(C.view(torch.int16), want)
    finally:
        ctx.set_yield_bound_us(1000)
        ctx.set_yield_every(4)


@pytest.mark.parametrize("n128,k,every", [(False, 32 * 992, 1024), (True, 32 * 991, 1024), (False, 32 * 1000, 512)])
def test_large_tiles_look_before_their_epilogue_however_rarely_they_are_asked_to(env, n128, k, every):
    """Looks further apart than a tile is long, or whose last one lies far before its end: a pause asked
    for mid-tile is found before the output is written, and holds the workers until it is ended."""
    import time
    B, ctx, torch = env
    m, n = 512, 1024
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k + every)
    A = torch.randn(1, m, k, device="cuda", generator=gen).to(torch.bfloat16)
    Bt = torch.randn(1, n, k, device="cuda", generator=gen).to(torch.bfloat16)
    C = torch.empty(1, m, n, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C, n128=n128)
    torch.cuda.synchronize()
    ctx.launch_native(kern)
    torch.cuda.synchronize()
    want = C.view(torch.int16).clone()
    ctx.set_yield_bound_us(100000)
    ctx.set_yield_every(every)
    try:
        spans = []
        for share in (0.0, 0.0, 0.3, 0.7):                # of an undisturbed run: before and after its middle
            C.fill_(float("nan"))
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            job = ctx.launch_ptb(kern, kern.total_blocks, coverage=True)
            if share:
                while time.perf_counter() < t0 + share * spans[-1]:
                    pass
                job.preempt(pause=True)
                time.sleep(0.004)
                job.pump()
                assert job.progress()[2] == B.JOB_RUNNING
                assert torch.isnan(C).all()
                job.end_pause()
            assert job.wait() == B.JOB_COMPLETE
            if not share:
                spans.append(time.perf_counter() - t0)
            assert (job.coverage()["count"] == 1).all()
            job.free()
            assert torch.equal(C.view(torch.int16), want)
        assert spans[-1] < 0.002                          # (otherwise the pauses prove nothing)
    finally:
        ctx.set_yield_bound_us(1000)
        ctx.set_yield_every(4)
