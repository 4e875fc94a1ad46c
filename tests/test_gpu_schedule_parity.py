"""GPU parity: block coverage and indexing of the three launch forms against the oracle,
bit for bit, plus SAXPY / reduction outputs; all calls go through the C ABI."""
import time

import numpy as np
import pytest

import tally_inputs as TI
from oracle import kernels as OK
from oracle import schedules as OS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2410_07381_amd.binding as B
    assert torch.cuda.is_available(), "these tests need the MI355X"
    hi, be = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = B.Context(hi, be)
    yield B, ctx, torch
    ctx.close()


def _saxpy_oracle(base, runner):
    a = dict(base, y=base["y"].copy())
    cov = runner(a)
    return a["y"], cov


# ------------------------------------------------------------------ configuration 0
def test_cfg0_saxpy_ptb_three_preemptions(env):
    """N = 2^20, grid 4096 x 256, 256 workers, 3 preemptions at seeded counter values,
    each followed by a resume."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    base = TI.saxpy_inputs(n=1 << 20, config_index=0)
    grid = OK.grid_of("saxpy", base)
    assert grid == (4096, 1, 1)
    pts = TI.preempt_points(4096, 3, config_index=0)
    assert len(pts) == 3 and all(1 <= p <= 4095 for p in pts)

    x, y = dev(base["x"]), dev(base["y"])
    torch.cuda.synchronize()
    k = B.saxpy(x, y, base["a"])
    assert k.grid == grid
    job = ctx.launch_ptb(k, 256, coverage=True, stop_at=pts[0])
    seen = []
    for nxt in pts[1:] + [None]:
        st = job.wait()
        done, total, _ = job.progress()
        seen.append(done)
        assert st == B.JOB_STOPPED and total == 4096
        job.resume(stop_at=nxt)
    assert job.wait() == B.JOB_COMPLETE
    assert seen == pts and job.progress()[0] == 4096
    rec = job.coverage()
    job.free()

    want_y, (cov, log) = _saxpy_oracle(
        base, lambda a: OS.run_ptb("saxpy", grid, a, 256, preempt_points=pts, seed=0))
    assert log == pts + [4096]
    assert_cover_equal(rec, cov)
    assert (rec["worker"] < 256).all()
    assert_close_rel(host(y), want_y, 1e-6)


@pytest.mark.parametrize("n,workers,chunk,pts", [
    (5000, 4, 1, [3, 11]),          # ragged last block
    (5000, 7, 3, [1, 19]),          # chunked fetch, stop inside a chunk
    (256 * 33, 64, 1, [10]),        # more workers than blocks
    (1000, 2, 1, []),
])
def test_saxpy_ptb_small(env, n, workers, chunk, pts):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    base = TI.saxpy_inputs(n=n, config_index=0)
    grid = OK.grid_of("saxpy", base)
    x, y = dev(base["x"]), dev(base["y"])
    torch.cuda.synchronize()
    k = B.saxpy(x, y, base["a"])
    stops = pts + [None]
    job = ctx.launch_ptb(k, workers, chunk=chunk, coverage=True, stop_at=stops[0])
    for nxt in stops[1:]:
        assert job.wait() == B.JOB_STOPPED
        job.resume(stop_at=nxt)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    want_y, (cov, _) = _saxpy_oracle(
        base, lambda a: OS.run_ptb("saxpy", grid, a, workers, preempt_points=pts, seed=1))
    assert_cover_equal(rec, cov)
    assert_close_rel(host(y), want_y, 1e-6)


def test_saxpy_up_to_the_largest_count(env):
    """2^32 - 1 elements as workers that take several blocks per fetch: the element after the last
    one has no 32-bit index.  fma(1.5, 1, 2) = 3.5 everywhere, exactly."""
    B, ctx, torch = env
    n = 2**32 - 1
    x, y = torch.ones(n, device="cuda"), torch.full((n,), 2.0, device="cuda")
    torch.cuda.synchronize()
    k = B.saxpy(x, y, 1.5)
    assert k.total_blocks == 2**24
    job = ctx.launch_ptb(k, 512, chunk=1024)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    torch.cuda.synchronize()
    assert bool((y == 3.5).all())
    k = x = y = None
    torch.cuda.empty_cache()


def test_degenerate_schedules(env):
    """A zero-block segment (preempted before the first fetch), one worker, a chunk and a
    slice larger than the whole grid, an empty input."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    base = TI.saxpy_inputs(n=256 * 7 + 3, config_index=0)          # 8 blocks
    grid = OK.grid_of("saxpy", base)
    want_y, (cov0, _) = _saxpy_oracle(base, lambda a: OS.run_ptb("saxpy", grid, a, 1, preempt_points=[], seed=0))

    def fresh():
        x, y = dev(base["x"]), dev(base["y"])
        torch.cuda.synchronize()
        return B.saxpy(x, y, base["a"]), y

    k, y = fresh()                                                  # stop before anything ran
    job = ctx.launch_ptb(k, 4, coverage=True, stop_at=0)
    assert job.wait() == B.JOB_STOPPED and job.progress()[0] == 0
    assert (job.coverage()["count"] == 0).all()
    job.resume()
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert (rec["count"] == 1).all() and (rec["segment"] == 1).all()
    assert_close_rel(host(y), want_y, 1e-6)

    k, y = fresh()                                                  # one worker, in order
    job = ctx.launch_ptb(k, 1, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert_cover_equal(rec, cov0)
    assert (rec["worker"] == 0).all()
    assert_close_rel(host(y), want_y, 1e-6)

    k, y = fresh()                                                  # one fetch takes the grid
    job = ctx.launch_ptb(k, 3, chunk=1000, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert (rec["count"] == 1).all() and len(set(rec["worker"].tolist())) == 1
    assert_close_rel(host(y), want_y, 1e-6)

    k, y = fresh()                                                  # one slice takes the grid
    job = ctx.launch_sliced(k, 1000, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    assert (job.coverage()["count"] == 1).all()
    job.free()
    assert_close_rel(host(y), want_y, 1e-6)

    empty = torch.zeros(0, device="cuda")
    with pytest.raises(B.TallyError):
        B.saxpy(empty, empty, 1.0)


def test_saxpy_native_and_sliced(env):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    base = TI.saxpy_inputs(n=256 * 16, config_index=0)        # the paper's 16-block example
    grid = OK.grid_of("saxpy", base)
    x, y = dev(base["x"]), dev(base["y"])
    y2 = dev(base["y"])
    torch.cuda.synchronize()
    job = ctx.launch_sliced(B.saxpy(x, y, base["a"]), 4, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    want_y, (cov, _) = _saxpy_oracle(base, lambda a: OS.run_sliced("saxpy", grid, a, 4))
    assert_cover_equal(rec, cov)
    assert rec["bx"][4:8].tolist() == [4, 5, 6, 7]             # sub-kernel 2: offset 4
    assert_close_rel(host(y), want_y, 1e-6)
    ctx.launch_native(B.saxpy(x, y2, base["a"]))
    torch.cuda.synchronize()
    assert (host(y2).view(np.uint32) == host(y).view(np.uint32)).all()


@pytest.mark.parametrize("in_flight", [2, 3, 8])
def test_sliced_several_slices_in_flight(env, in_flight):
    """More than one sub-kernel enqueued at a time (the paper enqueues one): coverage and
    results are those of the one-at-a-time schedule, and a preemption drains every slice
    that was already enqueued before the job reports STOPPED."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    base = TI.saxpy_inputs(n=256 * 33 + 17, config_index=0)        # 34 blocks, ragged tail
    grid = OK.grid_of("saxpy", base)
    x, y = dev(base["x"]), dev(base["y"])
    torch.cuda.synchronize()
    job = ctx.launch_sliced(B.saxpy(x, y, base["a"]), 5, max_in_flight=in_flight, coverage=True)
    job.preempt()
    all_enqueued = 5 * in_flight >= 34                             # then nothing is left to stop
    assert job.wait() == (B.JOB_COMPLETE if all_enqueued else B.JOB_STOPPED)
    done = job.progress()[0]
    assert done == min(5 * in_flight, 34)                          # exactly the enqueued slices
    job.resume()                                                   # no-op on a complete job
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    first = min(in_flight, 7)                                      # slices before the preemption
    want_y, (cov, resumes) = _saxpy_oracle(
        base, lambda a: OS.run_sliced("saxpy", grid, a, 5, preempt_after_slices=[first]))
    assert resumes == ([] if all_enqueued else [done])
    assert_cover_equal(rec, cov)
    assert_close_rel(host(y), want_y, 1e-6)


def test_sliced_preempt_and_resume_segments(env):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    base = TI.saxpy_inputs(n=256 * 10, config_index=0)
    grid = OK.grid_of("saxpy", base)
    x, y = dev(base["x"]), dev(base["y"])
    torch.cuda.synchronize()
    job = ctx.launch_sliced(B.saxpy(x, y, base["a"]), 4, coverage=True)
    job.preempt()                        # first slice is already enqueued and will finish
    assert job.wait() == B.JOB_STOPPED
    assert job.progress()[0] == 4
    job.preempt()                        # no-op on a stopped job
    job.resume()
    job.preempt()
    assert job.wait() == B.JOB_STOPPED and job.progress()[0] == 8
    job.resume()
    assert job.wait() == B.JOB_COMPLETE
    job.resume()                         # no-op on a complete job
    rec = job.coverage()
    job.free()
    want_y, (cov, resumes) = _saxpy_oracle(
        base, lambda a: OS.run_sliced("saxpy", grid, a, 4, preempt_after_slices=[1, 2]))
    assert resumes == [4, 8]
    assert_cover_equal(rec, cov)
    assert_close_rel(host(y), want_y, 1e-6)


# ------------------------------------------------------------------ multi-dimensional grid
def test_ptb_three_dimensional_grid_mapping(env):
    """Batched 32-wide GEMM tiles give a (gx, gy, gz) grid: the rebuilt block indices
    must follow x-fastest order in both transformed forms."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_bf16_close
    g = TI.gemm_inputs(m=150, n=200, k=64, config_index=1, batch=3)
    a = dict(g, C=np.zeros((3, 150, 200), np.uint16))
    grid = OK.grid_of("gemm_bf16_small", a)
    assert grid == (7, 5, 3)
    A, Bt = dev(g["A"]), dev(g["Bt"])
    Cp, Cs = dev(a["C"]), dev(a["C"])
    torch.cuda.synchronize()
    job = ctx.launch_ptb(B.gemm_bf16(A, Bt, Cp, small=True), 5, coverage=True, stop_at=17)
    assert job.wait() == B.JOB_STOPPED
    job.resume()
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    cov, _ = OS.run_ptb("gemm_bf16_small", grid, a, 5, preempt_points=[17], seed=4)
    assert_cover_equal(rec, cov)
    assert_bf16_close(host(Cp), a["C"])
    job = ctx.launch_sliced(B.gemm_bf16(A, Bt, Cs, small=True), 7, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    b = dict(g, C=np.zeros((3, 150, 200), np.uint16))
    cov, _ = OS.run_sliced("gemm_bf16_small", grid, b, 7)
    assert_cover_equal(rec, cov)
    assert (host(Cs) == host(Cp)).all()


# ------------------------------------------------------------------ asynchronous preemption
@pytest.mark.parametrize("workers,chunk", [(256, 1), (512, 8)])
def test_async_flag_preemption_prefix_and_exactly_once(env, workers, chunk):
    """Raise the real flag from the host while workers run.  The observed progress value is
    fed to the oracle as its preemption point; at the drain exactly the prefix has run."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal
    n = 1 << 28
    x = torch.rand(n, device="cuda")
    nb = n // 4096
    partial = torch.zeros(nb, device="cuda")
    torch.cuda.synchronize()
    k = B.reduce_sum(x, partial)
    pts = []
    job = ctx.launch_ptb(k, workers, chunk=chunk, coverage=True)
    for attempt in range(3):
        time.sleep(0.0001 if chunk == 1 else 0.00004)
        job.preempt()
        st = job.wait()
        done, total, _ = job.progress()
        if st == B.JOB_COMPLETE:
            break
        assert st == B.JOB_STOPPED and 0 <= done < total and done % chunk == 0
        lat = job.preempt_latency_us()
        assert 0 < lat < 5e4
        rec = job.coverage()
        assert (rec["count"][:done] == 1).all() and (rec["count"][done:] == 0).all()
        pts.append(done)
        job.resume()
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert len(pts) >= 1, "the kernel finished before any preemption landed"
    cov, log = OS.run_ptb(None, (nb, 1, 1), {}, workers, preempt_points=pts, seed=7, chunk=chunk)
    assert log == pts + [nb]
    assert_cover_equal(rec, cov)
    from gpu_util import oracle_block_sums, assert_close_rel
    sample = [0, nb - 1] + [int(v) for v in np.random.default_rng(3).integers(nb, size=1500)]
    idx, want = oracle_block_sums(host(x), sample)
    assert_close_rel(host(partial)[idx], want, 2e-6)


def test_many_preemptions_in_a_row_keep_exactly_once(env):
    """Sixty asynchronous preempt / drain / resume cycles on one job: the task counter is
    never reset (the base moves after every drain, the word accumulates every failed fetch
    and 2^31 per request, wrapping several times), yet every block runs exactly once, each
    drain leaves a prefix, and the segments are the ones the oracle gets from the same
    progress values."""
    B, ctx, torch = env
    from gpu_util import host, assert_cover_equal, oracle_block_sums, assert_close_rel
    n = 1 << 28
    x = torch.rand(n, device="cuda")
    nb = n // 4096
    partial = torch.zeros(nb, device="cuda")
    torch.cuda.synchronize()
    k = B.reduce_sum(x, partial)
    workers, chunk = 256, 4                      # slow enough (about 0.3 ms alone) to be caught
    pts = []
    job = ctx.launch_ptb(k, workers, chunk=chunk, coverage=True)
    for cycle in range(60):
        job.preempt()
        st = job.wait()
        done = job.progress()[0]
        if st == B.JOB_COMPLETE:
            break
        assert st == B.JOB_STOPPED and done % chunk == 0 and (not pts or done >= pts[-1])
        pts.append(done)
        job.resume()
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert len(pts) >= 10, pts
    assert (rec["count"] == 1).all()
    # (a request that found nothing new to stop repeats the progress value: an empty segment,
    # on the GPU and in the oracle alike)
    cov, log = OS.run_ptb(None, (nb, 1, 1), {}, workers, preempt_points=pts, seed=9, chunk=chunk)
    assert log == pts + [nb]
    assert_cover_equal(rec, cov)
    sample = [0, nb - 1] + [int(v) for v in np.random.default_rng(5).integers(nb, size=500)]
    idx, want = oracle_block_sums(host(x), sample)
    assert_close_rel(host(partial)[idx], want, 2e-6)


def test_preemption_reaches_workers_that_fill_the_gpu(env):
    """The largest worker count of the softmax kernel leaves no register free on any compute
    unit: the flag must still reach the workers (the relay is resident before them) and the
    job must drain long before it would have finished."""
    import time
    B, ctx, torch = env
    from gpu_util import host
    x = torch.randn((65536, 2048), device="cuda")
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    k = B.softmax_f32(x, y)
    w = ctx.max_workers(k)
    job = ctx.launch_ptb(k, w, chunk=2)
    t0 = time.perf_counter()
    while job.progress()[0] < 64 and time.perf_counter() - t0 < 1.0:
        pass
    job.preempt()
    assert job.wait() == B.JOB_STOPPED
    done, total, _ = job.progress()
    assert 0 < done < total // 2, (done, total)          # the whole kernel takes ~1.5 ms
    job.resume()
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    torch.cuda.synchronize()
    from gpu_util import oracle_softmax_rows, assert_close_rel
    assert_close_rel(host(y)[::4099], oracle_softmax_rows(host(x)[::4099]), 1e-5, 1e-7)


@pytest.mark.parametrize("op", ["saxpy", "softmax"])
def test_preemption_reaches_workers_right_behind_another_job(env, op):
    """The same where the job before has only just drained: the scheduler frees it and launches the
    next one on the word that its last worker sent, when its relay still has to look once more, and
    to report.  The second job's relay has to be on the GPU before its workers all the same."""
    B, ctx, torch = env
    if op == "saxpy":
        x, y = torch.zeros(1 << 26, device="cuda"), torch.zeros(1 << 26, device="cuda")
        long = B.saxpy(x, y, 1.0)                         # 2^18 blocks one by one: 3 ms
        short = B.saxpy(x[:1 << 20], y[:1 << 20], 1.0)
    else:
        x = torch.zeros((65536, 2048), device="cuda")
        long = B.softmax_f32(x, x)
        short = B.softmax_f32(x[:4096], x[:4096])
    u, v = torch.zeros(64, device="cuda"), torch.zeros(64, device="cuda")
    request = [B.saxpy(u, v, 1.0)]
    torch.cuda.synchronize()
    cfg = (B.CFG_PTB, ctx.max_workers(long), 1)
    s = ctx.scheduler()
    try:
        for rep in range(40):
            s.submit_be(short, cfg)
            s.submit_be(long, cfg)
            while s.stats()["be_kernels_done"] < 2 * rep + 1:
                s.poll()
            t0 = time.perf_counter()
            while time.perf_counter() - t0 < 1e-4:        # (the long job is on the GPU by now)
                pass
            s.submit_hi(request)
            while s.poll():
                pass
            while s.stats()["be_kernels_done"] < 2 * rep + 2:
                s.poll()
            assert s.stats()["n_preempts"] == rep + 1     # it stopped for the request, and went on
    finally:
        s.close()


# ------------------------------------------------------------------ reduction, configuration 2 shape
@pytest.mark.parametrize("slice_blocks", [1, 8, 64])
def test_reduce_sliced_ragged(env, slice_blocks):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_cover_equal, assert_close_rel
    n = 4096 * 37 + 123
    xs = TI.reduce_inputs(n=n, config_index=2)["x"]
    nb = OK.grid_of("reduce_sum", {"n": n})[0]
    x, partial, total = dev(xs), dev(np.zeros(nb, np.float32)), dev(np.zeros(1, np.float64))
    torch.cuda.synchronize()
    job = ctx.launch_sliced(B.reduce_sum(x, partial), slice_blocks, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    ctx.launch_native(B.reduce_final(partial, total))
    torch.cuda.synchronize()
    a = {"x": xs, "n": n, "partial": np.zeros(nb, np.float32)}
    cov, _ = OS.run_sliced("reduce_sum", (nb, 1, 1), a, slice_blocks)
    assert_cover_equal(rec, cov)
    assert_close_rel(host(partial), a["partial"], 2e-6)
    f = {"partial": a["partial"], "count": nb, "total": np.zeros(1, np.float64)}
    OS.run_native("reduce_final", (1, 1, 1), f)
    assert_close_rel(host(total), f["total"], 1e-6)


def test_reduce_all_ones_exact_all_forms(env):
    B, ctx, torch = env
    from gpu_util import host
    n = 1 << 22
    x = torch.ones(n, device="cuda")
    for form in ("native", "sliced", "ptb", "ptb_chunk"):
        partial = torch.zeros(n // 4096, device="cuda")
        total = torch.zeros(1, device="cuda", dtype=torch.float64)
        torch.cuda.synchronize()
        k = B.reduce_sum(x, partial)
        if form == "native":
            ctx.launch_native(k)
        else:
            job = (ctx.launch_sliced(k, 100) if form == "sliced" else
                   ctx.launch_ptb(k, 512, chunk=4 if form == "ptb_chunk" else 1))
            assert job.wait() == B.JOB_COMPLETE
            job.free()
        ctx.launch_native(B.reduce_final(partial, total))
        torch.cuda.synchronize()
        assert (host(partial) == 4096.0).all(), form
        assert host(total)[0] == float(n), form


# ------------------------------------------------------------------ error behaviour
def test_error_paths(env):
    B, ctx, torch = env
    import ctypes as C
    x = torch.zeros(1024, device="cuda")
    y = torch.zeros(1024, device="cuda")
    k = B.saxpy(x, y, 1.0)
    lib = B.lib()
    j = C.c_void_p()
    assert lib.tally_launch_sliced(ctx.h, C.byref(k.desc), 0, 1, 0, C.byref(j)) == B.ERR_INVALID_ARG
    assert lib.tally_launch_ptb(ctx.h, C.byref(k.desc), 0, 1, 0, C.byref(j)) == B.ERR_INVALID_ARG
    assert lib.tally_launch_ptb(ctx.h, C.byref(k.desc), 4, 0, 0, C.byref(j)) == B.ERR_INVALID_ARG
    # more workers than are resident at once: the kernel could not be preempted promptly
    mw = ctx.max_workers(k)
    assert mw >= B.device_info()["num_cus"] and mw % B.device_info()["num_cus"] == 0
    assert lib.tally_launch_ptb(ctx.h, C.byref(k.desc), mw + 1, 1, 0, C.byref(j)) == B.ERR_INVALID_ARG
    bad = B.KernelDesc(k.desc.kernel_id, k.desc.grid, k.desc.block, k.desc.args, k.desc.args_size)
    bad.grid.x += 1                                     # not the kernel's logical grid
    assert lib.tally_launch_native(ctx.h, C.byref(bad), 0) == B.ERR_INVALID_ARG
    bad.grid.x -= 1
    bad.kernel_id = 99
    assert lib.tally_launch_native(ctx.h, C.byref(bad), 0) == B.ERR_INVALID_ARG
    bad.kernel_id = k.desc.kernel_id
    bad.args_size -= 4
    assert lib.tally_launch_native(ctx.h, C.byref(bad), 0) == B.ERR_INVALID_ARG
    assert lib.tally_preempt(None) == B.ERR_INVALID_ARG
    # decode attention is a two-phase kernel: only the original form exists
    q = torch.zeros((2, 128), dtype=torch.int16, device="cuda")
    kv = torch.zeros((64, 2, 128), dtype=torch.int16, device="cuda")
    out = torch.zeros((2, 128), dtype=torch.int16, device="cuda")
    scratch = torch.zeros(B.attn_decode_scratch_bytes(2), dtype=torch.uint8, device="cuda")
    ka = B.attn_decode_bf16(q, kv, kv, out, scratch)
    assert lib.tally_launch_ptb(ctx.h, C.byref(ka.desc), 4, 1, 0, C.byref(j)) == B.ERR_UNSUPPORTED
    assert lib.tally_launch_sliced(ctx.h, C.byref(ka.desc), 4, 1, 0, C.byref(j)) == B.ERR_UNSUPPORTED
    with pytest.raises(B.TallyError):
        ctx.max_workers(ka)
    # state machine: resume of a complete job and preempt of a complete job are no-ops
    job = ctx.launch_ptb(k, 2)
    assert job.wait() == B.JOB_COMPLETE
    job.preempt()
    job.resume()
    assert job.progress()[2] == B.JOB_COMPLETE
    job.free()
    torch.cuda.synchronize()


# ------------------------------------------------------------------ freeing a running job
@pytest.mark.parametrize("form,workers", [("gemm", 16), ("saxpy", 64), ("saxpy", 512), ("sliced", 0)])
def test_freeing_a_running_job_finishes_what_was_launched(env, form, workers):
    """tally_job_free waits for the launches in flight: workers run their whole grid whether or not
    their slot was used before (here the first job of a context), and nobody is asked to pause; a
    sliced job runs the sub-kernels enqueued so far and no others."""
    B, _, torch = env
    ctx = B.Context(torch.cuda.Stream(), torch.cuda.Stream())
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workers)
    if form == "gemm":
        A, Bt = (torch.randn(1, r, 2048, device="cuda", generator=gen).to(torch.bfloat16) for r in (2048, 1024))
        out = torch.empty(1, 2048, 1024, dtype=torch.bfloat16, device="cuda")
        kern = B.gemm_bf16(A, Bt, out)
        torch.cuda.synchronize()
        ctx.launch_native(kern)
        torch.cuda.synchronize()
        want = out.clone()
        out.fill_(-3.0)
    else:
        x = torch.randn(1 << 25, device="cuda", generator=gen)
        out = torch.zeros(1 << 25, device="cuda")
        kern = B.saxpy(x, out, 1.5)
        want = 1.5 * x                                    # (added to zero: exactly the rounded product)
    torch.cuda.synchronize()
    if form == "sliced":
        job = ctx.launch_sliced(kern, 8192, max_in_flight=2)
        want[2 * 8192 * 256:] = 0.0
    else:
        job = ctx.launch_ptb(kern, workers)
    assert job.progress()[2] == B.JOB_RUNNING
    job.free()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    ctx.close()


# ------------------------------------------------------------------ workers in teams
@pytest.mark.parametrize("workers,chunk,blocks", [(256, 1, 256), (256, 1, 1031), (261, 1, 2000), (519, 1, 519),
                                                  (519, 3, 5003), (1024, 2, 2048), (1790, 1, 9000), (2047, 1, 9000), (300, 16, 4801)])
def test_teams_of_workers_run_every_block_once(env, workers, chunk, blocks):
    """From 256 workers on short blocks fetch through their team's word, a batch at a time.  Teams of
    eight and the odd last one, grids that one fetch each covers exactly and ones that end inside a
    batch, stops at given counter values and on requests: always a prefix, every block once."""
    B, ctx, torch = env
    n = blocks * 256 - 100
    gen = torch.Generator(device="cuda")
    gen.manual_seed(workers + blocks)
    x, y0 = (torch.randn(n, device="cuda", generator=gen) for _ in range(2))
    y = y0.clone()
    torch.cuda.synchronize()
    want = (1.5 * x.double() + y0.double()).float()       # the product is exact in 64 bits: one rounding
    job = ctx.launch_ptb(B.saxpy(x, y, 1.5), workers, chunk=chunk, coverage=True, stop_at=blocks // 3)
    assert job.wait() == B.JOB_STOPPED and job.progress()[0] == blocks // 3
    for at in (blocks // 3 + 1, blocks // 2):
        count = job.coverage()["count"]
        done = job.progress()[0]
        assert (count[:done] == 1).all() and (count[done:] == 0).all()
        job.resume(stop_at=at)
        assert job.wait() == B.JOB_STOPPED and job.progress()[0] == at
    job.resume()
    for _ in range(50):
        job.preempt()
        if job.wait() == B.JOB_COMPLETE:
            break
        done = job.progress()[0]
        count = job.coverage()["count"]
        assert (count[:done] == 1).all() and (count[done:] == 0).all()
        job.resume()
    assert job.wait() == B.JOB_COMPLETE
    assert (job.coverage()["count"] == 1).all()
    job.free()
    torch.cuda.synchronize()
    # a fused multiply-add rounds once, the 64-bit sum and its conversion at most once more (2^-53 of it)
    assert ((y - want).abs() <= 2.0 ** -23 * want.abs()).all()


# ------------------------------------------------------------------ slices, stopped and resumed
@pytest.mark.parametrize("slice_blocks,in_flight", [(1, 1), (7, 1), (64, 3), (300, 2), (40, 13), (40, 14), (2000, 1),
                                                    (511, 1), (512, 1), (512, 2), (700, 1)])
def test_slices_stop_and_go_on(env, slice_blocks, in_flight):
    """Stopped again and again, from launches that cover the grid at once to ones of a single block:
    always whole slices, a prefix, every block once, and no more than max_in_flight slices beyond those
    that the last visit found ended."""
    B, ctx, torch = env
    blocks = 1500
    n = blocks * 256 - 77
    gen = torch.Generator(device="cuda")
    gen.manual_seed(slice_blocks)
    x, y0 = (torch.randn(n, device="cuda", generator=gen) for _ in range(2))
    y = y0.clone()
    torch.cuda.synchronize()
    want = (1.5 * x.double() + y0.double()).float()       # the product is exact in 64 bits: one rounding
    job = ctx.launch_sliced(B.saxpy(x, y, 1.5), slice_blocks, max_in_flight=in_flight, coverage=True)
    job.preempt()                                         # exactly the first max_in_flight have been enqueued
    st = job.wait()
    done = job.progress()[0]
    assert done == min(slice_blocks * in_flight, blocks)
    for round_ in range(40):
        count = job.coverage()["count"]
        assert (count[:done] == 1).all() and (count[done:] == 0).all()
        if st == B.JOB_COMPLETE:
            break
        assert st == B.JOB_STOPPED and done % slice_blocks == 0
        job.resume()
        for _ in range(round_ % 4 * 8):                   # now and then let it get ahead first
            job.pump()
        ended = job.progress()[0]
        job.preempt()
        st, before = job.wait(), done
        done = job.progress()[0]
        assert min(before + slice_blocks * in_flight, blocks) <= done <= ended + slice_blocks * in_flight
    if st != B.JOB_COMPLETE:
        job.resume()
        assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert (rec["count"] == 1).all()
    torch.cuda.synchronize()
    # a fused multiply-add rounds once, the 64-bit sum and its conversion at most once more (2^-53 of it)
    assert ((y - want).abs() <= 2.0 ** -23 * want.abs()).all()


@pytest.mark.parametrize("in_flight", [1, 2])
def test_a_stop_lets_no_more_than_max_in_flight_slices_run(env, in_flight):
    """Slices of two rounds of GEMM tiles, stopped at changing moments between two visits of the
    host: whatever the moment, at most max_in_flight sub-kernels run beyond those that the last
    visit found ended.  Always whole slices, a prefix, every block once, the numbers of one launch."""
    B, ctx, torch = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(in_flight)
    A, Bt = (torch.randn(10, 8192, 512, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    C = torch.empty(10, 8192, 8192, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C)                          # 10240 blocks, a slice takes tens of microseconds
    torch.cuda.synchronize()
    ctx.launch_native(kern)
    torch.cuda.synchronize()
    want = C.clone()
    C.fill_(-3.0)
    torch.cuda.synchronize()
    job = ctx.launch_sliced(kern, 512, max_in_flight=in_flight, coverage=True)
    for round_ in range(100):
        until = time.perf_counter() + 1e-6 * (10 + round_ * 13 % 70)
        while time.perf_counter() < until:
            job.pump()
        ended, _, st = job.progress()
        job.preempt()
        job.wait()
        done, _, st = job.progress()
        assert done % 512 == 0 and done <= ended + 512 * in_flight, round_
        count = job.coverage()["count"]
        assert (count[:done] == 1).all() and (count[done:] == 0).all()
        if st == B.JOB_COMPLETE:
            break
        assert st == B.JOB_STOPPED
        job.resume()
    assert job.wait() == B.JOB_COMPLETE and round_ >= 4
    job.free()
    torch.cuda.synchronize()
    assert torch.equal(C, want)


@pytest.mark.parametrize("workers,chunk,blocks,stop_at", [
    (8, 4, 32, None), (8, 4, 33, None), (8, 4, 63, 40), (8, 4, 41, 35), (8, 4, 5, None), (8, 4, 31, 3), (7, 3, 50, 23),
    (256, 4, 1024 + 203, None), (256, 16, 300, 299), (300, 2, 1000, 601), (512, 4, 2048 + 700, 2049)])
def test_last_round_of_fetches_is_shared(env, workers, chunk, blocks, stop_at):
    """The last round of a grid that whole fetches do not divide: every block once, the prefix at a
    stop inside it, and the bits of the original form."""
    B, ctx, torch = env
    rows, cols = 4 * blocks - 1, 260
    g = torch.Generator(device="cuda")
    g.manual_seed(blocks)
    x = torch.randn(rows, cols, device="cuda", generator=g)
    want, y = torch.zeros_like(x), torch.zeros_like(x)
    torch.cuda.synchronize()
    ctx.launch_native(B.softmax_f32(x, want))
    job = ctx.launch_ptb(B.softmax_f32(x, y), workers, chunk=chunk, coverage=True, stop_at=stop_at)
    st = job.wait()
    if stop_at is not None:
        assert st == B.JOB_STOPPED and job.progress()[0] == stop_at
        rec = job.coverage()
        assert (rec["count"][:stop_at] == 1).all() and (rec["count"][stop_at:] == 0).all()
        job.resume()
        st = job.wait()
    assert st == B.JOB_COMPLETE and job.progress()[0] == blocks
    rec = job.coverage()
    job.free()
    assert (rec["count"] == 1).all() and (rec["bx"] == np.arange(blocks)).all()
    torch.cuda.synchronize()
    assert torch.equal(y, want)


def test_requests_around_a_shared_last_round_leave_a_prefix(env):
    """Requests at growing delays, on jobs nearly half of whose blocks are their last round."""
    B, ctx, torch = env
    workers, chunk, blocks = 64, 8, 64 * 8 + 64 * 6 + 1
    rows, cols = 4 * blocks, 8192
    x = torch.randn(rows, cols, device="cuda")
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    k = B.softmax_f32(x, y)
    for attempt in range(24):
        job = ctx.launch_ptb(k, workers, chunk=chunk, coverage=True)
        t0 = time.perf_counter()
        while time.perf_counter() - t0 < 6e-6 * attempt:
            pass
        segments = 0
        job.preempt()
        while job.wait() == B.JOB_STOPPED:
            done = job.progress()[0]
            rec = job.coverage()
            assert done < blocks and (rec["count"][:done] == 1).all() and (rec["count"][done:] == 0).all()
            segments += 1
            job.resume()
            if segments < 3:
                job.preempt()
        rec = job.coverage()
        job.free()
        assert (rec["count"] == 1).all()
    torch.cuda.synchronize()
    # (1e-5 of the sum of a row, as for the row kernels' other comparisons)
    ref = torch.softmax(x[:: 97].double(), dim=1)
    assert (y[:: 97].double() - ref).abs().max() <= 1e-5 * ref.max() + 1e-7


@pytest.mark.parametrize("tile,m,n", [("256", 768, 512), ("256", 1024, 768), ("256", 1024, 2048), ("256", 1536, 2048),
                                      ("128", 768, 512), ("128", 1024, 768), ("128", 1024, 1536), ("128", 2048, 2048)])
@pytest.mark.parametrize("k", [32, 96, 160, 224, 352, 416, 736, 1312])
def test_parts_of_blocks_as_tiles_straight_to_lds(env, tile, m, n, k):
    """256 workers on so few blocks that each takes a part, 32x64, 64x64, 128x64 or 128x128: fewer stages than
    the part keeps on their way, as many, one to four and more beyond, a last stage half full; a job preempted
    with a pause and resumed; the same bits as one worker's whole blocks and as the original form's."""
    B, ctx, torch = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n + k)
    A = torch.randn(1, m, k, device="cuda", generator=gen).to(torch.bfloat16)
    Bt = torch.randn(1, n, k, device="cuda", generator=gen).to(torch.bfloat16)
    C = torch.full((1, m, n), 7.0, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C, n128=tile == "128")
    torch.cuda.synchronize()

    def bits(run):
        C.fill_(7.0)
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        return C.clone()

    def job(workers, preempt=False):
        j = ctx.launch_ptb(kern, workers)
        if preempt:
            j.preempt(pause=True)
            j.end_pause()
        while j.wait() != B.JOB_COMPLETE:
            j.resume()
        j.free()

    want = bits(lambda: job(1))
    assert torch.equal(bits(lambda: job(256)), want)
    assert torch.equal(bits(lambda: job(256, preempt=True)), want)
    assert torch.equal(bits(lambda: ctx.launch_native(kern)), want)
