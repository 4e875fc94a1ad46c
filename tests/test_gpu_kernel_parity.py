"""GPU parity of the workload kernels (GEMM, GEMV, softmax, LayerNorm, decode attention) in
their native and transformed forms against the CPU oracle, element by element, and on
sampled tiles at the full benchmark sizes."""
import numpy as np
import pytest

import tally_inputs as TI
from gemm_tiles import GEMM_TILES
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


def _run_form(B, ctx, torch, kernel, form):
    if form == "native":
        ctx.launch_native(kernel)
    elif form == "native_hi":
        ctx.launch_native(kernel, hi=True)
    else:
        if form == "sliced":
            job = ctx.launch_sliced(kernel, 3)
        elif form == "ptb":
            job = ctx.launch_ptb(kernel, 5)
        else:                                             # preempted half way, then resumed
            job = ctx.launch_ptb(kernel, 3, chunk=2, stop_at=max(1, kernel.total_blocks // 2))
            job.wait()
            job.resume()
        assert job.wait() == B.JOB_COMPLETE
        job.free()
    torch.cuda.synchronize()


FORMS = ["native", "sliced", "ptb", "ptb_preempted"]


# ------------------------------------------------------------------ GEMM, 256-wide tiles
@pytest.mark.parametrize("form", FORMS)
def test_gemm_bf16_forms(env, form):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n, k, batch = 512, 768, 320, 2                    # 3 x 2 x 2 tiles, 5 k-steps
    g = TI.gemm_inputs(m, n, k, config_index=1, batch=batch)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16", OK.grid_of("gemm_bf16", a), a)
    A, Bt, Cd = dev(g["A"]), dev(g["Bt"]), dev(np.zeros((batch, m, n), np.uint16))
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, Cd)
    assert kern.grid == (3, 2, 2)
    _run_form(B, ctx, torch, kern, form)
    assert_bf16_close(host(Cd), a["C"])


@pytest.mark.parametrize("k", [32, 64, 96, 128])
@pytest.mark.parametrize("form", ["native", "ptb"])
def test_gemm_short_k(env, k, form):
    """One to four k-steps: fewer than the LDS ring has stages (prologue and drain paths)."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n = 256, 512
    g = TI.gemm_inputs(m, n, k, config_index=3, scale=0.25)
    a = dict(g, C=np.zeros((1, m, n), np.uint16))
    OS.run_native("gemm_bf16", OK.grid_of("gemm_bf16", a), a)
    A, Bt, Cd = dev(g["A"]), dev(g["Bt"]), dev(np.zeros((1, m, n), np.uint16))
    torch.cuda.synchronize()
    _run_form(B, ctx, torch, B.gemm_bf16(A, Bt, Cd), form)
    assert_bf16_close(host(Cd), a["C"])


@pytest.mark.parametrize("n128", [False, True])
@pytest.mark.parametrize("k", [32, 96, 128, 160, 224])
def test_gemm_stage_ends(env, k, n128):
    """K-loop ends: one to four 64-wide LDS stages, the last one whole or half full (its upper
    half must count as zero whatever lies beyond the row's end: NaN here), several tiles per
    worker; same tolerance as every bf16 product."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n = 512, 384 if n128 else 512
    name = "gemm_bf16_n128" if n128 else "gemm_bf16"
    g = TI.gemm_inputs(m, n, k, config_index=3, scale=0.25)
    a = dict(g, C=np.zeros((1, m, n), np.uint16))
    OS.run_native(name, OK.grid_of(name, a), a)
    Ap = torch.full((1, m, k + 40), 0x7FC0, dtype=torch.int16, device="cuda")
    Bp = torch.full((1, n, k + 40), 0x7FC0, dtype=torch.int16, device="cuda")
    Ap[:, :, :k], Bp[:, :, :k] = dev(g["A"]), dev(g["Bt"])
    for form in FORMS:
        Cd = torch.full((1, m, n), 0x7FC0, dtype=torch.int16, device="cuda")
        torch.cuda.synchronize()
        _run_form(B, ctx, torch, B.gemm_bf16(Ap[:, :, :k], Bp[:, :, :k], Cd, n128=n128), form)
        assert_bf16_close(host(Cd), a["C"])


def test_gemm_training_step_shapes(env):
    """Shapes of the transformer-layer step: attention scores (batched, K = 128, 2048 x 2048
    outputs per batch) and the second FFN product (K = 16384), persistent workers; the
    oracle recomputes whole batches / tiles."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    g = TI.gemm_inputs(2048, 2048, 128, config_index=3, batch=3, scale=0.25)
    A, Bt = dev(g["A"]), dev(g["Bt"])
    Cd = torch.zeros((3, 2048, 2048), dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, Cd)
    assert kern.grid == (8, 8, 3)
    job = ctx.launch_ptb(kern, 256)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    a = dict(g, C=np.zeros((3, 2048, 2048), np.uint16))
    OS.run_native("gemm_bf16", OK.grid_of("gemm_bf16", a), a)
    assert_bf16_close(host(Cd), a["C"])
    g = TI.gemm_inputs(512, 256, 16384, config_index=3, scale=1.0 / 128.0)
    A, Bt = dev(g["A"]), dev(g["Bt"])
    Cd = torch.zeros((1, 512, 256), dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    job = ctx.launch_ptb(B.gemm_bf16(A, Bt, Cd), 256)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    a = dict(g, C=np.zeros((1, 512, 256), np.uint16))
    OS.run_native("gemm_bf16", OK.grid_of("gemm_bf16", a), a)
    assert_bf16_close(host(Cd), a["C"])


@pytest.mark.parametrize("form", FORMS)
def test_gemm_n128_forms(env, form):
    """256-row x 128-column tiles (n a multiple of 128 only): 3 x 2 x 2 tiles, 6 k-steps."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n, k, batch = 512, 384, 192, 2
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16_n128", OK.grid_of("gemm_bf16_n128", a), a)
    A, Bt, Cd = dev(g["A"]), dev(g["Bt"]), dev(np.zeros((batch, m, n), np.uint16))
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, Cd, n128=True)
    assert kern.grid == (3, 2, 2)
    _run_form(B, ctx, torch, kern, form)
    assert_bf16_close(host(Cd), a["C"])


@pytest.mark.parametrize("k", [32, 96, 2048])
def test_gemm_n128_attention_value_shape(env, k):
    """The P.V product of the training-like step: 2048 x 128 outputs per batch entry."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n, batch = 2048, 128, 2
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.05)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16_n128", OK.grid_of("gemm_bf16_n128", a), a)
    A, Bt, Cd = dev(g["A"]), dev(g["Bt"]), dev(np.zeros((batch, m, n), np.uint16))
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, Cd, n128=True)
    assert kern.grid == (1, 8, 2)
    job = ctx.launch_ptb(kern, 256)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    assert_bf16_close(host(Cd), a["C"])


@pytest.mark.parametrize("variant", ["big", "n128", "small"])
def test_gemm_padded_leading_dimensions(env, variant):
    """Operands stored with rows longer than k (views of padded buffers, batch pitch larger
    than the matrix): same result as the oracle gets from the unpadded arrays."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n, k, batch = (512, 512, 160, 2) if variant == "big" else ((256, 384, 96, 2) if variant == "n128"
                                                                    else (100, 70, 64, 2))
    name = {"big": "gemm_bf16", "n128": "gemm_bf16_n128", "small": "gemm_bf16_small"}[variant]
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native(name, OK.grid_of(name, a), a)
    Ap = torch.full((batch, m + 3, k + 24), 0x7FC0, dtype=torch.int16, device="cuda")   # NaN padding
    Bp = torch.full((batch, n + 1, k + 8), 0x7FC0, dtype=torch.int16, device="cuda")
    Ap[:, :m, :k] = dev(g["A"])
    Bp[:, :n, :k] = dev(g["Bt"])
    Cd = torch.zeros((batch, m, n), dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    kern = B.gemm_bf16(Ap[:, :m, :k], Bp[:, :n, :k], Cd, small=(variant == "small"),
                       n128=(variant == "n128"))
    job = ctx.launch_ptb(kern, 7)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    assert_bf16_close(host(Cd), a["C"])
    bad = torch.zeros((1, 256, 256 + 4), dtype=torch.int16, device="cuda")              # pitch not a multiple of 8
    with pytest.raises(B.TallyError):
        B.gemm_bf16(bad[:, :, :256], bad[:, :, :256], torch.zeros((1, 256, 256), dtype=torch.int16, device="cuda"))


def test_gemm_rejects_unaligned_output(env):
    B, ctx, torch = env
    A = torch.zeros((1, 256, 64), dtype=torch.int16, device="cuda")
    Cbuf = torch.zeros(256 * 256 + 8, dtype=torch.int16, device="cuda")
    with pytest.raises(B.TallyError):
        B.gemm_bf16(A, A, Cbuf[1:1 + 256 * 256].view(1, 256, 256))


def test_gemm_identity_is_exact(env):
    B, ctx, torch = env
    from gpu_util import dev, host
    eye = TI.to_bf16_bits(np.eye(256, dtype=np.float32))[None]
    Bt = TI.normal_bf16(np.random.default_rng(5), (1, 512, 256), 1 / 64)
    A, Btd, Cd = dev(eye), dev(Bt), dev(np.zeros((1, 256, 512), np.uint16))
    torch.cuda.synchronize()
    ctx.launch_native(B.gemm_bf16(A, Btd, Cd))
    torch.cuda.synchronize()
    assert (host(Cd)[0] == Bt[0].T).all()                # I . B = B bit for bit


def test_gemm_cfg1_full_size_sampled_tiles(env):
    """M = N = K = 4096 in persistent-worker form with 256 workers (the benchmark's launch
    configuration); the oracle recomputes a seeded sample of whole 256x256 tiles."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    g = TI.gemm_inputs(4096, 4096, 4096, config_index=1)
    A, Bt = dev(g["A"]), dev(g["Bt"])
    Cd = torch.zeros((1, 4096, 4096), dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    kern = B.gemm_bf16(A, Bt, Cd)
    assert kern.grid == (16, 16, 1)
    job = ctx.launch_ptb(kern, 256, coverage=True)
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    assert (rec["count"] == 1).all()
    idx = np.arange(256)
    assert (rec["bx"] == idx % 16).all() and (rec["by"] == idx // 16).all()
    got = host(Cd)
    rng = np.random.default_rng(11)
    for t in [0, 255] + [int(v) for v in rng.integers(1, 255, 3)]:
        bx, by = t % 16, t // 16
        a = dict(g, C=np.zeros((1, 4096, 4096), np.uint16))
        OK.exec_block("gemm_bf16", (bx, by, 0), (16, 16, 1), a)
        r, c = slice(by * 256, by * 256 + 256), slice(bx * 256, bx * 256 + 256)
        assert_bf16_close(got[0, r, c], a["C"][0, r, c])
    # all-ones / 64: every output is exactly 1 (property that holds at any size)
    ones = TI.to_bf16_bits(np.full((1, 4096, 4096), 1 / 64, np.float32))
    A1 = dev(ones)
    torch.cuda.synchronize()
    ctx.launch_native(B.gemm_bf16(A1, A1, Cd))
    torch.cuda.synchronize()
    assert (host(Cd) == 0x3F80).all()


@pytest.mark.parametrize("m,n,k,batch", [(512, 512, 96, 1), (256, 512, 96, 3), (256, 768, 96, 4), (1024, 1024, 96, 1), (512, 1024, 96, 4),
                                         (512, 768, 64, 8), (2048, 1536, 160, 1), (2048, 4352, 160, 1)])
@pytest.mark.parametrize("n128", [False, True])
def test_gemm_original_form_covers(env, m, n, k, batch, n128):
    """The original form's tiles by the size of the output, on both sides of each line (256 tiles of
    32x32, 192 of 32x64, 192, 256 and 512 of 64x64; short k; 96 and 272 of 256x128), operands with
    NaN beyond k, nothing written behind C."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    name = "gemm_bf16_n128" if n128 else "gemm_bf16"
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native(name, OK.grid_of(name, a), a)
    Ap = torch.full((batch, m, k + 40), 0x7FC0, dtype=torch.int16, device="cuda")
    Bp = torch.full((batch, n, k + 8), 0x7FC0, dtype=torch.int16, device="cuda")
    Ap[:, :, :k], Bp[:, :, :k] = dev(g["A"]), dev(g["Bt"])
    buf = torch.full((batch * m * n + 8,), 0x7FC0, dtype=torch.int16, device="cuda")
    Cd = buf[:batch * m * n].view(batch, m, n)
    torch.cuda.synchronize()
    ctx.launch_native(B.gemm_bf16(Ap[:, :, :k], Bp[:, :, :k], Cd, n128=n128))
    torch.cuda.synchronize()
    assert_bf16_close(host(Cd), a["C"])
    assert (host(buf[batch * m * n:]) == 0x7FC0).all()


def _ptb_parts_case(B, torch, m, n, k, batch, n128):
    from gpu_util import dev
    name = "gemm_bf16_n128" if n128 else "gemm_bf16"
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    grid = OK.grid_of(name, a)
    OS.run_native(name, grid, a)
    A, Bt = dev(g["A"]), dev(g["Bt"])
    Cd = torch.full((batch, m, n), 0x7FC0, dtype=torch.int16, device="cuda")
    torch.cuda.synchronize()
    return a["C"], Cd, B.gemm_bf16(A, Bt, Cd, n128=n128), grid


def _check_blocks(got, want, grid, tn, done):
    """Blocks [0, done) of the grid hold the product, the others what was there before (NaN)."""
    from gpu_util import assert_bf16_close
    for idx in range(grid[0] * grid[1] * grid[2]):
        bx, by, bz = idx % grid[0], idx // grid[0] % grid[1], idx // (grid[0] * grid[1])
        r, c = slice(by * 256, by * 256 + 256), slice(bx * tn, bx * tn + tn)
        if idx < done:
            assert_bf16_close(got[bz, r, c], want[bz, r, c])
        else:
            assert (got[bz, r, c] == 0x7FC0).all()


@pytest.mark.parametrize("m,n,batch", [(256, 256, 3), (512, 768, 2), (768, 1024, 2), (1024, 1536, 2)])
@pytest.mark.parametrize("k", [96, 1056])
@pytest.mark.parametrize("n128", [False, True])
def test_gemm_workers_take_parts_of_blocks(env, m, n, batch, k, n128):
    """Grids of fewer blocks than workers (3 to 96 blocks, 256 workers: every size of part):
    coverage by whole blocks, a stop between blocks and the rest from there."""
    B, ctx, torch = env
    from gpu_util import host
    want, Cd, kern, grid = _ptb_parts_case(B, torch, m, n, k, batch, n128)
    total, tn = kern.total_blocks, 128 if n128 else 256
    stop = total // 2 + 1
    job = ctx.launch_ptb(kern, 256, chunk=2, coverage=True, stop_at=stop)
    assert job.wait() == B.JOB_STOPPED and job.progress()[0] == stop
    torch.cuda.synchronize()
    _check_blocks(host(Cd), want, grid, tn, stop)
    job.resume()
    assert job.wait() == B.JOB_COMPLETE and job.progress()[0] == total
    rec = job.coverage()
    job.free()
    torch.cuda.synchronize()
    _check_blocks(host(Cd), want, grid, tn, total)
    idx = np.arange(total)
    assert (rec["count"] == 1).all() and (rec["worker"] < 256).all()
    assert (rec["segment"] == (idx >= stop)).all()
    assert (rec["bx"] == idx % grid[0]).all() and (rec["bz"] == idx // (grid[0] * grid[1])).all()


@pytest.mark.parametrize("m,n,n128", [(512, 512, False), (1024, 1024, False), (2048, 2048, False), (512, 512, True)])
def test_gemm_parts_preempted_anywhere(env, m, n, n128):
    """A request at any moment leaves whole blocks: those below the progress are finished, parts
    handed out after the request included, and the others are untouched."""
    import time
    B, ctx, torch = env
    from gpu_util import host
    want, Cd, kern, grid = _ptb_parts_case(B, torch, m, n, 512, 1, n128)
    tn = 128 if n128 else 256
    for delay_us in (0, 2, 4, 6, 8, 10, 12, 15, 20, 30):
        Cd.fill_(0x7FC0)
        torch.cuda.synchronize()
        job = ctx.launch_ptb(kern, 256, coverage=True)
        t0 = time.perf_counter()
        while (time.perf_counter() - t0) * 1e6 < delay_us:
            pass
        job.preempt()
        state = job.wait()
        done, total, _ = job.progress()
        assert (state == B.JOB_COMPLETE) == (done == total)
        torch.cuda.synchronize()
        _check_blocks(host(Cd), want, grid, tn, done)
        job.resume()
        assert job.wait() == B.JOB_COMPLETE
        assert (job.coverage()["count"] == 1).all()
        job.free()
        torch.cuda.synchronize()
        _check_blocks(host(Cd), want, grid, tn, total)


@pytest.mark.parametrize("m,n,workers", [(256, 1792, 5), (768, 1024, 5), (1024, 1280, 9), (256, 2560, 8)])
@pytest.mark.parametrize("k", [96, 2048])
def test_gemm_last_round_in_parts(env, m, n, workers, k):
    """Grids one to several rounds long whose last round is handed out in halves (7 and 12 blocks
    on 5 workers, 20 on 9, 10 on 8): coverage by whole blocks, a stop between blocks, requests at
    any moment, the rest from there."""
    import time
    B, ctx, torch = env
    from gpu_util import host
    want, Cd, kern, grid = _ptb_parts_case(B, torch, m, n, k, 1, False)
    total = kern.total_blocks
    stop = workers + 1
    job = ctx.launch_ptb(kern, workers, coverage=True, stop_at=stop)
    assert job.wait() == B.JOB_STOPPED and job.progress()[0] == stop
    torch.cuda.synchronize()
    _check_blocks(host(Cd), want, grid, 256, stop)
    job.resume()
    assert job.wait() == B.JOB_COMPLETE
    rec = job.coverage()
    job.free()
    torch.cuda.synchronize()
    _check_blocks(host(Cd), want, grid, 256, total)
    idx = np.arange(total)
    assert (rec["count"] == 1).all() and (rec["worker"] < workers).all()
    assert (rec["bx"] == idx % grid[0]).all() and (rec["by"] == idx // grid[0]).all()
    for delay_us in (0, 5, 10, 15, 20, 30, 40, 50, 60, 80):
        Cd.fill_(0x7FC0)
        torch.cuda.synchronize()
        job = ctx.launch_ptb(kern, workers, coverage=True)
        t0 = time.perf_counter()
        while (time.perf_counter() - t0) * 1e6 < delay_us:
            pass
        job.preempt()
        state = job.wait()
        done = job.progress()[0]
        assert (state == B.JOB_COMPLETE) == (done == total)
        torch.cuda.synchronize()
        _check_blocks(host(Cd), want, grid, 256, done)
        job.resume()
        assert job.wait() == B.JOB_COMPLETE
        assert (job.coverage()["count"] == 1).all()
        job.free()
        torch.cuda.synchronize()
        _check_blocks(host(Cd), want, grid, 256, total)


# ------------------------------------------------------------------ GEMM, 32-wide ragged tiles
@pytest.mark.parametrize("form", FORMS)
def test_gemm_small_forms(env, form):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    m, n, k, batch = 300, 520, 96, 2
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16_small", OK.grid_of("gemm_bf16_small", a), a)
    A, Bt, Cd = dev(g["A"]), dev(g["Bt"]), dev(np.zeros((batch, m, n), np.uint16))
    torch.cuda.synchronize()
    _run_form(B, ctx, torch, B.gemm_bf16(A, Bt, Cd, small=True), form)
    assert_bf16_close(host(Cd), a["C"])


@pytest.mark.parametrize("m,n,k,batch", [(1, 1, 32, 1), (31, 33, 64, 1), (33, 31, 96, 3), (32, 64, 224, 1),
                                         (64, 30, 256, 1), (17, 101, 288, 2), (40, 36, 544, 1), (65, 95, 800, 1)])
def test_gemm_small_edges(env, m, n, k, batch):
    """Rows and columns past the matrix, K that ends in half a 64-wide chunk, fewer chunks than
    waves, one, two and more rounds of chunks per wave, output rows that no wide store may touch;
    what lies beyond K and between the rows is NaN, and nothing is written behind C."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16_small", OK.grid_of("gemm_bf16_small", a), a)
    Ap = torch.full((batch, m + 2, k + 40), 0x7FC0, dtype=torch.int16, device="cuda")
    Bp = torch.full((batch, n + 2, k + 8), 0x7FC0, dtype=torch.int16, device="cuda")
    Ap[:, :m, :k], Bp[:, :n, :k] = dev(g["A"]), dev(g["Bt"])
    for form in FORMS:
        buf = torch.full((batch * m * n + 8,), 0x7FC0, dtype=torch.int16, device="cuda")
        Cd = buf[:batch * m * n].view(batch, m, n)
        torch.cuda.synchronize()
        _run_form(B, ctx, torch, B.gemm_bf16(Ap[:, :m, :k], Bp[:, :n, :k], Cd, small=True), form)
        assert_bf16_close(host(Cd), a["C"])
        assert (host(buf[batch * m * n:]) == 0x7FC0).all()


@pytest.mark.parametrize("k", [32, 64, 96, 160, 224])
@pytest.mark.parametrize("m,n,batch", [(70, 130, 20), (33, 127, 64), (70, 130, 64), (64, 64, 400), (130, 65, 128), (127, 129, 171)])
def test_gemm_small_original_form_larger_tiles(env, m, n, k, batch):
    """Grids that the original form covers with 32x64 (180 and 256 of them), 64x64 (384 and 400) and
    128x64 tiles (512 and 513): rows and columns past the matrix, one to four stages, a last stage
    half full, NaN beyond K and between the rows, nothing written behind C."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16_small", OK.grid_of("gemm_bf16_small", a), a)
    Ap = torch.full((batch, m + 1, k + 40), 0x7FC0, dtype=torch.int16, device="cuda")
    Bp = torch.full((batch, n + 1, k + 8), 0x7FC0, dtype=torch.int16, device="cuda")
    Ap[:, :m, :k], Bp[:, :n, :k] = dev(g["A"]), dev(g["Bt"])
    buf = torch.full((batch * m * n + 8,), 0x7FC0, dtype=torch.int16, device="cuda")
    Cd = buf[:batch * m * n].view(batch, m, n)
    torch.cuda.synchronize()
    ctx.launch_native(B.gemm_bf16(Ap[:, :m, :k], Bp[:, :n, :k], Cd, small=True), hi=True)
    torch.cuda.synchronize()
    assert_bf16_close(host(Cd), a["C"])
    assert (host(buf[batch * m * n:]) == 0x7FC0).all()


@pytest.mark.parametrize("k", [160, 192, 224, 544, 1056])
@pytest.mark.parametrize("m,n,batch", [(1, 1, 1), (17, 33, 3), (70, 130, 8), (128, 768, 1), (100, 880, 1), (15, 16, 384), (256, 256, 1),
                                       (17, 50, 48)])
def test_gemm_one_wave_tiles(env, m, n, k, batch):
    """Up to 640 tiles of 16x16 the original form takes tiles of a single wave from the third stage
    on: rows and columns past the matrix, three to seventeen stages, a last stage half full, NaN beyond K and between the rows, nothing written
    behind C; the same bits as one worker's 32x32 blocks."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    g = TI.gemm_inputs(m, n, k, config_index=3, batch=batch, scale=0.125)
    a = dict(g, C=np.zeros((batch, m, n), np.uint16))
    OS.run_native("gemm_bf16_small", OK.grid_of("gemm_bf16_small", a), a)
    Ap = torch.full((batch, m + 1, k + 40), 0x7FC0, dtype=torch.int16, device="cuda")
    Bp = torch.full((batch, n + 1, k + 8), 0x7FC0, dtype=torch.int16, device="cuda")
    Ap[:, :m, :k], Bp[:, :n, :k] = dev(g["A"]), dev(g["Bt"])
    buf = torch.full((batch * m * n + 8,), 0x7FC0, dtype=torch.int16, device="cuda")
    Cd = buf[:batch * m * n].view(batch, m, n)
    kern = B.gemm_bf16(Ap[:, :m, :k], Bp[:, :n, :k], Cd, small=True)
    torch.cuda.synchronize()
    job = ctx.launch_ptb(kern, 1)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    torch.cuda.synchronize()
    one_worker = Cd.clone()
    Cd.fill_(0x7FC0)
    torch.cuda.synchronize()
    ctx.launch_native(kern, hi=True)
    torch.cuda.synchronize()
    assert torch.equal(Cd, one_worker)
    assert_bf16_close(host(Cd), a["C"])
    assert (host(buf[batch * m * n:]) == 0x7FC0).all()
    if m % 256 == 0:
        C2 = torch.full((batch, m, n), 0x7FC0, dtype=torch.int16, device="cuda")
        A2, B2 = Ap[:, :m, :k].contiguous(), Bp[:, :n, :k].contiguous()
        torch.cuda.synchronize()
        ctx.launch_native(B.gemm_bf16(A2, B2, C2))
        torch.cuda.synchronize()
        assert torch.equal(C2, one_worker)


@pytest.mark.parametrize("k", [160, 288, 320, 352, 768])
@pytest.mark.parametrize("m,n,batch", [(200, 1000, 1), (250, 1001, 1), (33, 5000, 1), (50, 4100, 1), (512, 1024, 1), (17, 50, 200), (40, 50, 100)])
def test_gemm_one_wave_tiles_of_two_blocks(env, m, n, k, batch):
    """640 to 2048 blocks of 16x16: tiles of one wave with two of them for k from three stages to eight, 16x32 or
    32x16 by which side has an odd number, ring tiles for other k; a last stage half full, columns of tiles
    that do not divide by eight, NaN beyond K and between the rows, nothing written behind C; the same bits as
    one worker's 32x32 blocks."""
    B, ctx, torch = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n + k)
    nan = float("nan")
    Ap = torch.full((batch, m + 1, k + 40), nan, dtype=torch.bfloat16, device="cuda")
    Bp = torch.full((batch, n + 1, k + 8), nan, dtype=torch.bfloat16, device="cuda")
    Ap[:, :m, :k] = torch.randn(batch, m, k, device="cuda", generator=gen)
    Bp[:, :n, :k] = torch.randn(batch, n, k, device="cuda", generator=gen)
    buf = torch.full((batch * m * n + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
    Cd = buf[:batch * m * n].view(batch, m, n)
    kern = B.gemm_bf16(Ap[:, :m, :k], Bp[:, :n, :k], Cd, small=True)
    torch.cuda.synchronize()
    job = ctx.launch_ptb(kern, 256)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    torch.cuda.synchronize()
    want = Cd.clone()
    Cd.fill_(7.0)
    torch.cuda.synchronize()
    ctx.launch_native(kern, hi=True)
    torch.cuda.synchronize()
    assert torch.equal(Cd, want) and bool((buf[batch * m * n:] == 7.0).all())
    row, col = m - 1, n - 1
    ref = (Ap[:, row, :k].double() * Bp[:, col, :k].double()).sum(1)
    mag = (Ap[:, row, :k].double() * Bp[:, col, :k].double()).abs().sum(1)
    assert ((Cd[:, row, col].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + k * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("m,n,k,batch", [(8192, 16, 416, 1), (2001, 1, 544, 1), (1000, 100, 800, 1), (113, 112, 352, 1), (17, 16, 800, 1),
                                         (300, 20, 416, 12), (33, 50, 352, 50), (2032, 112, 416, 1), (8190, 64, 480, 1), (1003, 200, 352, 1)])
def test_gemm_one_wave_tiles_of_narrow_outputs(env, m, n, k, batch):
    """Fewer panels of tiles than dies, along either side, and more; panels of a batch that do not divide by eight."""
    test_gemm_one_wave_tiles_of_two_blocks(env, m, n, k, batch)
    test_gemm_one_wave_tiles_of_two_blocks(env, n, m, k, batch)


def _us_of_launches(torch, launches_of, stream, launches=40, attempts=7):
    """Median time of one launch on `stream`, of each way of launching, in turn."""
    us = [[] for _ in launches_of]
    torch.cuda.synchronize()
    for attempt in range(attempts):
        for t, launch in zip(us, launches_of):
            with torch.cuda.stream(stream):
                torch.cuda._sleep(400000)                  # (the launches below queue up behind it)
                e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                e0.record(stream)
                for _ in range(launches):
                    launch()
                e1.record(stream)
                e1.synchronize()
                t.append(e0.elapsed_time(e1) * 1000 / launches)
    return [sorted(t)[attempts // 2] for t in us]


@pytest.mark.parametrize("m,n,k,batch,small", [(5632, 512, 768, 3, False), (1280, 2560, 2400, 3, False), (3328, 3072, 6304, 1, False),
                                               (4096, 768, 576, 3, False), (1000, 2300, 768, 1, True), (400, 1200, 2048, 1, True),
                                               (128, 3072, 768, 1, True), (90, 3400, 1536, 1, True)])
def test_tiles_that_need_the_whole_gpu_are_not_slower(env, m, n, k, batch, small):
    """A product alone on the GPU has all tiles to choose from, beside a best-effort job (here a stopped
    one) only some of them."""
    B, ctx, torch = env
    A, Bt = (torch.randn(batch, r, k, device="cuda").to(torch.bfloat16) for r in (m, n))
    kern = B.gemm_bf16(A, Bt, torch.empty(batch, m, n, dtype=torch.bfloat16, device="cuda"), small=small)
    launch, hi = lambda: ctx.launch_native(kern, hi=True), ctx._streams[0]
    x, y = torch.zeros(4096, device="cuda"), torch.zeros(4096, device="cuda")
    torch.cuda.synchronize()
    alone, beside = [], []
    for attempt in range(3):
        alone += _us_of_launches(torch, [launch], hi, 10, 3)
        job = ctx.launch_ptb(B.saxpy(x, y, 1.0), 1, stop_at=3)
        assert job.wait() == B.JOB_STOPPED
        beside += _us_of_launches(torch, [launch], hi, 10, 3)
        job.resume()
        job.wait()
        job.free()
    assert min(alone) < 1.1 * min(beside), (alone, beside)


@pytest.mark.parametrize("m,n,k", [(8192, 16, 1536), (2032, 112, 1536), (4096, 32, 2048), (2048, 64, 4096), (8192, 8, 768)])
def test_a_narrow_product_takes_no_longer_than_its_transpose(env, m, n, k):
    """The two ask for the same work; with a narrow one on a few of the eight dies it took 1.6 to 5 times as long."""
    B, ctx, torch = env
    A, Bt = (torch.randn(1, r, k, device="cuda").to(torch.bfloat16) for r in (m, n))
    kerns = [B.gemm_bf16(A, Bt, torch.empty(1, m, n, dtype=torch.bfloat16, device="cuda"), small=True),
             B.gemm_bf16(Bt, A, torch.empty(1, n, m, dtype=torch.bfloat16, device="cuda"), small=True)]
    narrow, wide = _us_of_launches(torch, [lambda k=k: ctx.launch_native(k, hi=True) for k in kerns], ctx._streams[0])
    assert narrow < 1.35 * wide, (narrow, wide)


@pytest.mark.parametrize("m,n,k,batch", [
    (512, 500, 1568, 1), (500, 512, 2080, 1),
    (225, 1250, 544, 5), (399, 1200, 1056, 1),
    (300, 3000, 512, 1), (1, 16300, 2080, 1), (1000, 1025, 544, 1),
    (777, 1777, 544, 1), (100, 900, 576, 12),
    (1500, 1500, 544, 1), (413, 741, 544, 12),
    (1025, 2047, 544, 1), (256, 8192, 512, 1), (129, 65, 512, 128),
    (1000, 2300, 512, 1), (1000, 2300, 800, 1), (384, 8000, 544, 1),
    (2000, 2001, 544, 1), (1024, 1024, 1056, 3), (2048, 4100, 576, 1),
    (1024, 1000, 320, 1), (1025, 2047, 128, 1), (413, 741, 160, 12), (999, 2300, 256, 1), (1500, 1500, 2080, 1)])
def test_gemm_tiles_whose_operands_go_straight_to_lds(env, m, n, k, batch):
    """Products between a few small tiles and one large tile per compute unit, while no
    best-effort job is there: fewer stages than the ring has places, as many and more, odd and even, a last
    stage half full, rows and columns past the matrix, bands of tiles that are cut short; and the tiles taken
    beside a job (here a stopped one) give the same bits."""
    B, ctx, torch = env
    test_gemm_one_wave_tiles_of_two_blocks(env, m, n, k, batch)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n + k)
    A = torch.randn(batch, m, k, device="cuda", generator=gen).to(torch.bfloat16)
    Bt = torch.randn(batch, n, k, device="cuda", generator=gen).to(torch.bfloat16)
    C = torch.full((batch, m, n), 7.0, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C, small=True)
    x, y = torch.zeros(4096, device="cuda"), torch.zeros(4096, device="cuda")
    torch.cuda.synchronize()
    ctx.launch_native(kern)
    torch.cuda.synchronize()
    alone = C.clone()
    C.fill_(7.0)
    torch.cuda.synchronize()
    job = ctx.launch_ptb(B.saxpy(x, y, 1.0), 1, stop_at=3)
    assert job.wait() == B.JOB_STOPPED
    ctx.launch_native(kern, hi=True)
    torch.cuda.synchronize()
    job.resume()
    job.wait()
    job.free()
    assert torch.equal(C, alone)


@pytest.mark.parametrize("tile,m,n,k,batch", [
    ("256", 256, 256, 96, 1), ("256", 512, 512, 1056, 1), ("256", 512, 768, 288, 1), ("256", 1024, 1024, 544, 1),
    ("256", 1024, 2048, 2080, 1), ("256", 2048, 2048, 64, 1), ("256", 4352, 4864, 96, 1), ("256", 1280, 1280, 2048, 1),
    ("128", 256, 384, 1056, 1), ("128", 512, 768, 2048, 3), ("small", 100, 300, 416, 2), ("small", 300, 1000, 1024, 1),
    ("small", 1000, 2300, 768, 1), ("small", 130, 65, 96, 128), ("small", 127, 129, 224, 171)])
def test_gemm_bits_do_not_depend_on_form_or_schedule(env, tile, m, n, k, batch):
    """Every tile that any form covers the product with adds in the same order: one worker, several,
    enough for parts of blocks, jobs stopped so near the end that the rest is done in parts, slices
    and the original form give the same bits, those of a NaN included (0x7FC0 in the ragged GEMM)."""
    B, ctx, torch = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n + k)
    A = torch.randn(batch, m, k, device="cuda", generator=gen).to(torch.bfloat16)
    Bt = torch.randn(batch, n, k, device="cuda", generator=gen).to(torch.bfloat16)
    A[:, ::37, 3] = float("inf")                          # times a zero, and times anything else
    Bt[:, ::11, 3] = 0.0
    C = torch.empty(batch, m, n, dtype=torch.bfloat16, device="cuda")
    kern = B.gemm_bf16(A, Bt, C, small=tile == "small", n128=tile == "128")
    total = kern.total_blocks

    def bits(launch):
        C.fill_(7.0)
        torch.cuda.synchronize()
        job = launch()
        while job is not None and job.wait() != B.JOB_COMPLETE:
            job.resume()
        if job is not None:
            job.free()
        torch.cuda.synchronize()
        return C.view(torch.int16).clone()

    want = bits(lambda: ctx.launch_ptb(kern, 1))
    nan = want[:, ::37, ::11]
    assert bool(((nan & 0x7FFF) > 0x7F80).all()) and (tile != "small" or bool((nan == 0x7FC0).all()))
    for what, launch in [("native", lambda: ctx.launch_native(kern)), ("slices", lambda: ctx.launch_sliced(kern, total // 3 + 1)),
                         ("5 workers", lambda: ctx.launch_ptb(kern, 5)), ("256 workers", lambda: ctx.launch_ptb(kern, 256)),
                         ("1 block left", lambda: ctx.launch_ptb(kern, 256, stop_at=total - 1)),
                         ("3 blocks left", lambda: ctx.launch_ptb(kern, 256, stop_at=max(total - 3, 0)))]:
        assert torch.equal(bits(launch), want), what


@pytest.mark.parametrize("tile,cover", list(GEMM_TILES))
def test_every_tile_that_covers_a_product(env, tile, cover):
    for shape in GEMM_TILES[tile, cover]:
        test_gemm_bits_do_not_depend_on_form_or_schedule(env, tile, *shape)


# ------------------------------------------------------------------ GEMV
@pytest.mark.parametrize("n,k,form", [(130, 96, "native"), (130, 96, "ptb_preempted"),
                                      (4096, 4096, "native_hi"), (4096, 11008, "native_hi"),
                                      (11008, 4096, "native_hi"), (1000, 2056, "sliced"),
                                      # the original form takes a row in batches of eight, then four
                                      # loads per lane, then singles: rows shorter than a batch, fewer
                                      # rows than a workgroup has waves, ragged ends of every loop
                                      (5, 8, "native"), (3, 520, "native_hi"), (1031, 4104, "native"),
                                      (300, 11264, "native_hi"), (37, 11272, "native")])
def test_gemv(env, n, k, form):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    g = TI.gemv_inputs(n=n, k=k, scale=1 / 64 if k == 4096 and n == 4096 else 0.02, config_index=1)
    a = dict(g, y=np.zeros(n, np.uint16))
    OS.run_native("gemv_bf16", OK.grid_of("gemv_bf16", a), a)
    x, W, y = dev(g["x"]), dev(g["W"]), dev(np.zeros(n, np.uint16))
    torch.cuda.synchronize()
    _run_form(B, ctx, torch, B.gemv_bf16(x, W, y), form)
    assert_bf16_close(host(y), a["y"])


@pytest.mark.parametrize("k", [8, 504, 512, 520, 1024, 1032, 1536, 1544, 2040, 2048, 2056, 2560, 2568, 3072, 3080, 3584, 3592, 4088, 4096, 4104, 6152, 8200, 11008])
def test_gemv_row_ends(env, k):
    """Every number of vectors that a lane can have left behind the whole batches, each with the last one whole,
    one lane and all but one: nothing beyond a row or x is read (NaNs lie there), and both forms give the same bits."""
    B, ctx, torch = env
    n = 9
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    wide = torch.full((n * k + 4096,), float("nan"), device="cuda", dtype=torch.bfloat16)
    wide[:n * k] = torch.randn(n * k, device="cuda", generator=g).to(torch.bfloat16)
    xs = torch.full((k + 4096,), float("nan"), device="cuda", dtype=torch.bfloat16)
    xs[:k] = torch.randn(k, device="cuda", generator=g).to(torch.bfloat16)
    W, x = wide[:n * k].view(n, k), xs[:k]
    y, z = (torch.zeros(n, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    torch.cuda.synchronize()
    _run_form(B, ctx, torch, B.gemv_bf16(x, W, y), "native")
    _run_form(B, ctx, torch, B.gemv_bf16(x, W, z), "ptb")
    assert torch.equal(y.view(torch.int16), z.view(torch.int16))
    p = W.double() * x.double()
    # one bf16 rounding, and k fp32 additions of at most the sum of magnitudes
    bound = p.sum(1).abs() * 2.0 ** -8 + k * 2.0 ** -24 * p.abs().sum(1)
    assert ((y.double() - p.sum(1)).abs() <= bound).all()


# ------------------------------------------------------------------ softmax / LayerNorm
@pytest.mark.parametrize("rows,cols,form", [(37, 2048, "native"), (37, 2048, "ptb_preempted"),
                                            (37, 2048, "sliced"), (1536, 128, "native_hi"),
                                            (9, 8192, "ptb"), (5, 100, "native"),
                                            (3, 4096, "native")])
def test_softmax(env, rows, cols, form):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_close_rel
    xs = TI.rows_f32(rows, cols, scale=2.0, config_index=3)
    xs[0, :] = 0.25                                       # constant row
    xs[rows - 1, 0] = 60.0                                # one dominant entry
    a = {"x": xs, "y": np.zeros_like(xs), "rows": rows, "cols": cols}
    OS.run_native("softmax_f32", OK.grid_of("softmax_f32", a), a)
    x, y = dev(xs), dev(np.zeros_like(xs))
    torch.cuda.synchronize()
    _run_form(B, ctx, torch, B.softmax_f32(x, y), form)
    got = host(y)
    assert_close_rel(got, a["y"], 1e-5, 1e-7)
    assert np.allclose(got.sum(axis=1, dtype=np.float64), 1.0, atol=1e-5)


@pytest.mark.parametrize("rows,cols,form", [(41, 4096, "native"), (41, 4096, "ptb_preempted"),
                                            (41, 4096, "sliced"), (128, 768, "native_hi"),
                                            (6, 8192, "ptb"), (5, 100, "native")])
def test_layernorm(env, rows, cols, form):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_close_rel
    li = TI.layernorm_inputs(rows, cols, scale=1.0)
    a = dict(li, y=np.zeros_like(li["x"]))
    OS.run_native("layernorm_f32", OK.grid_of("layernorm_f32", a), a)
    x, g, b, y = dev(li["x"]), dev(li["gamma"]), dev(li["beta"]), dev(np.zeros_like(li["x"]))
    torch.cuda.synchronize()
    _run_form(B, ctx, torch, B.layernorm_f32(x, g, b, y, li["eps"]), form)
    assert_close_rel(host(y), a["y"], 1e-5, 2e-6)


@pytest.mark.parametrize("cols", [4, 100, 256, 260, 512, 516, 1024, 1028, 2048, 2052, 4096, 4100, 8188, 8192])
@pytest.mark.parametrize("op", ["softmax", "layernorm"])
def test_rows_width_edges(env, op, cols):
    """Both sides of every width at which the kernel or the registers per lane change, an odd
    number of rows, workers that take several blocks at once (rows in flight, a last fetch cut
    short), one worker with the whole grid, slices; negative rows (a lane past the end must not
    count as zero); nothing is written behind the last row; in place."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_close_rel
    rows = 61
    if op == "softmax":
        xs = TI.rows_f32(rows, cols, scale=2.0, config_index=3)
        xs[1::3] -= 50.0
        a = {"x": xs, "y": np.zeros_like(xs), "rows": rows, "cols": cols}
        make, abs_ = lambda x, y: B.softmax_f32(x, y), 1e-7
        OS.run_native("softmax_f32", OK.grid_of("softmax_f32", a), a)
    else:
        li = TI.layernorm_inputs(rows, cols, scale=1.0)
        xs, a = li["x"], dict(li, y=np.zeros_like(li["x"]))
        g, b = dev(li["gamma"]), dev(li["beta"])
        make, abs_ = lambda x, y: B.layernorm_f32(x, g, b, y, li["eps"]), 2e-6
        OS.run_native("layernorm_f32", OK.grid_of("layernorm_f32", a), a)
    for workers, chunk in [(None, 0), (None, 5), (3, 3), (1, 64), (2, 1)]:
        buf = torch.full((rows + 1, cols), 7.0, device="cuda")
        y = buf[:rows]
        x = dev(xs) if chunk != 3 else y                  # (3, 3): in place
        y.copy_(dev(xs))
        torch.cuda.synchronize()
        kern = make(x, y)
        if workers:
            job = ctx.launch_ptb(kern, workers, chunk=chunk)
        elif chunk:
            job = ctx.launch_sliced(kern, chunk)
        else:
            job = None
            ctx.launch_native(kern)
        if job:
            assert job.wait() == B.JOB_COMPLETE
            job.free()
        torch.cuda.synchronize()
        assert_close_rel(host(y), a["y"], 1e-5, abs_)
        assert (host(buf[rows]) == 7.0).all()


@pytest.mark.parametrize("op", ["softmax", "layernorm"])
def test_rows_up_to_the_largest_count(env, op):
    """2^32 - 1 rows (2^30 blocks, the most a grid may have, 64 GiB in place): the last block's end
    has no 32-bit row number, and neither has the row after the last one that a worker asks for.
    Every row is the same, so the oracle's first rows are all of it; a row that is run twice in
    place would differ."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_close_rel
    rows, cols = 2**32 - 1, 4
    one = np.array([[0.5, -1.0, 2.0, 0.0]], np.float32)
    x = torch.empty((rows, cols), device="cuda")
    x.copy_(dev(one).expand(rows, cols))
    if op == "softmax":
        a = {"x": one, "y": np.zeros_like(one), "rows": 1, "cols": cols}
        kern = B.softmax_f32(x, x)
        OS.run_native("softmax_f32", OK.grid_of("softmax_f32", a), a)
    else:
        g, b = np.ones(cols, np.float32), np.zeros(cols, np.float32)
        a = {"x": one, "y": np.zeros_like(one), "gamma": g, "beta": b, "rows": 1, "cols": cols, "eps": 1e-5}
        kern = B.layernorm_f32(x, dev(g), dev(b), x, 1e-5)
        OS.run_native("layernorm_f32", OK.grid_of("layernorm_f32", a), a)
    assert kern.total_blocks == 2**30
    torch.cuda.synchronize()
    job = ctx.launch_ptb(kern, 512, chunk=4096)
    assert job.wait() == B.JOB_COMPLETE
    job.free()
    torch.cuda.synchronize()
    assert_close_rel(host(x[:1]), a["y"], 1e-5, 2e-6)
    assert bool((x == x[:1]).all())
    kern = x = None
    torch.cuda.empty_cache()


@pytest.mark.parametrize("count", [1, 3, 4, 5, 1023, 8191, 8192, 8197, 65536, 70001])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_reduce_final_edges(env, count, offset):
    """Fewer partials than a vector, ends of a trip of 2048 vectors, starts off a 16-byte
    boundary; doubles hold the sum of these floats to 2^-50 of the largest partial sum."""
    B, ctx, torch = env
    from gpu_util import dev, host
    p = TI.reduce_inputs(n=count + offset + 1, config_index=2)["x"].reshape(-1)
    buf = dev(p)
    total = dev(np.zeros(1, np.float64))
    torch.cuda.synchronize()
    ctx.launch_native(B.reduce_final(buf[offset:offset + count], total))
    torch.cuda.synchronize()
    want = float(np.sum(p[offset:offset + count].astype(np.float64)))
    assert abs(host(total)[0] - want) <= 1e-12 * max(1.0, abs(want))


# ------------------------------------------------------------------ decode attention
@pytest.mark.parametrize("tokens,heads,scale", [(2048, 32, 0.02), (777, 3, 1.0), (5, 2, 1.0)])
def test_attn_decode(env, tokens, heads, scale):
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    at = TI.attn_decode_inputs(tokens, heads, 128, scale=scale)
    a = dict(at, out=np.zeros((heads, 128), np.uint16))
    OS.run_native("attn_decode_bf16", OK.grid_of("attn_decode_bf16", a), a)
    q, Kc, Vc = dev(at["q"]), dev(at["K"]), dev(at["V"])
    out = dev(np.zeros((heads, 128), np.uint16))
    scratch = torch.zeros(B.attn_decode_scratch_bytes(heads), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    kern = B.attn_decode_bf16(q, Kc, Vc, out, scratch)
    ctx.launch_native(kern, hi=True)
    torch.cuda.synchronize()
    assert_bf16_close(host(out), a["out"])
    # the scratch serves later calls as it is
    first = host(out).copy()
    for _ in range(3):
        out.zero_()
        ctx.launch_native(kern, hi=True)
    torch.cuda.synchronize()
    assert (host(out) == first).all()


@pytest.mark.parametrize("tokens,heads", [(3840, 3), (3841, 3), (4081, 16), (4096, 17), (9001, 4)])
def test_attn_decode_waves_per_workgroup(env, tokens, heads):
    """Both sides of the lines between four and eight waves per workgroup (16 heads, 256 tokens per
    workgroup), a last split that is short or nearly empty."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    at = TI.attn_decode_inputs(tokens, heads, 128, scale=0.5)
    a = dict(at, out=np.zeros((heads, 128), np.uint16))
    OS.run_native("attn_decode_bf16", OK.grid_of("attn_decode_bf16", a), a)
    out = dev(np.zeros((heads, 128), np.uint16))
    scratch = torch.full((B.attn_decode_scratch_bytes(heads),), 0xFF, dtype=torch.uint8, device="cuda")
    q, Kc, Vc = dev(at["q"]), dev(at["K"]), dev(at["V"])
    torch.cuda.synchronize()
    ctx.launch_native(B.attn_decode_bf16(q, Kc, Vc, out, scratch), hi=True)
    torch.cuda.synchronize()
    assert_bf16_close(host(out), a["out"])


def test_attn_decode_longest_cache(env):
    """16 splits x 2048 tokens is the longest cache one call takes; one token more is refused."""
    B, ctx, torch = env
    from gpu_util import dev, host, assert_bf16_close
    tokens, heads = 16 * 2048, 2
    at = TI.attn_decode_inputs(tokens, heads, 128, scale=0.5)
    a = dict(at, out=np.zeros((heads, 128), np.uint16))
    OS.run_native("attn_decode_bf16", OK.grid_of("attn_decode_bf16", a), a)
    q, Kc, Vc = dev(at["q"]), dev(at["K"]), dev(at["V"])
    out = dev(np.zeros((heads, 128), np.uint16))
    scratch = torch.zeros(B.attn_decode_scratch_bytes(heads), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    ctx.launch_native(B.attn_decode_bf16(q, Kc, Vc, out, scratch), hi=True)
    torch.cuda.synchronize()
    assert_bf16_close(host(out), a["out"])
    Kbig = torch.zeros((tokens + 1, heads, 128), dtype=torch.int16, device="cuda")
    with pytest.raises(B.TallyError):
        B.attn_decode_bf16(q, Kbig, Kbig, out, scratch)
