"""CPU-side checks: the shared library loads, exports every symbol the header declares,
and its host-only functions (Eq. 1, selection rule) agree with the oracle."""
import os
import re

import pytest

from oracle import profiler as OP

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def B():
    import paper_2410_07381_amd.binding as B
    return B


def test_library_exports_every_declared_symbol(B):
    hdr = open(os.path.join(ROOT, "include", "tally.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(tally_[a-z0-9_]+)\s*\(", hdr))
    assert len(declared) >= 25
    for name in sorted(declared):
        assert hasattr(B.lib(), name), f"{name} is declared in tally.h but not exported"
    assert declared == set(B.EXPORTS)


def test_struct_sizes_match_the_header(B):
    import ctypes as C
    assert C.sizeof(B.SaxpyArgs) == 24 and C.sizeof(B.ReduceSumArgs) == 24
    assert C.sizeof(B.GemmArgs) == 72 and C.sizeof(B.GemvArgs) == 32
    assert C.sizeof(B.CoverRec) == 24 and C.sizeof(B.Config) == 20
    assert C.sizeof(B.KernelDesc) == 48


@pytest.mark.parametrize("parts", [2, 4, 8, 16, 64])
def test_parts_of_a_block_that_did_not_run_once_each_show_in_its_count(B, parts):
    """Parts run any number of times, lost ones made up for by carries of others among them: only
    once each counts as one execution of the block."""
    import itertools
    import random
    w = 64 // parts

    def count(runs):
        which = sum(r * (((1 << w) - 1) << (p * w)) for p, r in enumerate(runs)) % 2**64
        return B.parts_executions(sum(runs) * w, which)

    assert count([1] * parts) == 1 and count([0] * parts) == 0
    if parts <= 8:
        cases = itertools.product(range(4), repeat=parts) if parts < 8 else itertools.product(range(3), repeat=8)
    else:
        rng = random.Random(parts)
        cases = [[rng.choice([0, 1, 1, 1, 2, 3]) for _ in range(parts)] for _ in range(2000)]
        for p in range(parts - 1):            # lost, doubled, and a sum that carries put right
            cases += [[1] * p + [0, 1] + [1] * (parts - p - 2), [1] * p + [2, 1] + [1] * (parts - p - 2),
                      [1] * p + [3, 0] + [1] * (parts - p - 2), [1] * p + [0, 2] + [1] * (parts - p - 2)]
        cases.append([2] * parts)
    for runs in cases:
        runs = list(runs)
        if any(r != 1 for r in runs) and any(runs):
            assert count(runs) == B.PARTS_UNEVEN, runs


def test_eq1_matches_oracle(B):
    for lat, w, c, tot in [(1.0, 256, 1, 65536), (2.0, 16, 1, 16), (0.5, 512, 4, 4096)]:
        assert B.ptb_turnaround_ms(lat, w, c, tot) == pytest.approx(
            OP.ptb_turnaround_ms(lat, w * c, tot), rel=1e-12)


def _m(kind, param, lat, turn):
    return {"kind": kind, "param": param, "latency_ms": lat, "turnaround_ms": turn}


@pytest.mark.parametrize("threshold", [0.0316, 1.0, 0.001, 0.0095])
def test_selection_rule_matches_oracle(B, threshold):
    ms = [_m(0, 256, 1.30, 0.005), _m(0, 512, 1.10, 0.010), _m(0, 2048, 1.00, 0.040),
          _m(1, 4096, 1.05, 0.066), _m(1, 512, 1.20, 0.009), _m(1, 64, 1.10, 0.010),
          _m(0, 128, 1.10, 0.010)]
    o = OP.select_config([dict(m, kind="ptb" if m["kind"] == 0 else "sliced") for m in ms], threshold)
    got = ms[B.select_config(ms, threshold)]
    assert (got["param"], got["kind"]) == (o["param"], 0 if o["kind"] == "ptb" else 1)


def test_error_strings_and_null_handling(B):
    assert B.lib().tally_strerror(0) == b"ok"
    assert b"invalid" in B.lib().tally_strerror(B.ERR_INVALID_ARG)
    assert B.lib().tally_select_config(None, 0, 1.0) == B.ERR_INVALID_ARG
    assert B.lib().tally_preempt(None) == B.ERR_INVALID_ARG
    assert B.lib().tally_job_free(None) == B.ERR_INVALID_ARG


def test_bench_refuses_more_than_one_gpu():
    """The method is a per-GPU mechanism and this build measures one GPU: asking for more
    ends with a message and a non-zero status, before anything touches a GPU."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=60)
    assert r.returncode == 2 and "one GPU" in r.stderr and r.stdout.strip() == ""


def test_entry_points_exist():
    import importlib
    g = importlib.import_module("__graft_entry__")
    assert callable(g.build) and callable(g.smoke)


def test_header_is_plain_c():
    """The boundary is a C ABI: the header compiles as C99 (and as C++) on its own, and a C
    program that only includes it sees the struct sizes the binding assumes."""
    import subprocess
    import tempfile
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    hdr = os.path.join(root, "include", "tally.h")
    for cc, std, lang in (("gcc", "-std=c99", "c"), ("g++", "-std=c++11", "c++")):
        r = subprocess.run([cc, std, "-Wall", "-Wextra", "-pedantic", "-fsyntax-only", "-x", lang, hdr],
                           capture_output=True, text=True, timeout=60)
        assert r.returncode == 0 and r.stderr.strip() == "", r.stderr
    prog = ('#include <stdio.h>\n#include "tally.h"\nint main(void){printf("%zu %zu %zu %zu %zu\\n",'
            'sizeof(tally_gemm_bf16_args),sizeof(tally_kernel_desc),sizeof(tally_cover_rec),'
            'sizeof(tally_config),sizeof(tally_sched_run_t));return 0;}\n')
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "s.c"), os.path.join(d, "s")
        open(src, "w").write(prog)
        subprocess.run(["gcc", "-std=c99", "-I", os.path.join(root, "include"), src, "-o", exe],
                       check=True, timeout=60)
        out = subprocess.run([exe], capture_output=True, text=True, timeout=10).stdout.split()
    import ctypes as C
    import paper_2410_07381_amd.binding as B
    assert [int(v) for v in out] == [C.sizeof(B.GemmArgs), C.sizeof(B.KernelDesc), C.sizeof(B.CoverRec),
                                     C.sizeof(B.Config), C.sizeof(B.SchedRun)]


def test_every_mirrored_struct_has_the_header_layout(B, tmp_path):
    """Field by field: a C program that includes only the header prints offsetof() of every
    field the binding's ctypes structures name (a field the header does not have fails to
    compile) and sizeof() of every structure; both must be what ctypes computed."""
    import ctypes as C
    import subprocess
    pairs = [(B.Dim3, "tally_dim3"), (B.SaxpyArgs, "tally_saxpy_args"),
             (B.ReduceSumArgs, "tally_reduce_sum_args"), (B.ReduceFinalArgs, "tally_reduce_final_args"),
             (B.GemmArgs, "tally_gemm_bf16_args"), (B.GemvArgs, "tally_gemv_bf16_args"),
             (B.SoftmaxArgs, "tally_softmax_f32_args"), (B.LayerNormArgs, "tally_layernorm_f32_args"),
             (B.AttnDecodeArgs, "tally_attn_decode_args"), (B.KernelDesc, "tally_kernel_desc"),
             (B.CoverRec, "tally_cover_rec"), (B.Config, "tally_config"), (B.BeItem, "tally_be_item"),
             (B.SchedRun, "tally_sched_run_t"), (B.SchedOpts, "tally_sched_opts"),
             (B.SchedStats, "tally_sched_stats_t")]
    lines, want = [], []
    for cls, cname in pairs:
        lines.append('printf("%%zu\\n", sizeof(%s));' % cname)
        want.append(C.sizeof(cls))
        for fname, _ in cls._fields_:
            lines.append('printf("%%zu\\n", offsetof(%s, %s));' % (cname, fname))
            want.append(getattr(cls, fname).offset)
    src = tmp_path / "layout.c"
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "tally.h"\nint main(void){\n'
                   + "\n".join(lines) + "\nreturn 0;}\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-I", os.path.join(root, "include"), str(src), "-o", str(exe)],
                   check=True, timeout=60)
    got = [int(v) for v in subprocess.run([str(exe)], capture_output=True, text=True, timeout=10).stdout.split()]
    assert got == want


def _device_code(B, tmp_path):
    """The built library's code object for the GPU, and a way to run one of the LLVM tools on it."""
    import subprocess
    llvm = "/opt/rocm/llvm/bin"
    tools = {t: os.path.join(llvm, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf", "llvm-objdump")}
    if not all(os.path.exists(t) for t in tools.values()):
        pytest.skip("LLVM binary tools not installed")
    fat, co = str(tmp_path / "fat.bin"), str(tmp_path / "dev.co")
    subprocess.run([tools["llvm-objcopy"], "-O", "binary", "--only-section=.hip_fatbin", B.LIB_PATH, fat], check=True)
    subprocess.run([tools["clang-offload-bundler"], "--unbundle", "--type=o", f"--input={fat}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={co}"], check=True)
    return lambda tool, *args: subprocess.run([tools[tool], *args, co], check=True, capture_output=True, text=True).stdout


def test_workers_write_gemm_outputs_past_the_caches(B, tmp_path):
    """The best-effort forms keep the caches for the high-priority job: workers write large blocks, and the
    parts of 32x64 to 128x128 that few blocks are handed out in, with non-temporal stores (the one or two
    other stores of 16 bytes in a kernel are those of the coverage record)."""
    run = _device_code(B, tmp_path)
    names = [l.split()[-1] for l in run("llvm-readelf", "-sW").splitlines() if " FUNC " in l and "ptb_kernel" in l]
    names = [n for n in names if "GemmRingT" in n or "GemmBodyT" in n]
    assert sum("GemmRingT" in n for n in names) >= 8 and any("GemmRingT" not in n for n in names)
    for name in names:
        code = run("llvm-objdump", "-d", f"--disassemble-symbols={name}")
        stores = [l for l in code.splitlines() if "store_dwordx4" in l]
        past = sum(" nt" in l for l in stores)
        assert past > 0 and len(stores) - past <= 2 and "store_short" not in code, name


def test_gemv_keeps_its_buffer_descriptors_in_scalar_registers(B, tmp_path):
    """The end of a row is read through a buffer that ends with it; were the row's number not known to be the
    same in a wave, each of those loads would be a loop over the lanes' descriptors."""
    run = _device_code(B, tmp_path)
    names = [l.split()[-1] for l in run("llvm-readelf", "-sW").splitlines() if " FUNC " in l and "native_kernel" in l and "GemvBody" in l]
    assert len(set(names)) == 1
    code = run("llvm-objdump", "-d", f"--disassemble-symbols={names[0]}")
    assert code.count("buffer_load_dwordx4") >= 2 * (1 + 2 + 3 + 4 + 5 + 6 + 7 + 8)
    assert code.count("v_readfirstlane_b32") <= 2


@pytest.fixture(scope="module")
def gemm_rules(tmp_path_factory):
    """The rules for the tiles of a GEMM as a program: for every m, n, k, batch, columns of the operator's large blocks
    (0: the ragged one) and what else is on the GPU, the tile that is chosen."""
    import subprocess
    src = tmp_path_factory.mktemp("rules") / "rules.cpp"
    src.write_text(r"""
#include <cstdio>
#include <set>
#include <tuple>
#include "gemm_cover.h"
using namespace tally;
int main() {
  const char *names[] = {"32x32", "32x64", "64x64", "128x64", "256x128", "256x256", "wave16", "wave16x32", "wave32x16"};
  const uint32_t tiles[][2] = {{16, 16}, {16, 32}, {32, 16}};
  tally_gemm_bf16_args a{};
  uint32_t large, how;
  while (scanf("%u %u %u %u %u %u", &a.m, &a.n, &a.k, &a.batch, &large, &how) == 6) {
    const int c = (int)(large ? gemm_cover(a, how, large) : gemm_cover_small(a, how)), ring = c - (int)GemmCover::kRing;
    // every tile of the output once, by the workgroups of the grid, and how many the busiest and the idlest die have
    std::set<std::tuple<uint32_t, uint32_t, uint32_t>> seen;
    size_t runs = 0, most = 0, least = ~(size_t)0, want = 0;
    uint32_t x, y, z, tm = 0, tn = 0;
    if (ring >= 0) { tm = kRings[ring][0]; tn = kRings[ring][1]; }
    else if (c >= (int)GemmCover::kWave16) { tm = tiles[c - (int)GemmCover::kWave16][0]; tn = tiles[c - (int)GemmCover::kWave16][1]; }
    if (tm) {
      const uint32_t X = cdiv(a.n, tn), Y = cdiv(a.m, tm), T = X * Y * a.batch;
      const uint32_t in = a.m > a.n ? X : Y, at = cdiv((uint64_t)(a.m > a.n ? Y : X) * a.batch, 8);
      want = T;
      for (uint32_t die = 0; die < 8; ++die) {
        size_t here = 0;
        if (ring >= 0) {
          for (uint32_t id = die; id < cdiv(T, 8) * 8; id += 8)
            if (ring_tile(a, tm, tn, id, &x, &y, &z)) { ++here; if (x < X && y < Y && z < a.batch) seen.insert({x, y, z}); }
        } else {
          for (uint32_t i = 0; i < in; ++i)
            for (uint32_t p = 0; p < at; ++p)
              if (wave_tile(a, tm, tn, die, i, p, &x, &y, &z)) { ++here; if (x < X && y < Y && z < a.batch) seen.insert({x, y, z}); }
        }
        runs += here;
        most = here > most ? here : most;
        least = here < least ? here : least;
      }
    }
    if (ring >= 0) printf("%ux%u/%u", kRings[ring][0], kRings[ring][1], kRings[ring][3]);
    else printf("%s", names[c]);
    printf(" %d %zu %zu\n", seen.size() == want && runs == want, most, least);
  }
  return 0;
}
""")
    exe = src.with_suffix("")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_07381_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", csrc, str(src), "-o", str(exe)], check=True, timeout=60)

    def rules(cases):
        lines = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True,
                               check=True, timeout=60).stdout.split("\n")
        return [(l.split()[0], *map(int, l.split()[1:])) for l in lines if l]
    return rules


LARGE = {"small": 0, "128": 128, "256": 256}
SHARED, BESIDE = 4, 2                     # as in gemm_cover.h


def test_the_shapes_of_each_tile_reach_it(gemm_rules):
    """The GPU tests run every kernel that an original form chooses from; a rule that changes shows here."""
    from gemm_tiles import GEMM_TILES
    cases = [(key, s) for key, shapes in GEMM_TILES.items() for s in shapes]
    for (key, s), got in zip(cases, gemm_rules([(*s, LARGE[key[0]], 0) for key, s in cases])):
        assert got[0] == key[1] and got[1] == 1, (key, s, got)
    rings = {"32x32/8", "32x64/6", "64x64/5", "64x96/4", "128x64/3", "96x96/3", "128x64/5", "96x96/5", "128x96/4", "128x128/4"}
    for tile in LARGE:
        assert {c for t, c in GEMM_TILES if t == tile} >= rings | {"wave16", "wave16x32", "wave32x16"}


def test_gemm_tiles_are_dealt_out_to_all_dies(gemm_rules):
    """Each tile goes to one workgroup, and no die has more than a panel, or a tile, beyond its share: for tall and
    wide outputs, few panels, batches."""
    import random
    rng = random.Random(1)
    cases = [(8192, 16, 1536, 1), (2032, 112, 1536, 1), (4096, 32, 2048, 1), (16, 8192, 768, 1), (17, 16, 768, 50), (1, 1, 768, 1)]
    cases += [(rng.randint(1, 2500), rng.randint(1, 2500), 32 * rng.randint(5, 60), rng.choice([1, 1, 3, 12])) for _ in range(400)]
    cases += [(rng.randint(1, 5000), rng.randint(1, 60), 32 * rng.randint(5, 60), rng.choice([1, 1, 3, 12])) for _ in range(200)]
    for (m, n, k, batch), (tile, once, most, least) in zip(cases, gemm_rules([(*c, 0, 0) for c in cases])):
        if tile in ("64x64", "128x64", "32x32", "32x64"):
            continue                                       # (a plain grid)
        assert once == 1, (m, n, k, batch)
        if tile.startswith("wave"):
            tm, tn = {"wave16": (16, 16), "wave16x32": (16, 32), "wave32x16": (32, 16)}[tile]
            panel = -(-n // tn) if m > n else -(-m // tm)
            assert most - least <= panel and panel <= 64, (m, n, k, batch)
        else:
            assert most - least <= 1, (m, n, k, batch)


def test_products_beside_others_take_tiles_that_fit_there(gemm_rules):
    """Beside best-effort workgroups no tile needs more than a 16x16 one of a wave or those through registers have."""
    import random
    rng = random.Random(2)
    cases = [(rng.randint(1, 3000), rng.randint(1, 3000), 32 * rng.randint(1, 130), rng.choice([1, 1, 3, 12])) for _ in range(400)]
    for how in (SHARED, SHARED | BESIDE):
        for (m, n, k, batch), got in zip(cases, gemm_rules([(*c, 0, how) for c in cases])):
            assert "/" not in got[0]
            if how & BESIDE and got[0].startswith("wave"):
                assert got[0] == "wave16" and -(-m // 16) * -(-n // 16) * batch <= 256


def test_a_client_that_a_request_holds_back_keeps_its_place(tmp_path):
    """Best-effort clients are served first come, first served.  One whose turn has come while a request arrives
    is not launched; it goes on waiting in its place and not behind those that came later."""
    import subprocess
    src = tmp_path / "admission.cpp"
    src.write_text(r"""
#include <cstdio>
#include "admission.h"
struct Client { uint64_t ticket = 0; tally::Demand resident{0, 0, 0}; };
int main() {
  Client c[3];
  uint64_t last = 0;
  const tally::Demand whole{131072, 4, 352}, small{16384, 4, 64};
  auto go = [&](uint32_t i, const tally::Demand &d, bool request) {
    const bool in = tally::admit(c, 3, i, d, 163840, &last, [&]() { return !request; });
    if (in) c[i].resident = d;
    return (int)in;
  };
  int r[9];
  r[0] = go(0, whole, false);              // 0 has the GPU
  r[1] = go(1, whole, false);              // 1 waits, then 2
  r[2] = go(2, small, false);
  c[0].resident = {0, 0, 0};               // 0 leaves
  r[3] = go(2, small, false);              // not before 1
  r[4] = go(1, whole, true);               // 1's turn, and a request arrives
  r[5] = go(2, small, false);              // still not before 1
  r[6] = go(0, whole, false);              // 0 comes again, behind both
  r[7] = go(1, whole, false);
  r[8] = go(2, small, false);              // fits beside 1
  for (int i = 0; i < 9; ++i) printf("%d ", r[i]);
  return 0;
}
""")
    exe = tmp_path / "admission"
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_07381_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(src), "-o", str(exe)], check=True, timeout=60)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=10).stdout.split()
    assert out == list("100000011")


def test_static_scratch_is_a_global_symbol_of_the_device_code(B, tmp_path):
    """The runtime finds a device variable by name among the code object's global symbols.
    A file-scope static device array referenced from host code is given global binding by
    the compiler; attributes that keep it local (an unnamed namespace, `used`) make the
    lookup at context creation fail.  Checked on the built library, no GPU needed."""
    import shutil
    import subprocess
    llvm = "/opt/rocm/llvm/bin"
    tools = [os.path.join(llvm, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
    if not all(os.path.exists(t) for t in tools):
        pytest.skip("LLVM binary tools not installed")
    fat, co = str(tmp_path / "fat.bin"), str(tmp_path / "dev.co")
    subprocess.run([tools[0], "-O", "binary", "--only-section=.hip_fatbin", B.LIB_PATH, fat], check=True)
    subprocess.run([tools[1], "--unbundle", "--type=o", f"--input={fat}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={co}"], check=True)
    syms = subprocess.run([tools[2], "-s", co], check=True, capture_output=True, text=True).stdout
    rows = [l.split() for l in syms.splitlines() if "static_scratch" in l]
    assert rows, "the static scratch array is missing from the device code"
    assert all(r[4] == "GLOBAL" and r[3] == "OBJECT" for r in rows), rows
    assert int(rows[0][2]) == 128 * 16 * 130 * 4
