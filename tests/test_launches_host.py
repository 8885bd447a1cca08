"""What the library launches for calls of sizes that no test runs, on the CPU: a recorder takes the place of the HIP runtime's
launch functions, refuses what no launch takes (2^32 lanes in one dimension), and writes down the rest.  Pointers are never followed."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORDER = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } Dim;
static struct { const void* f; const char* name; } known[4096];
static int count, error;
static Dim grid, block;
static void* handle;
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void* s) { (void)lds; (void)s; grid = g; block = b; return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* lds, void** s) { *g = grid; *b = block; *lds = 0; *s = NULL; return 0; }
void** __hipRegisterFatBinary(const void* d) { (void)d; return &handle; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterVar(void** h, void* v, char* a, char* b, int e, size_t s, int c, int g) {
  (void)h; (void)v; (void)a; (void)b; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** h, const void* f, char* d, const char* name, unsigned t, void* a, void* b, void* c, void* e, int* w) {
  (void)h; (void)d; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
  if (count < 4096) { known[count].f = f; known[count++].name = name; }
}
int hipGetLastError(void) { int e = error; error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)256; return 0; }
int hipLaunchKernel(const void* f, Dim g, Dim b, void** args, size_t lds, void* s) {
  const char* name = "?";
  int i;
  (void)lds; (void)s;
  for (i = 0; i < count; ++i) if (known[i].f == f) name = known[i].name;
  if ((uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32 || (uint64_t)g.z * b.z >> 32 || !g.x || !g.y || !g.z) {
    error = 9;
    return 9;
  }
  printf("[\"%s\", %u, %u, %u, %u", name, g.x, g.y, g.z, b.x);
  if (strstr(name, "WalkArgs"))                /* its first 13 words: pointers, sizes, first id, seed, length */
    for (i = 0; i < 13; ++i) printf(", %llu", ((unsigned long long*)args[0])[i]);
  printf("]\n");
  fflush(stdout);
  return 0;
}
"""

CALLS = """
import ctypes as C, json, sys
C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)        # its symbols come before those of the HIP runtime
lib = C.CDLL(sys.argv[2])
class Csr(C.Structure):
    _fields_ = [("num_nodes", C.c_int64), ("num_entries", C.c_int64), ("offsets", C.c_void_p), ("offset_bits", C.c_int32),
                ("nbrs", C.c_void_p), ("weights", C.c_void_p)]
class Alias(C.Structure):
    _fields_ = [("prob", C.c_void_p), ("alias", C.c_void_p), ("packed", C.c_void_p)]
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """launches(code): runs `code` behind the recorder; returns the recorded launches and what it printed as "rc"."""
    from paper_2407_15452_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build_lib()
    where = tmp_path_factory.mktemp("recorder")
    (where / "recorder.c").write_text(RECORDER)
    shim = str(where / "recorder.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", shim, str(where / "recorder.c")], check=True)

    def run(code):
        r = subprocess.run([sys.executable, "-c", CALLS + code, shim, binding.LIB_PATH], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        lines = [json.loads(line) for line in r.stdout.splitlines()]
        return [x for x in lines if isinstance(x, list)], [x["rc"] for x in lines if isinstance(x, dict)]

    return run


@pytest.mark.parametrize("walks", [(1 << 28) - 1, (1 << 28) + 1, 1 << 30, (1 << 32) + 5])
@pytest.mark.parametrize("weighted", [False, True])
def test_walks_beyond_one_launch(launches, walks, weighted):
    """Every number of walks that is accepted is launched, each walk once, whatever the lanes per walk: 2^30 walks at 4 lanes
    are 2^32 lanes, which one launch does not take."""
    length, first_id, starts, out = 10, 77, 1 << 40, 1 << 44
    for bits in (32, 64):
        for p, q in ((None, None), (0.5, 2.0), (1.0, 2.0), (1.0, 0.5), (1.0, 1.0)):
            call = ("gs_node2vec_walk(C.byref(g), a, C.c_void_p(%d), C.c_int64(%d), C.c_uint64(%d), C.c_int32(%d), C.c_float(%r), "
                    "C.c_float(%r), C.c_uint64(5), C.c_void_p(%d), None)" % (starts, walks, first_id, length, p, q, out) if p else
                    "gs_random_walk(C.byref(g), a, C.c_void_p(%d), C.c_int64(%d), C.c_uint64(%d), C.c_int32(%d), C.c_uint64(5), "
                    "C.c_void_p(%d), None)" % (starts, walks, first_id, length, out))
            got, rc = launches("g = Csr(1000, 9000, 256, %d, 512, None)\na = %s\nprint(json.dumps({'rc': lib.%s}))\n" % (
                bits, "C.byref(Alias(768, 1024, 1280))" if weighted else "None", call))
            assert rc == [0], (bits, p, q)
            done = 0
            for name, gx, gy, gz, threads, *args in got:
                part = args[9]
                assert args[5] == starts + 4 * done and args[6] == out + 4 * done * length and args[10] == first_id + done
                assert gy == gz == 1 and gx * threads >= part > 0
                done += part
            assert done == walks


@pytest.mark.parametrize("weighted,entries,walks,p,q,lanes", [
    (True, 9 << 20, 114_688, 1.0, 0.5, 4), (True, 9 << 20, 114_689, 1.0, 0.5, 2), (True, 9 << 20, 229_377, 1.0, 0.5, 1),
    (True, 9 << 20, 114_689, 4.0, 0.25, 2), (True, 1 << 23, 262_144, 4.0, 0.25, 4), (True, 1 << 20, 524_288, 4.0, 0.25, 4),
    (True, 9 << 20, 4_000_000, 1.0, 0.5, 1), (True, 1 << 20, 4_000_000, 1.0, 0.5, 1), (True, 1 << 21, 4_000_000, 4.0, 0.25, 2),
    (True, 9 << 20, 1_048_577, 4.0, 0.25, 1), (False, 9 << 20, 260_000, 1.0, 0.5, 2), (False, 9 << 20, 524_289, 1.0, 0.5, 1),
    (False, 9 << 20, 1_048_576, 4.0, 0.25, 2), (False, 9 << 20, 1_048_577, 4.0, 0.25, 1), (False, 1 << 20, 1_048_577, 1.0, 0.5, 0),
    (False, 1 << 21, 1_048_577, 4.0, 0.25, 0), (False, 1 << 21, 1_048_577, 1.0, 0.5, 1), (False, 3, 1_048_577, 4.0, 0.25, 1),
    (True, 9 << 20, 262_144, 1.0, 2.0, 4), (True, 9 << 20, 262_145, 1.0, 2.0, 2), (False, 9 << 20, 262_145, 1.0, 2.0, 0),
    (True, 9 << 20, 4_000_000, 0.5, 2.0, 4), (False, 9 << 20, 163_841, 0.5, 2.0, 0)])
def test_lanes_per_walk(launches, weighted, entries, walks, p, q, lanes):
    """Launches of many walks that take few attempts a step take narrower teams than those that take many (0: the state machine)."""
    got, rc = launches("g = Csr(100000, %d, 256, 32, 512, None)\na = %s\nprint(json.dumps({'rc': lib.gs_node2vec_walk(C.byref(g), a, "
                       "C.c_void_p(256), C.c_int64(%d), C.c_uint64(0), C.c_int32(10), C.c_float(%r), C.c_float(%r), C.c_uint64(5), "
                       "C.c_void_p(512), None)}))\n" % (entries, "C.byref(Alias(768, 1024, 1280))" if weighted else "None", walks, p, q))
    assert rc == [0] and len(got) == 1
    assert ("node2vec_team_kernelIiiLb%dELi%dE" % (weighted, lanes) if lanes else "node2vec_kernelIii") in got[0][0]


@pytest.mark.parametrize("walks", [100, 200_000])
def test_width_of_positions(launches, walks):
    """64-bit arithmetic only for graphs of 2^31 entries and more, not for all with 64-bit offsets."""
    for bits, entries, types in ((32, (1 << 31) - 1, "ii"), (64, (1 << 31) - 1, "li"), (64, 1 << 31, "ll")):
        got, rc = launches("g = Csr(100000, %d, 256, %d, 512, None)\nprint(json.dumps({'rc': lib.gs_node2vec_walk(C.byref(g), None, "
                           "C.c_void_p(256), C.c_int64(%d), C.c_uint64(0), C.c_int32(10), C.c_float(0.5), C.c_float(2.0), "
                           "C.c_uint64(5), C.c_void_p(512), None)}))\n" % (entries, bits, walks))
        assert rc == [0] and len(got) == 1 and ("kernelI" + types) in got[0][0], got


STEP = """
def step(call, pairs, nodes, dim, dtype=0, k=5, ws=1 << 50):
    p = [C.c_void_p(1 << (20 + i)) for i in range(12)]
    head = p[:{'gs_sgns_step': 2, 'gs_sgns_momentum_step': 4, 'gs_sgns_adam_step': 6}[call]]
    rates = {'gs_sgns_step': [0.1], 'gs_sgns_momentum_step': [0.1, 0.9], 'gs_sgns_adam_step': [0.1, 0.9, 0.999, 1e-8]}[call]
    tail = [C.c_int64(3)] if call == 'gs_sgns_adam_step' else []
    form = [C.c_int32(dtype)] if call != 'gs_sgns_adam_step' else []
    return getattr(lib, call)(*head, C.c_int64(nodes), C.c_int32(dim), *form, *p[6:9], C.c_int64(pairs), C.c_int32(k),
                              *[C.c_float(r) for r in rates], *tail, p[9], p[10], C.c_size_t(ws), None)
"""


@pytest.mark.parametrize("dtype,dim,pairs,more", [
    (0, 256, 49_152, False), (0, 256, 49_153, True), (0, 256, 65_536, True), (0, 256, 65_537, False), (0, 256, 98_304, False),
    (0, 256, 98_305, True), (0, 256, 131_072, True), (0, 256, 131_073, False), (0, 256, 600_000, False), (0, 128, 65_536, False),
    (1, 256, 49_152, False), (1, 256, 49_153, True), (1, 256, 72_000, True), (1, 256, 200_000, True), (2, 400, 32_769, True)])
def test_forward_waves(launches, dtype, dim, pairs, more):
    """The forward kernel for one more wave per SIMD: with fp32 tables where its waves come in fewer turns."""
    got, rc = launches(STEP + "print(json.dumps({'rc': step('gs_sgns_step', %d, 100000, %d, %d)}))\n" % (pairs, dim, dtype))
    assert rc == [0]
    forward = [x[0] for x in got if "sgns_forward_kernel" in x[0]]
    assert len(forward) == 1 and ("Li256ELi%dEEEv" % (0 if not more else (4 if dim <= 256 else 3))) in forward[0], forward


@pytest.mark.parametrize("pairs", [2_000, 100_000, 500_000])
@pytest.mark.parametrize("dtype,dim,k,rows", [(1, 256, 1, 2), (1, 136, 0, 2), (2, 200, 1, 2), (1, 256, 2, 6), (1, 512, 1, 2), (2, 264, 1, 2), (1, 512, 2, 4),
                                              (1, 128, 1, 6), (0, 256, 1, 3), (1, 520, 1, 2)])
def test_forward_rows_in_flight(launches, pairs, dtype, dim, k, rows):
    """16-bit rows: no block of rows much longer than the terms of a pair, all of whose reads are made."""
    got, rc = launches(STEP + "print(json.dumps({'rc': step('gs_sgns_step', %d, 100000, %d, %d, %d)}))\n" % (pairs, dim, dtype, k))
    assert rc == [0]
    (name,) = [x[0] for x in got if "sgns_forward_kernel" in x[0]]
    vpl = -(-dim // 64) if dim <= 64 else 2 if dim <= 128 else 4 if dim <= 256 else 8 if dim <= 512 else 16
    assert "Li%dELi%dE" % (vpl, rows) in name, name


@pytest.mark.parametrize("call,nodes,dim,dtype,once", [
    ("gs_sgns_momentum_step", 131_072, 128, 0, 0), ("gs_sgns_momentum_step", 131_073, 128, 0, 1),
    ("gs_sgns_momentum_step", 262_144, 128, 1, 0), ("gs_sgns_momentum_step", 262_145, 128, 2, 1),
    ("gs_sgns_adam_step", 87_381, 128, 0, 0), ("gs_sgns_adam_step", 87_382, 128, 0, 1),
    ("gs_sgns_adam_step", 139_810, 100, 0, 0), ("gs_sgns_adam_step", 139_811, 100, 0, 1)])
def test_dense_pass_past_the_caches(launches, call, nodes, dim, dtype, once):
    """Tables of more than 256 MB in all (320 MB where a workgroup's lanes are not whole rows), and no others, are read and
    written past the caches."""
    got, rc = launches(STEP + "print(json.dumps({'rc': step('%s', 50000, %d, %d, %d)}))\n" % (call, nodes, dim, dtype))
    assert rc == [0]
    dense = [x[0] for x in got if "dense_rest_kernel" in x[0]]
    assert len(dense) == 1 and ("ELb%dEEEv" % once) in dense[0], dense


@pytest.mark.parametrize("call", ["gs_sgns_momentum_step", "gs_sgns_adam_step"])
@pytest.mark.parametrize("dim,nodes", [(512, 33_554_432), (516, 33_554_432), (516, 33_554_433), (680, 50_331_651), (4, 2_000_000_000),
                                       (1024, 100_000_000)])
def test_dense_pass_reaches_every_row(launches, call, dim, nodes):
    """Launches in one layer and in several: as many workgroups as cover the rows (two per row's worth of lanes), at most one
    layer's remainder more, all within what a launch takes."""
    got, rc = launches(STEP + "print(json.dumps({'rc': step('%s', 50000, %d, %d)}))\n" % (call, nodes, dim))
    assert rc == [0]
    (name, gx, gy, gz, threads), = [x for x in got if "dense_rest_kernel" in x[0]]
    rows = 256 // (dim // 4) * 2
    assert gy == 2 and threads == 256 and 0 <= gx * gz * rows - nodes < rows * (gz + 1)
    assert gz == -(-(-(-nodes // rows)) // (1 << 23))


def test_launches_of_alias_tables(launches):
    """Short segments pay for the launches that other sizes would need; none of them only looks for long ones."""
    got, rc = launches("p = [C.c_void_p(1 << (20 + i)) for i in range(6)]\nprint(json.dumps({'rc': lib.gs_alias_build(p[0], C.c_int32(32), "
                       "C.c_int64(10000), C.c_int64(100000), *p[1:5], C.c_size_t(1 << 40), None)}))\n")
    assert rc == [0]
    names = [x[0].split("kernel")[0].split("gs")[1].lstrip("0123456789") for x in got]
    assert names == ["zero_u64_", "alias_build_", "alias_build_wave_", "alias_build_wave_", "alias_build_wave_", "alias_build_rows_"]


@pytest.mark.parametrize("segments", [(1 << 31) - 1, 1 << 31, (1 << 31) + 8])
def test_long_segments_among_very_many(launches, segments):
    """Sizes on the host are 64 bits wide: segments of more than 2048 entries are looked for however many segments there are."""
    got, rc = launches("p = [C.c_void_p(1 << (20 + i)) for i in range(6)]\nprint(json.dumps({'rc': lib.gs_alias_build(p[0], C.c_int32(64), "
                       "C.c_int64(%d), C.c_int64(1 << 33), *p[1:5], C.c_size_t(1 << 45), None)}))\n" % segments)
    assert rc == [0] and "alias_build_rows_kernel" in got[-1][0]


@pytest.mark.parametrize("call,pairs,nodes,k,how", [
    ("gs_sgns_step", 54_613, 65_536, 5, "place"), ("gs_sgns_step", 54_614, 65_536, 5, "group"), ("gs_sgns_step", 54_614, 65_537, 5, "place"),
    ("gs_sgns_step", 109_226, 65_537, 5, "place"), ("gs_sgns_step", 109_227, 65_537, 5, "group"), ("gs_sgns_step", 2_000_000, 1 << 24, 5, "group"),
    ("gs_sgns_step", 786_431, (1 << 24) + 1, 5, "place"), ("gs_sgns_step", 786_432, (1 << 24) + 1, 5, "radix"),
    ("gs_sgns_momentum_step", 109_227, 70_000, 5, "group"), ("gs_sgns_momentum_step", 786_432, (1 << 24) + 1, 5, "place"),
    ("gs_sgns_adam_step", 109_227, 70_000, 5, "group"), ("gs_sgns_adam_step", 109_226, 70_000, 5, "place")])
def test_ways_of_large_steps(launches, call, pairs, nodes, k, how):
    """Counters, grouped records (up to 2^24 rows) and sorted ones (beyond; without an optimizer)."""
    got, rc = launches(STEP + "print(json.dumps({'rc': step('%s', %d, %d, 64, 0, %d)}))\n" % (call, pairs, nodes, k))
    assert rc == [0]
    names = " ".join(x[0] for x in got)
    assert ("group_bucket_kernel" in names, "radix_scatter_kernel" in names, "sgns_clear_kernel" in names) == (
        how == "group", how == "radix", how != "group")


@pytest.mark.parametrize("call,pairs,nodes,how", [
    ("gs_sgns_step", 5_592_405, 1 << 24, "group"), ("gs_sgns_step", 5_592_406, 1 << 24, "radix"), ("gs_sgns_step", 20_000_000, 1 << 23, "group"),
    ("gs_sgns_step", 20_000_000, (1 << 23) + 1, "radix"), ("gs_sgns_step", 20_000_000, 5_000, "group"), ("gs_sgns_momentum_step", 5_592_406, 1 << 24, "group")])
def test_steps_beyond_the_buckets(launches, call, pairs, nodes, how):
    """More than 2^25 terms on more than 2^23 rows are sorted: each of the most buckets that there are would be split."""
    got, rc = launches(STEP + "print(json.dumps({'rc': step('%s', %d, %d, 8)}))\n" % (call, pairs, nodes))
    assert rc == [0]
    names = " ".join(x[0] for x in got)
    assert ("group_bucket_kernel" in names, "radix_scatter_kernel" in names) == (how == "group", how == "radix")


@pytest.mark.parametrize("n,nodes,few", [((3 << 19) - 1, 60_000, 1), (3 << 19, 60_000, 1), (3 << 20, 60_000, 1), ((3 << 20) + 1, 60_000, 0), (1 << 19, (1 << 20) - 1, 1), ((1 << 19) + 1, (1 << 20) - 1, 0),
                                         (9_000, 1, 0), (9_000, 3, 1)])
def test_scans_of_a_sort(launches, n, nodes, few):
    got, rc = launches("p = [C.c_void_p(1 << (20 + i)) for i in range(5)]\nrc = lib.gs_sort_pairs(*p[:2], C.c_int64(%d), C.c_int64(%d), *p[2:], C.c_size_t(1 << 50), None)\n"
                       "print(json.dumps({'rc': rc}))\n" % (n, nodes))
    assert rc == [0]
    scans = [x for x in got if "radix_scan" in x[0]]
    assert scans and all(("radix_scan_few_kernel" in x[0], x[4]) == ((True, 256) if few else (False, 1024)) for x in scans), scans


@pytest.mark.parametrize("pairs,nodes,k,dim,bytes", [
    (2_000_000, 4_000_000, 5, 128, 1_448_071_680), (200_000, 60_000, 5, 64, 96_867_840), (1_100_000, 5_000, 1, 32, 224_405_248),
    (1_100_000, 100_000, 5, 64, 483_285_504)])
def test_ways_of_large_steps_in_smaller_workspaces(launches, pairs, nodes, k, dim, bytes):
    """A workspace that holds no grouped records holds sorted ones: the sizes are those that these records took before
    there were others, with counts of 8-bit digits."""
    for ws, how in ((1 << 50, "group"), (bytes, "radix")):
        got, rc = launches(STEP + "print(json.dumps({'rc': step('gs_sgns_step', %d, %d, %d, 0, %d, %d)}))\n" % (pairs, nodes, dim, k, ws))
        assert rc == [0]
        names = " ".join(x[0] for x in got)
        assert ("group_bucket_kernel" in names, "radix_scatter_kernel" in names) == (how == "group", how == "radix"), how


def test_workspaces_grow_with_the_batch(launches):
    """Also where a larger batch takes fewer and larger tiles, or fewer rows per bucket."""
    got, rc = launches("f = lib.gs_sgns_step_workspace_bytes\nf.restype = C.c_size_t\nfor n in (10000, 1000000, 4000000, 1 << 24):\n"
                       "  last = 0\n  for i in range(2000):\n    b = int(2000 * 1.0045 ** i)\n"
                       "    now = f(C.c_int64(b), C.c_int64(n), C.c_int32(5), C.c_int32(64), C.c_int32(0))\n"
                       "    if now < last: print(json.dumps({'rc': [n, b]}))\n    last = now\n")
    assert rc == []


@pytest.mark.parametrize("nodes", [7, 3_000, 20_000, 300_000, 3_000_000])
def test_workspaces_grow_past_the_borders_of_buckets(launches, nodes):
    """Behind a border there are more buckets of fewer rows, and less room for the rows of those that are split."""
    got, rc = launches("f = lib.gs_sgns_step_workspace_bytes\nf.restype = C.c_size_t\nfor k in (0, 1, 5, 10):\n"
                       "  last, b = 0, 20000\n  while b < 1 << 23:\n"
                       "    now = f(C.c_int64(b), C.c_int64(%d), C.c_int32(k), C.c_int32(4), C.c_int32(0))\n"
                       "    if now < last: print(json.dumps({'rc': [k, b]}))\n    last, b = now, b + b // 500 + 1\n" % nodes)
    assert rc == []
