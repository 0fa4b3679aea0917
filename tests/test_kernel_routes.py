"""Which kernels a device call launches, without a GPU: the library runs in a child process with a stand-in for the
HIP runtime's launch that writes down the kernel's name and launch shape instead of launching.  Pointers are made up;
nothing follows them on the host."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <stddef.h>
#include <stdio.h>
typedef struct { unsigned x, y, z; } dim3_t;
static struct { const void *f; const char *name; } seen[8192];
static int n;
void __hipRegisterFunction(void **m, const void *f, char *dev, const char *name, unsigned t, void *a, void *b, void *c, void *d, int *w) {
  if (n < 8192) { seen[n].f = f; seen[n++].name = name; }
}
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
  const char *name = "?";
  for (int k = 0; k < n; ++k) if (seen[k].f == f) name = seen[k].name;
  printf("launch %s %u %u %u %zu\n", name, grid.x, grid.y, block.x, lds);
  fflush(stdout);
  return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
"""

CHILD = r"""
import ctypes as C, json, sys
sys.path.insert(0, {root!r})
from paper_2605_11582_amd import binding as B
L = B._declare(C.CDLL(B.LIB_PATH))                          # (without PyTorch)
P = 1 << 20
def view(rows, cols, n, g, kind, total=0):
    return B.View(rows, cols, n, g, kind, P, P, P, P if kind != 1 else None, total)
for c in json.loads({calls!r}):
    print("call", flush=True)
    k, st = c["call"], 0
    if k == "gemv": st = L.egt_sparse_gemv(C.byref(view(*c["w"])), P, P, None)
    elif k == "int4": st = L.egt_int4_gemv(P, P, *c["w"], P, P, None)
    else:
        count = c["count"]
        if k != "int4_batch": views = (B.View * count)(*[view(*c["w"]) for _ in range(count)])
        xs = (C.c_void_p * count)(*[P + (0 if c.get("shared") else 4096 * j) for j in range(count)])
        ys = (C.c_void_p * count)(*[P + (j << 24) for j in range(count)])
        if k == "gemv_batch": st = L.egt_sparse_gemv_batch(views, xs, ys, count, None)
        elif k == "int4_batch": st = L.egt_int4_gemv_batch(xs, xs, *c["w"], xs, ys, count, None)
        elif k == "gemm": st = L.egt_sparse_gemm_smallm(C.byref(views[0]), P, c["w"][1], P, c["w"][0], c["M"], None)
        else: st = L.egt_sparse_gemm_smallm_batch(views, xs, c["w"][1], ys, c["w"][0], c["M"], count, None)
    assert st == 0, (c, st)
"""


@pytest.fixture(scope="module")
def child(tmp_path_factory):
    """child(script, calls): the lines that the script prints with these calls and the stand-in for the launch."""
    cc = shutil.which("gcc")
    if not cc:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("route")
    lib = str(d / "launch.so")
    (d / "launch.c").write_text(STAND_IN)
    subprocess.run([cc, "-shared", "-fPIC", "-O1", str(d / "launch.c"), "-o", lib], check=True)

    def run(script, calls):
        env = dict(os.environ)
        env["LD_PRELOAD"] = " ".join(v for v in (lib, env.get("LD_PRELOAD", "")) if v)
        out = subprocess.run([sys.executable, "-c", script.replace("{root!r}", repr(ROOT)).replace("{calls!r}", repr(json.dumps(calls)))],
                             capture_output=True, text=True, env=env, timeout=120)
        assert out.returncode == 0, out.stderr[-2000:]
        return out.stdout.splitlines()
    return run


@pytest.fixture(scope="module")
def runs_of_plans(child):
    """runs_of_plans(tables): per table, for its plan as made and for each changed form of it: ([(kernel, grid x, threads, LDS
    bytes)], status, and the plan's grid, threads, LDS bytes and table bytes as made)."""
    def run(tables):
        res, lines = [], iter(child(PLANS, tables))
        for table in tables:
            res.append([])
            for _ in range(1 + len(table[5])):
                assert next(lines) == "call"
                seen = []
                while not (line := next(lines)).startswith("plan "):
                    name, gx, _, threads, lds = line.split()[1:]
                    seen.append((name, int(gx), int(threads), int(lds)))
                res[-1].append((seen, *(int(v) for v in line.split()[1:])))
        return res
    return run


@pytest.fixture(scope="module")
def launches(child):
    """launches(calls): per call the list of (kernel, grid x, grid y, threads) it launches."""
    def run(calls):
        res = []
        for line in child(CHILD, calls):
            if line == "call":
                res.append([])
            elif line.startswith("launch "):
                name, gx, gy, threads, _ = line.split()[1:]
                res[-1].append((name, int(gx), int(gy), int(threads)))
        assert len(res) == len(calls)
        return res
    return run


def _names(res):
    return [[name for name, *_ in call] for call in res]


@pytest.mark.parametrize("cols,n,M,hold", [(4096, 2, 16, True), (4160, 2, 16, False), (2048, 2, 32, True), (2112, 2, 17, False),
                                           (4096, 1, 16, True), (4224, 1, 5, False), (4096, 1, 17, False)])
def test_products_held_in_registers_have_a_wave_for_every_k_step(launches, cols, n, M, hold):
    # (the order of the sums of a row is then that of the other kernel, whichever a call or a batch takes)
    res = _names(launches([{"call": "gemm", "w": (1000, cols, n, 128 if cols % 128 == 0 else 64, 0), "M": M, "count": 1}]))
    assert len(res[0]) == 1 and ("k_smallm_hold" in res[0][0]) == hold, res


@pytest.mark.parametrize("w,M,count,hold", [
    ((11008, 2048, 2), 2, 2, False), ((11008, 1024, 2), 12, 3, False), ((11008, 1792, 2), 2, 2, False),
    ((12500, 2048, 2), 2, 2, True), ((7900, 2048, 2), 2, 2, True), ((11008, 2048, 2), 2, 1, True), ((11008, 1280, 2), 2, 4, True), ((11008, 2304, 2), 2, 2, True),
    ((3259, 512, 1), 2, 2, False), ((5000, 512, 1), 2, 2, True), ((3259, 512, 1), 2, 1, True)])
def test_batches_held_in_registers_where_that_pays(launches, w, M, count, hold):
    (call,) = launches([{"call": "gemm_batch", "w": (*w, 64, 0), "M": M, "count": count, "shared": True}])
    assert len(call) == 1 and ("k_smallm_hold" in call[0][0]) == hold, call


# (rows, cols, n_keep), tokens, members; whether the members' row tiles run as those of one matrix
@pytest.mark.parametrize("w,M,count,joint", [
    ((4096, 11008, 2), 5, 3, True), ((3254, 7936, 1), 22, 4, True), ((5437, 2688, 2), 20, 2, True), ((3843, 3328, 1), 33, 4, True), ((4234, 1792, 2), 50, 3, True), ((4338, 2624, 2), 26, 4, True),
    ((1024, 11008, 2), 5, 3, False),    # a tile a workgroup
    ((6293, 4160, 2), 5, 2, False), ((13824, 5120, 2), 8, 2, False),      # two rounds for two, three for four
    ((13211, 256, 1), 56, 4, False), ((1150, 768, 2), 38, 4, False), ((2831, 1216, 2), 53, 4, False),     # fewer K-steps than waves
    ((1102, 6336, 2), 25, 4, False),    # two token groups, two tiles a workgroup
])
def test_members_under_one_x_run_as_one_matrix_where_that_pays(launches, w, M, count, joint):
    (call,) = launches([{"call": "gemm_batch", "w": (*w, 64, 0), "M": M, "count": count, "shared": True}])
    assert len(call) == 1 and ("ks_joint" in call[0][0]) == joint, call


def test_a_batch_of_several_tokens_is_one_launch(launches):
    # (members under one X or each under its own)
    calls = [{"call": "gemm_batch", "w": (*s, 128, 0), "M": M, "count": 4, "shared": shared}
             for s in ((108, 128, 2), (18, 2048, 2), (1487, 1536, 2), (300, 4096, 1)) for M in (5, 16, 17, 24, 32, 64) for shared in (False, True)]
    for call, res in zip(calls, launches(calls)):
        assert len(res) == 1, (call, res)


def test_fp16_rows_of_one_token(launches):
    # (rows, cols, n_keep, group, value kind)
    short = [(5, 64), (300, 1024), (300, 2048), (4096, 2816), (7, 4064)]
    long = [(256, 4128), (11008, 4128), (256, 16416)]
    res = _names(launches([{"call": "gemv", "w": (*s, 2, 0, 1)} for s in short + long]))
    assert all(len(c) == 1 and "k_rows" in c[0] for c in res[:len(short)]), res
    assert all(len(c) == 1 and "k_sparse_generic_m1" in c[0] for c in res[len(short):]), res


@pytest.mark.parametrize("cols", [64, 1024, 2048, 2816, 4064])
def test_a_batch_of_short_fp16_rows_is_one_launch(launches, cols):
    (call,) = launches([{"call": "gemv_batch", "w": (300, cols, 2, 0, 1), "count": 4}])
    assert len(call) == 1 and "k_rows" in call[0][0] and call[0][2] == 4, call


# (rows, cols, n_keep, group, value kind); which rows run with exact codes on the matrix cores, on both sides of each line
@pytest.mark.parametrize("w,codes", [
    ((11008, 4096, 0, 128, 0), True), ((300, 40960, 0, 128, 0), False),                                   # rows differ; wider than x in LDS
    ((5, 64, 2, 64, 0), True), ((20000, 2816, 2, 128, 0), True), ((20000, 2816, 2, 256, 2), True), ((300, 4096, 2, 128, 0), False), ((300, 1024, 2, 128, 0), False),
    ((300, 1056, 2, 96, 0), False), ((300, 2880, 2, 12, 0), False), ((300, 2880, 3, 64, 0), False),          # groups that are no 32 << j, rows that keep three
    ((300, 4224, 1, 128, 0), True), ((300, 4096, 1, 128, 0), False),
    ((30000, 4096, 0, 64, 0), True), ((5460, 4160, 1, 64, 0), True), ((5461, 4160, 1, 64, 0), False), ((5461, 4160, 1, 32, 0), False),    # waves of a row, waves of a launch
    ((5460, 4160, 0, 64, 0), True), ((5461, 4160, 0, 64, 0), False), ((30000, 4096, 2, 32, 2), True), ((6552, 4128, 2, 32, 2), True), ((6553, 4128, 2, 32, 2), False),
    ((20000, 1696, 1, 32, 0), True), ((20001, 1696, 1, 32, 0), False), ((30000, 1696, 0, 32, 0), True), ((60000, 2112, 1, 64, 0), True),    # long rows, many rows
    ((2048, 4128, 1, 32, 0), True), ((2049, 4128, 1, 32, 0), False), ((2048, 8256, 0, 64, 0), True), ((2049, 8832, 0, 64, 0), False),
    ((2048, 8224, 2, 32, 0), True), ((2049, 8224, 2, 32, 0), False), ((2049, 8224, 2, 32, 2), False), ((5000, 5152, 2, 32, 2), True),
    ((300, 16384, 0, 32, 0), True), ((300, 16416, 0, 32, 0), False),
    ((300, 2816, 0, 0, 1), False),                                                                          # FP16 values
])
def test_rows_of_exact_codes(launches, w, codes):
    (call,) = launches([{"call": "gemv", "w": (*w, w[0] * w[1] // 2 // 8 * 8 if w[2] == 0 else 0)}])
    assert len(call) == 1 and ("k_codes" in call[0][0]) == codes, call


# (rows that differ, and the slots of the matrix)
@pytest.mark.parametrize("rows,cols,slots,codes", [(300, 736, 300 * 184 * 31 // 20, True), (300, 736, 300 * 184 * 31 // 20 + 8, False), (300, 768, 300 * 192 * 4, True), (20000, 2048, 20000 * 512 * 3, True)])
def test_short_rows_that_differ_of_exact_codes(launches, rows, cols, slots, codes):
    (call,) = launches([{"call": "gemv", "w": (rows, cols, 0, 32, 0, slots)}])
    assert len(call) == 1 and ("k_codes" in call[0][0]) == codes, call


@pytest.mark.parametrize("w,codes", [((5003, 2880, 64), True), ((70, 1536, 128), True), ((2278, 1504, 32), False), ((2400, 1504, 32), True), ((300, 384, 128), False), ((300, 2944, 128), False),
                                     ((300, 24512, 64), True), ((300, 24640, 64), False), ((24000, 4064, 32), True), ((6552, 4128, 32), True), ((6553, 4128, 32), False), ((300, 2880, 36), False),
                                     ((1024, 8224, 32), True), ((1025, 8224, 32), False)])
def test_dense_rows_of_exact_codes(launches, w, codes):
    (call,) = launches([{"call": "int4", "w": w}])
    assert len(call) == 1 and ("k_codes" in call[0][0]) == codes, call


@pytest.mark.parametrize("w", [(300, 1664, 128), (300, 1856, 64), (300, 2624, 64), (4000, 992, 32), (300, 1568, 32)])
def test_a_batch_of_dense_exact_codes_is_one_launch(launches, w):
    (call,) = launches([{"call": "int4_batch", "w": w, "count": 4}])
    assert len(call) == 1 and "k_codes_batchILi3E" in call[0][0] and call[0][2] == 4, call


@pytest.mark.parametrize("w", [(300, 1920, 2, 128, 0), (300, 2112, 1, 64, 0), (300, 4128, 2, 32, 2)])
def test_a_batch_of_exact_codes_is_one_launch(launches, w):
    (call,) = launches([{"call": "gemv_batch", "w": w, "count": 4}])
    assert len(call) == 1 and "k_codes_batch" in call[0][0] and call[0][2] == 4, call


# (rows, cols, n_keep, group, value kind), tiles of a wave: the second number (dense: the first) of the kernel's template arguments after the
# value kind; on both sides of each line
@pytest.mark.parametrize("w,kernel,tiles", [
    ((1536, 4096, 2, 128, 0), "k_sparse_m1_oneILi%dE", 1), ((1537, 4096, 2, 128, 0), "k_sparse_m1_oneILi%dE", 2), ((2305, 4096, 2, 128, 0), "k_sparse_m1_oneILi%dE", 4),
    ((1536, 4096, 2, 128, 2), "k_sparse_m1_oneILi%dE", 1), ((2304, 4096, 2, 128, 2), "k_sparse_m1_oneILi%dE", 2), ((2305, 4096, 2, 128, 2), "k_sparse_m1_oneILi%dE", 4),
    ((9216, 1024, 2, 128, 0), "k_sparse_m1ILi0ELi%dE", 1), ((9217, 1024, 2, 128, 0), "k_sparse_m1ILi0ELi%dE", 2), ((20482, 2048, 2, 128, 0), "k_sparse_m1ILi0ELi%dE", 4),
    ((1024, 16384, 2, 128, 0), "k_sparse_m1ILi0ELi%dE", 1), ((1025, 16384, 2, 128, 0), "k_sparse_m1ILi0ELi%dE", 4), ((1024, 11008, 2, 128, 2), "k_sparse_m1ILi0ELi%dE", 1),
    ((1025, 11008, 2, 128, 2), "k_sparse_m1ILi0ELi%dE", 2), ((3, 32768, 2, 128, 0), "k_sparse_m1ILi0ELi%dE", 1),
    ((1024, 4096, 2, 0, 1), "k_sparse_m1ILi1ELi%dE", 1), ((6144, 4096, 2, 0, 1), "k_sparse_m1ILi1ELi%dE", 2), ((6145, 4096, 2, 0, 1), "k_sparse_m1ILi1ELi%dE", 4),
    ((1024, 8192, 1, 128, 0), "k_sparse_m1_n1ILi0ELi%dE", 1), ((1025, 8192, 1, 128, 0), "k_sparse_m1_n1ILi0ELi%dE", 2),
    ((2048, 1920, 2, 128, 0), "k_codesILi0ELi64ELi32ELi%dE", 1), ((4098, 1920, 2, 128, 0), "k_codesILi0ELi64ELi32ELi%dE", 2), ((5121, 3072, 2, 128, 0), "k_codesILi0ELi64ELi32ELi%dE", 4)])
def test_tiles_of_a_wave(launches, w, kernel, tiles):
    (call,) = launches([{"call": "gemv", "w": (*w, 0)}])
    assert len(call) == 1 and kernel % tiles in call[0][0], call


@pytest.mark.parametrize("w,kernel,tiles", [((2048, 2048, 128), "k_int4_m1ILi%dE", 1), ((2049, 2048, 128), "k_int4_m1ILi%dE", 4), ((1024, 8192, 128), "k_int4_m1ILi%dE", 1), ((1025, 8192, 128), "k_int4_m1ILi%dE", 4),
                                            ((1024, 11008, 128), "k_int4_m1ILi%dE", 2), ((512, 20224, 256), "k_int4_m1ILi%dE", 2), ((513, 20224, 256), "k_int4_m1ILi%dE", 4), ((1024, 16384, 128), "k_int4_m1ILi%dE", 2), ((5120, 2880, 64), "k_codesILi3ELi32ELi32ELi%dE", 2), ((5121, 2880, 64), "k_codesILi3ELi32ELi32ELi%dE", 4)])
def test_tiles_of_a_wave_of_dense_rows(launches, w, kernel, tiles):
    (call,) = launches([{"call": "int4", "w": w}])
    assert len(call) == 1 and kernel % tiles in call[0][0], call


def test_matrices_of_many_tiles_reach_other_kernels_than_their_first_rows(launches):
    # (the GPU test of the same cases compares the two)
    from test_gpu_parity import MANY_TILES

    def call(rows, cols, g, form):
        if form == "dense":
            return {"call": "int4", "w": (rows, cols, g)}
        if isinstance(form, str) and form.isdigit():
            return {"call": "gemv", "w": (rows, cols, 0, g, 0, sum(int(form[r % len(form)]) for r in range(rows)) * (cols // 4))}
        n, kind = {"paired": (2, 2), "fp16": (2, 1)}.get(form, (form, 0))
        return {"call": "gemv", "w": (rows, cols, n, g, kind, 0)}
    many = _names(launches([call(*c) for c in MANY_TILES]))
    few = _names(launches([call(61, *c[1:]) for c in MANY_TILES]))
    for c, a, b in zip(MANY_TILES, many, few):
        assert len(a) == len(b) == 1 and a != b and a[0].split("IL")[0][-8:] == b[0].split("IL")[0][-8:], (c, a, b)


def test_rows_of_more_than_2048_columns_take_two_kernels_up_to_32_tokens_and_beyond(launches):
    # (those whose bits the GPU tests compare)
    from test_gpu_smallm_wide import MORE_THAN_2048
    for rows, cols, g, M in MORE_THAN_2048:
        few, many = _names(launches([{"call": "gemm", "w": (rows, cols, 2, g, 0), "M": m, "count": 1} for m in (32, M)]))
        assert len(few) == len(many) == 1 and "k_sparse_smallm_ks" in few[0] and "k_smallm_wide" in many[0], (rows, cols, few, many)


def test_members_as_one_matrix_have_three_tiles_a_workgroup_and_more_beyond_32_tokens(launches):
    # (the only forms of k_smallm_wide_ks_joint: the smallest sizes that run as one matrix, and sizes around the next rounds)
    calls = [{"call": "gemm_batch", "w": (16 * t - 3, 2048, 2, 128, 0), "M": M, "count": c, "shared": True}
             for M in (33, 64) for c in (2, 3, 4) for t in (*range(120, 400, 9), 512, 513, 640, 768, 769, 1024, 1025, 1300)]
    joint = 0
    for call, c in zip(launches(calls), calls):
        assert len(call) == 1 and "k_smallm_wide" in call[0][0], (c, call)
        if "ks_joint" in call[0][0]:
            tiles = -(-((c["w"][0] + 15) // 16 * c["count"]) // call[0][1])
            rounds = -(-tiles // 4)
            assert tiles >= 3 and f"ks_jointILi{3 if c['M'] <= 48 else 4}ELi{-(-tiles // rounds)}E" in call[0][0], (c, call)
            joint += 1
    assert joint > 40


# kind: 0 INT4, 1 FP16
@pytest.mark.parametrize("w,M,count,shared,wide", [
    ((1000, 4096, 2, 128, 0), 33, 1, True, "k_smallm_wide"), ((1000, 4096, 2, 128, 0), 64, 1, True, "k_smallm_wide"),
    ((4234, 1792, 2, 64, 0), 50, 3, True, "ks_joint"), ((4234, 1792, 2, 64, 0), 50, 3, False, "k_smallm_wide_batch"),
    ((1000, 4096, 2, 128, 0), 32, 1, True, None), ((1000, 4096, 2, 32, 0), 64, 1, True, None), ((1000, 4096, 2, 0, 1), 64, 1, True, None),
    ((1000, 4096, 1, 128, 0), 64, 1, True, None)])
def test_more_than_two_token_groups_take_one_pass(launches, w, M, count, shared, wide):
    (call,) = launches([{"call": "gemm_batch" if count > 1 else "gemm", "w": w, "M": M, "count": count, "shared": shared}])
    assert len(call) == 1 and ("k_smallm_wide" in call[0][0]) == (wide is not None) and (wide or "") in call[0][0], call


PLANS = r"""
import ctypes as C, json, sys
sys.path.insert(0, {root!r})
from paper_2605_11582_amd import binding as B
L = B._declare(C.CDLL(B.LIB_PATH))                          # (without PyTorch)
P = 1 << 20
for M, n, rows, cols, count, changes in json.loads({calls!r}):
    each = cols if isinstance(cols, list) else [cols]       # row lengths in turn
    views = [B.View(rows, each[k % len(each)], n, 128, 0, P, P, P, P) for k in range(count)]
    items = (B.GemmItem * count)()
    for k, v in enumerate(views):
        items[k].sparse, items[k].X, items[k].Y = C.pointer(v), P, P
    plan = B.GemmPlan()
    assert L.egt_gemm_stack_plan(items, count, M, None, 0, C.byref(plan)) == 0
    for change in [{}] + changes:
        p = B.GemmPlan.from_buffer_copy(plan)
        for field, value in change.items(): setattr(p, field, value)
        print("call", flush=True)
        print("plan", L.egt_gemm_stack_run(P, C.byref(p), None), plan.grid_x, plan.block_threads, plan.lds_bytes, plan.table_bytes, flush=True)
"""

ROWS_LDS = {(16, 2): 67584, (32, 2): 67584, (64, 2): 135168, (16, 1): 66560, (32, 1): 133120}            # k_smallm_rows, by most tokens and form
TILES_LDS = {(16, 2): (66560,), (32, 2): (79872, 116736), (64, 2): (159744,), (16, 1): (78848, 115712), (32, 1): (157696,)}   # k_stack_tiles: a row tile a wave, two


@pytest.mark.parametrize("top,n", list(TILES_LDS))
def test_a_plan_runs_only_in_the_form_its_table_was_laid_out_for(runs_of_plans, top, n):
    # tables of few workgroups, of more, and of 400 MB and more; every plan runs in its own form, and with the threads or LDS bytes
    # of another form it is refused where it always was: half of a matrix would stay unwritten where a workgroup of the
    # table owns sixteen row tiles and the kernel takes eight
    lds = (ROWS_LDS[top, n],) + TILES_LDS[top, n]
    sixteen = top == (64 if n == 2 else 32)
    changes = [{"lds_bytes": v, "block_threads": t} for v in lds for t in (256, 512, 1024)]
    tables = [(top, n, 1024, 4096, 1), (top, n, 1024, 4096, 40), (top, n, 8192, 8192, 30)]
    # (kernel, LDS bytes of the launch) of each table
    forms = ["k_smallm_rows", "k_stack_tiles", "k_stack_tiles"]
    own = [lds[0], lds[1], lds[-1]]
    for table, form, at, res in zip(tables, forms, own, runs_of_plans([(*t, changes) for t in tables])):
        (launched, status, grid, threads, lds_bytes, table_bytes), rest = res[0], res[1:]
        assert status == 0 and len(launched) == 1 and form in launched[0][0] and lds_bytes == at, (table, res[0])
        assert launched[0][1:] == (grid, threads, lds_bytes), (table, res[0])
        assert threads == (1024 if form == "k_smallm_rows" and sixteen else 512)
        two = len(TILES_LDS[top, n]) == 2 and at == lds[-1]
        for change, (again, st, *_) in zip(changes, rest):
            pair = (change["block_threads"], change["lds_bytes"])
            ok = pair == (threads, lds_bytes)
            if not two:
                # k_smallm_rows takes every table of its tiles a workgroup; with sixteen of them the number of its waves is free in
                # a large table (plans that a caller kept)
                ok = ok or pair == ((1024 if sixteen else 512), lds[0]) or (sixteen and grid >= 128 and pair in [(512, lds[0]), (1024, lds[1])])
            assert (st == 0) == ok and len(again) == (1 if ok else 0) and st in (0, 2), (table, change, st)
            if ok:                                           # sixteen tiles: the waves name the kernel; it gets its own LDS
                kernel = ("k_smallm_rows" if pair[0] == 1024 else "k_stack_tiles") if sixteen else ("k_smallm_rows" if pair[1] == lds[0] else "k_stack_tiles")
                assert kernel in again[0][0] and again[0][2] == pair[0], (table, change, again)
                assert again[0][3] == ({"k_smallm_rows": lds[0], "k_stack_tiles": lds[1]}[kernel] if sixteen else pair[1]), (table, change, again)


@pytest.mark.parametrize("M,n", [(17, 2), (32, 2), (4, 1), (16, 1)])
def test_two_tiles_a_wave_take_long_rows(runs_of_plans, M, n):
    # tables of 400 MB and more: with rows of fewer than 4096 columns a workgroup is over before two tiles a wave pay for the second
    # workgroup of a compute unit, whatever the other rows
    one, two = TILES_LDS[32 if n == 2 else 16, n]
    tables = [(M, n, 2048, cols, 400, []) for cols in (2560, 3968, 4096, 11008, [11008, 4096], [11008, 3968], [3968, 11008])]
    for (*_, cols, count, _), (res,) in zip(tables, runs_of_plans(tables)):
        launched, status, grid, threads, lds, _ = res
        tiles = 16 if min(cols if isinstance(cols, list) else [cols]) >= 4096 else 8
        assert status == 0 and len(launched) == 1 and lds == (two if tiles == 16 else one) and threads == 512, (cols, res)
        assert "k_stack_tiles" in launched[0][0] and grid == count * 2048 // (16 * tiles), (cols, res)


@pytest.mark.parametrize("M,n", [(4, 2), (16, 2), (17, 2), (32, 2), (4, 1), (16, 1)])
def test_large_tables_of_short_rows_keep_their_kernel(runs_of_plans, M, n):
    # rows of three and four K-steps in tables of 250 MB and more: k_smallm_rows, as before there was k_stack_tiles
    top, step = (32 if M > 16 else 16), 512 // n
    nbytes = lambda cols: 2048 * (n * (cols // 16) * 3 + 4 * (cols // 128))
    few, many = (lambda cols: 249_999_999 // nbytes(cols)), (lambda cols: -(-250_000_000 // nbytes(cols)))
    tables = [(M, n, 2048, c, many(c), []) for c in (2 * step, 3 * step, 3 * step - 128, 4 * step, 4 * step - 128, 4 * step + 128)]
    tables += [(M, n, 2048, c, few(c), []) for c in (3 * step, 4 * step)]
    tables += [(M, n, 2048, [step, 4 * step], 2 * many(step), []), (M, n, 2048, [4 * step, 4 * step + 128], 2 * many(4 * step), [])]
    want = [False, True, True, True, True, False, False, False, True, False]
    for (*_, cols, count, _), rows, (res,) in zip(tables, want, runs_of_plans(tables)):
        launched, status, grid, threads, lds, _ = res
        assert status == 0 and len(launched) == 1 and ("k_smallm_rows" in launched[0][0]) == rows, (cols, res)
        assert (lds == ROWS_LDS[top, n]) == rows and threads == 512 and grid == count * 16, (cols, res)


def test_a_plan_without_the_mark_of_two_tiles_a_wave_is_refused(runs_of_plans):
    # (30 descriptors of 160 bytes, 32 workgroups a matrix; the mark alone in a table without it is refused too)
    plain = 30 * 160 + 4 * 30 * 32
    two, one = runs_of_plans([(24, 2, 8192, 8192, 30, [{"table_bytes": plain}, {"table_bytes": plain + 32}, {"lds_bytes": 79872}, {"lds_bytes": 67584}]),
                              (24, 2, 4096, 1024, 30, [{"table_bytes": plain + 16}, {"table_bytes": plain + 16, "lds_bytes": 67584}])])
    assert [r[1] for r in two] == [0, 2, 2, 2, 2] and two[0][2:] == (30 * 32, 512, 116736, plain + 16), two
    assert [r[1] for r in one] == [0, 2, 2] and one[0][2:] == (30 * 32, 512, 79872, plain), one
