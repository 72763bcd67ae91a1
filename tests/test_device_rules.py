"""The plain arithmetic that the device code and the host share
(csrc/mce_internal.h), compiled for the host and run at the ends of its ranges."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = str(d / "rules.cpp"), str(d / "rules.so")
    with open(src, "w") as f:
        f.write('#include "mce_internal.h"\nusing namespace mce;\n' + SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_1801_00202_amd", "csrc"), "-o", lib, src])
    return ctypes.CDLL(lib)


SOURCE = r"""
// The totals after a lane search that holds `start` of each and takes `looks`
// times as many steps as can come between two looks, of 64 busy lanes, each
// child a node and a clique (more than there can be).
struct Totals {
    uint64_t count, nodes, children;
};
extern "C" void lane_totals(uint32_t start, uint32_t looks, Totals* out)
{
    LaneTotals t;
    t.children = t.nodes = t.cliques = start;
    for (uint32_t k = 0; k < looks; k++) {
        for (uint32_t i = 0; i < kLaneLookMax; i++) {
            t.step(64, 64);
            t.cliques += 64;
        }
        if (t.due()) t.add_to(*out);
    }
    t.add_to(*out);
}

// spare slots granted to `graphs` graphs one after the other, each of `units`
// units that want `chop` pieces
extern "C" uint64_t slots_granted(uint32_t graphs, uint32_t units, uint32_t chop, uint32_t limit)
{
    uint64_t asked = 0, granted = 0;
    for (uint32_t g = 0; g < graphs; g++) {
        granted += (uint64_t)units * (pieces_granted(asked, units, chop, limit) - 1u);
        asked += (uint64_t)units * (chop - 1u);
    }
    return granted;
}

// levels, chunks and lanes' levels; the bytes of both stacks
extern "C" uint64_t stacks(int lanes, uint32_t waves, uint32_t full_levels, uint32_t chunks, int deep, int lanes_deep,
                           uint32_t* out)
{
    StackNeeds need;
    need.chunks = chunks;
    need.deep = deep != 0;
    need.lanes_deep = lanes_deep != 0;
    const StackPlan p = plan_stacks(lanes != 0, waves, full_levels, 1024, need);
    out[0] = p.levels;
    out[1] = p.chunks;
    out[2] = p.lane_levels;
    return 1024ull * p.levels * p.chunks + 4ull * kLaneLevelWords * p.lane_levels * waves;
}

extern "C" int lanes(uint32_t n, uint64_t sum)
{
    DegreeSample d;
    if (DegreeSample::wanted(n, 1)) d.add(n);
    d.sum = sum;
    return d.lanes(1);
}
// a batch of `small` graphs of 100 vertices and `large` of n, of degree deg
extern "C" int batch_lanes(uint32_t small, uint32_t large, uint32_t n, uint32_t deg)
{
    DegreeSample d;
    for (uint32_t i = 0; i < small + large; i++) {
        const uint32_t k = i < small ? 100u : n;
        if (!DegreeSample::wanted(k, small + large)) continue;
        d.add(k);
        d.sum += (uint64_t)deg * degree_rows(k);
    }
    return d.lanes(small + large);
}
extern "C" uint32_t sampled_rows(uint32_t n)
{
    uint32_t k = 0;
    for (uint32_t i = 0; i < n; i += degree_stride(n)) k++;
    return k;
}

extern "C" int on_lists(uint32_t num_graphs, uint32_t large, uint32_t max_n)
{
    return order_on_lists(num_graphs, large, max_n);
}

// the same plan cut to an area: its wavefronts, levels, chunks and bytes
extern "C" uint64_t stacks_in(int lanes, uint64_t area, uint32_t waves, uint32_t full_levels, uint32_t frame,
                              uint32_t chunks, int deep, int lanes_deep, uint32_t* out)
{
    StackNeeds need;
    need.chunks = chunks;
    need.deep = deep != 0;
    need.lanes_deep = lanes_deep != 0;
    StackPlan p = plan_stacks(lanes != 0, waves, full_levels, frame, need);
    const uint32_t w = fit_stacks(lanes != 0, area, waves, frame, need, &p);
    out[0] = w;
    out[1] = p.levels;
    out[2] = p.chunks;
    return (uint64_t)frame * p.levels * p.chunks + 4ull * kLaneLevelWords * p.lane_levels * w;
}
"""


# up to the fold, at it, past 2^32 and twice past it
@pytest.mark.parametrize("start,looks", [(0, 3), ((1 << 31) - 1, 1), (1 << 31, 1), ((1 << 31) + (1 << 26), 1), (0, 70),
                                         (7, 150)])
def test_lane_totals_pass_32_bits(rules, start, looks):
    out = (ctypes.c_uint64 * 3)(1, 1, 1)
    rules.lane_totals(start, looks, out)
    assert list(out) == [1 + start + looks * (64 << 20)] * 3


# what the graphs ask for together passes 2^32: many graphs of one unit, fewer
# of many units (a large pool); exactly what there is; one more
@pytest.mark.parametrize("graphs,units,chop,limit,want", [
    (70000, 1, 65535, 131072, 2 * 65534),
    (200000, 1, 65535, 262144, 4 * 65534),
    (5000, 20, 65535, 1 << 25, 25 * 20 * 65534),
    (3, 5, 3, 30, 30),
    (4, 5, 3, 30, 30),
    (3, 5, 3, 29, 20),
    (10, 7, 1, 0, 0),
    (1 << 20, 1, 65535, 0, 0),
])
def test_batch_pieces_stay_within_the_pool(rules, graphs, units, chop, limit, want):
    rules.slots_granted.restype = ctypes.c_uint64
    assert rules.slots_granted(graphs, units, chop, limit) == want <= limit


# (lanes, waves, levels below the window, chunks asked, deep, lanes deep)
@pytest.mark.parametrize("args,want", [
    ((1, 2560, 2015, 0, 0, 0), (32, 2560, 16)),
    # a lane that ran out of its levels: the wavefronts' loops keep theirs
    ((1, 2560, 2015, 0, 0, 1), (32, 2560, 124)),
    # a loop that ran out: full depth, in 256 MiB or 64 chunks; lanes as before
    ((1, 2560, 2015, 0, 1, 0), (2015, 130, 16)),
    ((1, 3072, 999, 0, 1, 1), (999, 262, 124)),
    ((1, 2560, 16383, 0, 1, 0), (16383, 64, 16)),
    ((1, 100, 500, 0, 1, 0), (500, 100, 16)),
    # and one for every wavefront only when those run out too
    ((1, 2560, 2015, 2560, 1, 0), (2015, 2560, 16)),
    # without lanes
    ((0, 4096, 2040, 0, 0, 0), (64, 64, 0)),
    ((0, 4096, 2040, 0, 1, 1), (2040, 64, 0)),
    ((0, 4096, 2040, 4096, 1, 0), (2040, 4096, 0)),
    ((0, 16, 3, 0, 0, 0), (3, 16, 0)),
    ((1, 16, 0, 0, 1, 0), (1, 16, 16)),
])
def test_stack_plan(rules, args, want):
    rules.stacks.restype = ctypes.c_uint64
    out = (ctypes.c_uint32 * 3)()
    size = rules.stacks(*args, out)
    assert tuple(out) == want
    if not args[3]:  # (otherwise a chunk a wavefront was asked for)
        assert size <= (256 << 20) + (1 << 30)


AREA = 114 << 20


# (lanes, waves, levels below the window, frame, chunks asked, deep, lanes deep)
@pytest.mark.parametrize("args,want", [
    # the first try: all wavefronts, each with a chunk of what is left beside
    # the lanes' stacks
    ((1, 3072, 999, 1024, 0, 0, 0), (3072, 6, 3072)),
    ((1, 2560, 2015, 1024, 0, 0, 0), (2560, 13, 2560)),
    ((1, 2048, 250, 1024, 0, 0, 0), (2048, 25, 2048)),
    ((1, 256, 250, 1024, 0, 0, 0), (256, 32, 256)),
    # deep loops, deep lanes, both: fewer wavefronts
    ((1, 2560, 2015, 1024, 0, 1, 0), (57, 2015, 57)),
    ((1, 2560, 2015, 1024, 0, 0, 1), (463, 4, 463)),
    ((1, 2560, 2015, 1024, 0, 1, 1), (51, 2015, 51)),
    # without lanes the spill pool has the whole area
    ((0, 2048, 2044, 2048, 0, 0, 0), (2048, 64, 64)),
    ((0, 2048, 2044, 2048, 2048, 0, 0), (912, 64, 912)),
    ((0, 2048, 2044, 2048, 0, 1, 0), (2048, 2044, 28)),
    ((0, 2048, 2044, 2048, 2048, 1, 0), (28, 2044, 28)),
])
def test_stacks_in_a_fixed_area(rules, args, want):
    rules.stacks_in.restype = ctypes.c_uint64
    out = (ctypes.c_uint32 * 3)()
    size = rules.stacks_in(args[0], ctypes.c_uint64(AREA), *args[1:], out)
    assert tuple(out) == want and size <= AREA


def test_stacks_in_any_area(rules):
    rules.stacks_in.restype = ctypes.c_uint64
    out = (ctypes.c_uint32 * 3)()
    for area in (1, 1000, 1 << 15, 40000, 300000, 5 << 20, AREA, 1 << 33):
        for lanes in (0, 1):
            for waves in (1, 3, 12, 400, 3072, 8192):
                for levels in (1, 3, 5, 40, 2015):
                    for chunks in (0, waves):
                        for deep in (0, 1):
                            for lanes_deep in (0, 1):
                                size = rules.stacks_in(lanes, ctypes.c_uint64(area), waves, levels, 1024, chunks, deep,
                                                       lanes_deep, out)
                                w, lv, ch = out
                                # all in the area, or not one wavefront
                                assert w <= waves and (w == 0 or (size <= area and lv >= 1 and ch >= 1))
                                if w and (lanes or chunks):
                                    assert ch == w


@pytest.mark.parametrize("num_graphs,large,max_n,want", [
    (1, 0, 900, 1), (1, 1, 3000, 1), (2, 0, 1000, 0), (8, 1, 1500, 1), (9, 1, 1500, 0), (20001, 1, 1500, 0),
    (20001, 1, 4096, 0), (20001, 1, 4097, 1), (1 << 30, 1 << 27, 2000, 1), (1 << 30, (1 << 27) - 1, 2000, 0),
])
def test_batches_on_lists(rules, num_graphs, large, max_n, want):
    assert rules.on_lists(num_graphs, large, max_n) == want


@pytest.mark.parametrize("n", [0, 1, 2, 15, 16, 17, 31, 32, 33, 500, 1600, 2016, 16384])
def test_sampled_degrees(rules, n):
    rows = rules.sampled_rows(n)
    assert rows == min(n, rows) and (n <= 16) == (rows == n) and rows <= 16 and (n < 16 or rows >= 8)
    # every row of degree d: the mean is d, and the rule on both sides of its lines
    for d in {0, n // 12, n // 10, n // 8, n // 2, max(n - 1, 0)}:
        want = n > 2016 or d < 96 or d > 0.11 * n
        assert rules.lanes(n, ctypes.c_uint64(d * rows)) == want


@pytest.mark.parametrize("small,large,n,deg,want", [
    (0, 2, 1600, 130, 0), (0, 2, 1600, 95, 1), (0, 2, 1600, 177, 1), (2, 2, 1600, 130, 0), (3, 2, 1600, 130, 1),
    (0, 5, 860, 94, 1), (0, 5, 900, 97, 0), (0, 5, 2016, 150, 0), (0, 5, 2017, 150, 1), (5, 0, 0, 0, 1),
])
def test_batch_lanes(rules, small, large, n, deg, want):
    assert rules.batch_lanes(small, large, n, deg) == want
