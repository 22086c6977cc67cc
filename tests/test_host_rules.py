"""CPU: the host rules of csrc/analysis.cpp that no entry point hands out - the chunk descriptors of the merge path, the
chunks of a cut row, the pairs form's layout and the choice between the two forms of the sparse-times-dense product - each
against its definition written out (or the oracle's).  The file is compiled on its own, with a few plain functions around it."""
import ctypes as C
import math
import subprocess

import numpy as np
import pytest

import oracle
from paper_2603_07169_amd import build as lib_build

WRAPPER = r"""
#include "analysis.h"
#include <cstring>
using std::vector;
template <typename T> static void out(const vector<T>& v, T* p) { if (!v.empty()) std::memcpy(p, v.data(), sizeof(T) * v.size()); }
extern "C" {
void chunk_desc(int64_t m, const int32_t* rp, int64_t P, const int32_t* row, const int32_t* nz, int64_t snap, int32_t* desc) {
    vector<int32_t> d;
    spmv::merge_chunk_desc(m, rp, vector<int32_t>(row, row + P + 1), vector<int32_t>(nz, nz + P + 1), snap, &d);
    out(d, desc);
}
void cuts(int64_t m, const int32_t* rp, int64_t P, const int32_t* row, const int32_t* nz, int32_t* ranges) {
    vector<int32_t> r;
    spmv::cut_ranges(m, rp, vector<int32_t>(row, row + P + 1), vector<int32_t>(nz, nz + P + 1), &r);
    out(r, ranges);
}
int pair_layout(int64_t m, const int32_t* rp, const int32_t* packed, int32_t* rows, int32_t* desc, int64_t* blocks) {
    vector<int32_t> r, d;
    const bool kept = spmv::spmm_pair_layout(m, rp, vector<int32_t>(packed, packed + 2 * ((m + 15) / 16) + 2), &r, &d, blocks);
    out(r, rows);
    out(d, desc);
    return kept;
}
double busiest(const int32_t* desc, int64_t groups, int rows_per_group, int64_t S) {
    return spmv::spmm_busiest(spmv::spmm_group_steps(vector<int32_t>(desc, desc + 2 * groups + 2), rows_per_group), S);
}
int packed_splits(int64_t slices, int64_t groups) { return spmv::spmm_packed_splits(slices, groups); }
int pair_splits(int64_t slices, int64_t groups, int64_t blocks) { return spmv::spmm_pair_splits(slices, groups, blocks); }
int choice(const int32_t* pk, int64_t gk, const int32_t* pp, int64_t gp, int64_t blocks, int64_t m, int64_t K, int vec) {
    return spmv::spmm_pairs_choice(spmv::spmm_group_steps(vector<int32_t>(pk, pk + 2 * gk + 2), 16),
                                   spmv::spmm_group_steps(vector<int32_t>(pp, pp + 2 * gp + 2), 32), blocks, m, K, vec != 0);
}
int window_kernel(int elem, int staged, int rows, int xv, int sheet, int runs, int vec, int kept) {
    return static_cast<int>(spmv::window_kernel(elem, staged, rows, xv, sheet, runs != 0, vec != 0, kept != 0));
}
int sheets_pay(int elem, int64_t m, int64_t nnz, int64_t nb, int block_nnz, int rows_max, int common, int cus) {
    return spmv::sheets_pay(elem, m, nnz, nb, block_nnz, rows_max, common, cus);
}
int stream_lanes(int elem, int64_t m, int64_t nnz, int rows_max, int places, int common) {
    return spmv::stream_lanes(elem, m, nnz, rows_max, places, common);
}
int gather_choice(int64_t m, int64_t n, int64_t nnz, int plan, int bf16, int64_t max_len, int cus, int k) {
    return spmv::gather_choice(m, n, nnz, plan, bf16 != 0, max_len, cus, k);
}
int gather_pays(int64_t m, int64_t nnz, int plan, int bf16, int cus, int64_t chunks, int64_t most, int64_t lines, int64_t stretch_lines) {
    return spmv::gather_pays(m, nnz, plan, bf16 != 0, cus, chunks, most, lines, stretch_lines);
}
int gather_groups_choice(int64_t m, int64_t groups, int cus) { return spmv::gather_groups_choice(m, groups, cus); }
int rows_of_groups(int64_t m, const int32_t* rp) { return spmv::rows_of_groups(m, rp); }
int64_t gather_snap(int plan, int64_t max_len, int64_t items) { return spmv::gather_snap(plan, max_len, items); }
int common_len(int64_t m, const int32_t* rp) { return spmv::common_row_length(m, rp); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_rules")
    (d / "wrapper.cpp").write_text(WRAPPER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-pthread", f"-I{lib_build.INCLUDE}", f"-I{lib_build.CSRC}",
                    str(d / "wrapper.cpp"), str(lib_build.CSRC / "analysis.cpp"), "-o", str(d / "rules.so")], check=True)
    lib = C.CDLL(str(d / "rules.so"))
    lib.busiest.restype = C.c_double
    return lib


def P(a):
    return a.ctypes.data_as(C.c_void_p)


i64 = C.c_int64


def rowptr_of(lens):
    return np.concatenate(([0], np.cumsum(np.asarray(lens, dtype=np.int64)))).astype(np.int32)


def row_lengths(seed):
    """Rows around the snap length, empty rows, rows over many chunks and rows that end on a cut, shuffled differently."""
    rng = np.random.default_rng(seed)
    kinds = [rng.integers(0, 4, 300), np.array([255, 256, 257, 512, 513, 2047, 2048, 0, 0, 5000]), rng.integers(200, 700, 30),
             np.array([], int), rng.integers(0, 2, 50)]
    lens = np.concatenate([kinds[i] for i in rng.permutation(len(kinds))[:rng.integers(1, 6)]]).astype(int)
    return lens if lens.size else np.array([3])


@pytest.mark.parametrize("items,snap", [(1, 0), (7, 6), (100, 99), (256, 255), (257, 256), (2048, 256), (8192, 256), (100, 30)])
@pytest.mark.parametrize("seed", range(8))
def test_chunk_descriptors_move_cuts_inside_short_rows(rules, seed, items, snap):
    lens = row_lengths(seed)
    rp = rowptr_of(lens)
    row, nz = oracle.merge_path(rp, items)
    n = row.size
    desc = np.zeros(2 * n, np.int32)
    rules.chunk_desc(i64(lens.size), P(rp), i64(n - 1), P(row), P(nz), i64(snap), P(desc))
    want = []
    for i, k in zip(row.tolist(), nz.tolist()):
        if i < lens.size and k > rp[i] and lens[i] <= snap:
            k = int(rp[i])
        want += [i, k]
    assert desc.tolist() == want
    grown = np.diff(desc[0::2].astype(np.int64) + desc[1::2])
    assert np.all(np.diff(desc[1::2]) >= 0) and (grown.size == 0 or grown.max() <= items + snap)  # what the chunks' LDS is sized for
    assert grown.size == 0 or grown.min() > 0                                                      # and none is empty


@pytest.mark.parametrize("seed", range(8))
@pytest.mark.parametrize("items", [5, 64, 2048])
def test_chunks_of_a_cut_row(rules, seed, items):
    """Per split that falls inside a row: the first and the last chunk holding a part of it.  On the unmoved splits the same
    two numbers follow from the steps that take the row's first entry and finish it, as the merge-path kernel computes them."""
    lens = row_lengths(seed)
    rp = rowptr_of(lens)
    for snapped in (False, True):
        row, nz = oracle.merge_path_snapped(rp, items, min(30, items - 2)) if snapped else oracle.merge_path(rp, items)
        n = row.size
        got = np.zeros(2 * n, np.int32)
        rules.cuts(i64(lens.size), P(rp), i64(n - 1), P(row), P(nz), P(got))
        parts = {}
        for p in range(n - 1):                      # chunk p: its rows' pieces and the piece it cuts off at its end
            for i in range(row[p], min(row[p + 1], lens.size - 1) + 1):
                first, last = max(rp[i], nz[p]), min(rp[i + 1], nz[p + 1])
                if last > first or (row[p] <= i < row[p + 1]):
                    parts.setdefault(i, []).append(p)
        for q in range(n):
            i = int(row[q])
            inside = i < lens.size and nz[q] > rp[i]
            assert got[2 * q:2 * q + 2].tolist() == ([parts[i][0], parts[i][-1]] if inside else [-1, -1]), (q, i)
            if inside and not snapped:
                assert got[2 * q:2 * q + 2].tolist() == [(i + rp[i]) // items, (i + rp[i + 1]) // items]


@pytest.mark.parametrize("seed", range(10))
def test_pairs_layout_equals_the_oracles(rules, seed):
    rng = np.random.default_rng(seed)
    m = int(rng.choice([1, 31, 32, 33, 500, 4096, 9000]))
    lens = rng.choice([rng.poisson(20, m), rng.integers(0, 3000, m), np.where(rng.random(m) < 0.1, 300, 4)])
    rp = rowptr_of(lens)
    packed, _ = oracle.spmm_packed_layout(rp, oracle.spmm_row_order(rp))
    rows, desc, blocks = np.zeros(m, np.int32), np.zeros(2 * ((m + 31) // 32) + 2, np.int32), i64()
    kept = rules.pair_layout(i64(m), P(rp), P(packed), P(rows), P(desc), C.byref(blocks))
    want_rows = oracle.spmm_pair_row_order(rp)
    want_desc, want_blocks = oracle.spmm_pair_layout(rp, want_rows)
    assert np.array_equal(rows, want_rows) and np.array_equal(desc, want_desc) and blocks.value == want_blocks
    assert bool(kept) == oracle.spmm_pair_choice(m, 2048, want_blocks, packed)


def desc_of(steps):
    return np.stack([np.zeros(len(steps) + 1), np.append(steps, 1)], 1).astype(np.int32).reshape(-1).copy()


@pytest.mark.parametrize("rows_per_group", [16, 32])
def test_busiest_wavefront(rules, rows_per_group):
    """Against the average over the places a wavefront meets, taken at the worst of its starts; exact where every wavefront
    meets whole windows of the same lengths."""
    per_window = 4096 // rows_per_group
    rng = np.random.default_rng(3)
    for groups in (1, 15, 40, per_window, 3 * per_window + 17):
        steps = np.sort(rng.integers(0, 50, groups))[::-1]
        desc = desc_of(steps)
        taken = np.maximum(steps, 1)
        for S in (1, 2, 3, 4, 6, 8, 12, 16, 24, 64, 100, 256):
            distance = 16 * math.gcd(S, per_window // 16)
            place = np.arange(groups) % per_window % distance
            worst = max(taken[place == p].mean() for p in set(place.tolist()))
            want = max(taken.max(), worst * -(-groups // (16 * S)))
            got = rules.busiest(P(desc), i64(groups), rows_per_group, i64(S))
            assert abs(got - want) <= 1e-9 * want, (groups, S)
    window = np.sort(rng.integers(1, 90, per_window))[::-1]
    desc = desc_of(np.tile(window, 32))
    for S in (1, 2, 4, 8):
        exact = max(np.tile(window, 32)[split::S][wave::16].sum() for split in range(S) for wave in range(16))
        assert rules.busiest(P(desc), i64(32 * per_window), rows_per_group, i64(S)) == pytest.approx(exact)


def test_splits(rules):
    """The pairs form's: the fewest parts of all that are cheapest by the stated cost; the packed copy's: one workgroup per
    unit or more."""
    rng = np.random.default_rng(4)
    for _ in range(1500):
        slices, groups = int(np.exp(rng.uniform(0, 7))), int(np.exp(rng.uniform(0, 9)))
        blocks = int(groups * np.exp(rng.uniform(0, 5)))
        cost = [-(-slices * s // 256) * (250.0 + blocks / groups * 16 * -(-groups // (16 * s))) for s in range(1, min(256, groups) + 1)]
        assert rules.pair_splits(i64(slices), i64(groups), i64(blocks)) == 1 + int(np.argmin(cost)), (slices, groups, blocks)
        want = 1 if slices >= 256 else -(-256 // slices)
        assert rules.packed_splits(i64(slices), i64(groups)) == min(want, groups)


def test_choice_of_the_form(rules):
    """The estimate of both times, written out; and what it is for: few columns and very unequal rows take the packed copy,
    many columns and unaligned rows of C the pairs form."""
    rng = np.random.default_rng(5)

    def layouts(lens):
        rp = rowptr_of(lens)
        pk, _ = oracle.spmm_packed_layout(rp, oracle.spmm_row_order(rp))
        pp, blocks = oracle.spmm_pair_layout(rp, oracle.spmm_pair_row_order(rp))
        return pk, pp, blocks

    def pick(m, pk, pp, blocks, K, vec):
        return bool(rules.choice(P(pk), i64(pk.size // 2 - 1), P(pp), i64(pp.size // 2 - 1), i64(blocks), i64(m), i64(K), int(vec)))

    for m, lens in ((1, [5]), (700, rng.poisson(20, 700)), (5000, rng.integers(0, 200, 5000)), (4096, np.full(4096, 17)), (3000, rng.poisson(300, 3000))):
        pk, pp, blocks = layouts(lens)
        for K in (1, 16, 17, 64, 333, 1000, 4096, 20000, 2 ** 31 - 2 ** 22):
            for vec in (False, True):
                slices = -(-K // 16)
                sk = rules.packed_splits(i64(slices), i64(pk.size // 2 - 1))
                sp = rules.pair_splits(i64(slices), i64(pp.size // 2 - 1), i64(blocks))
                rk, rpairs = -(-slices * sk // 256), -(-slices * sp // 256)
                ek = rules.busiest(P(pk), i64(pk.size // 2 - 1), 16, i64(sk))
                ep = rules.busiest(P(pp), i64(pp.size // 2 - 1), 32, i64(sp))
                tk, tp = np.maximum(pk[1:-2:2], 1).sum(), pp[1:-2:2].sum()
                c = 1e-6 * m * K
                pairs = rpairs * (7.9 + 0.076 * ep + 0.066 * tp / (16 * sp)) + (0.82 if vec else 2.1) * c
                packed = rk * (6.0 + 0.049 * ek + 0.16 * tk / (16 * sk)) + (0.81 * c if vec else 2.75 + 2.8 * c)
                if abs(pairs - packed) > 1e-9 * packed:
                    assert pick(m, pk, pp, blocks, K, vec) == (pairs < packed), (m, K, vec)
    m = 16384
    usual = layouts(rng.poisson(20, m))
    assert not pick(m, *usual, 16, True) and not pick(m, *usual, 64, True) and pick(m, *usual, 4096, True) and pick(m, *usual, 333, False)
    tail = layouts(np.where(np.arange(m) % 200 == 0, 600, 20))
    assert not any(pick(m, *tail, K, True) for K in (16, 64, 1024, 4096))


POSITIONS, RUNS, SHEETS = range(3)


@pytest.mark.parametrize("elem", [2, 4])
@pytest.mark.parametrize("runs", [0, 1])
def test_kernel_of_a_windowed_product(rules, elem, runs):
    """From sheets only where there are some, the call's arrays allow 16-byte copies and two blocks' buffers (x vectors, values
    and 16 more, sheet, kept y) fit 64 KB; otherwise from the packed runs, or the positions."""
    other = RUNS if runs else POSITIONS
    for staged, rows, sheet in ((1024, 64, 192), (4096, 256, 304), (4095, 1023, 1040)):
        held = (elem * (staged + 16) + 15) // 16 * 16 + sheet
        kept = (4 * rows + 15) // 16 * 16
        fit, fit_kept = (32768 - held) // 16, (32768 - held - kept) // 16   # most x vectors
        k = lambda xv, vec=1, y=0, s=sheet: rules.window_kernel(elem, staged, rows, xv, s, runs, vec, y)
        assert k(fit) == SHEETS and k(fit + 1) == other
        assert k(fit_kept, y=1) == SHEETS and k(fit_kept + 1, y=1) == other and k(fit_kept + 1) == SHEETS
        assert k(fit, vec=0) == other and k(fit, s=0) == other
        assert k(0) == k(1) == SHEETS


@pytest.mark.parametrize("elem", [2, 4])
def test_which_matrices_get_sheets(rules, elem):
    """Not for rows of one length that meet on the same LDS banks, nor for long rows in a few blocks."""
    pay = lambda common, nnz, bn, rm, nb=10**6, m=None: rules.sheets_pay(elem, i64(m or nnz // max(common, 1)), i64(nnz), i64(nb), bn, rm, common, 256)
    small = {4: {32, 48, 64}, 2: {64}}[elem]                  # blocks of 1024 entries and 64 rows
    large = {4: {48, 64}, 2: {16}}[elem]                      # blocks as default_tile_shape makes them
    for L in range(65):
        assert pay(L, 1 << 20, 1024, 64) == (L not in small)
        rm = 256 if L <= 16 else 128 if L <= 32 else 64
        assert pay(L, 1 << 24, max(2048, (rm * L + 7) // 8 * 8), rm) == (L not in large)
    few = 256 if elem == 4 else 512
    for mean, none in ((31, False), (32, True), (61, True)):
        assert pay(0, 100_000 * mean, 1024, 64, nb=few, m=100_000) == (not none)
        assert pay(0, 100_000 * mean, 1024, 64, nb=few + 1, m=100_000)


def test_lanes_of_a_row(rules):
    lanes = lambda elem, mean, rm, places, common=0: rules.stream_lanes(elem, i64(1000), i64(1000 * mean), rm, places, common)
    for elem in (2, 4):
        assert [lanes(elem, 16, 128, p) for p in (5, 6)] == [2, 1] and [lanes(elem, 16, 64, p) for p in (10, 11)] == [2, 1]
        assert lanes(elem, 15, 128, 2) == 1
    assert lanes(4, 24, 128, 9, 24) == 2 and lanes(4, 24, 64, 11, 24) == 1 and lanes(2, 24, 128, 9, 24) == 1


@pytest.mark.parametrize("lens,want", [([64] * 9, 64), ([65] * 9, 0), ([0] * 9, 0), ([32] * 8 + [64] * 4, 64), ([32] * 8 + [64] * 3, 32),
                                       ([5] * 100 + [4] * 20 + [3], 5), (list(range(1, 60)), 0), ([16] * 10 + [161], 0)])
def test_common_row_length(rules, lens, want):
    rp = rowptr_of(lens)
    assert rules.common_len(i64(len(lens)), P(rp)) == want


@pytest.mark.parametrize("line", [64, 128, 129, 4096])
def test_common_row_length_of_a_sample(rules, line):
    """More rows than are looked at: lines of a grid whose end points have shorter rows, whatever the lines' length."""
    for m in (4097, 64 * line, 4096 * line // 8 + 1):
        at = np.arange(m) % line
        for length in (5, 27, 64):
            assert rules.common_len(i64(m), P(rowptr_of(np.where((at == 0) | (at == line - 1), length - 3, length)))) == length
    assert rules.common_len(i64(9000), P(rowptr_of([7, 8, 9] * 3000))) == 0


def test_gather_rule(rules):
    import paper_2603_07169_amd as s
    rules.gather_snap.restype = C.c_int64
    A, M = s.SPMV_PLAN_ADAPTIVE, s.SPMV_PLAN_MERGE
    for bf16, least in ((0, 7 << 16), (1, 3 << 17)):
        choice = lambda m, nnz, plan, longest, k=1, n=50000: rules.gather_choice(i64(m), i64(n), i64(nnz), plan, bf16, i64(longest), 256, k)
        assert choice(30000, least, A, 20) and not choice(30000, least - 1, A, 20)
        assert choice((1 << 17) + 1, 3 << 17, A, 20) and choice(1 << 17, 3 << 17, A, 20) == bool(bf16)
        items = -(-(30000 + least) // 256)
        assert choice(30000, least, A, items // 2) and not choice(30000, least, A, items // 2 + 1)  # half a chunk is the longest uncut row
        assert not choice(30000, least, A, items // 2, 4)                                           # chunks of a quarter the steps
        assert choice(10000, 1 << 16, M, 2000) and not choice(10000, (1 << 16) - 1, M, 2000)
        steps = -(-(10000 + (1 << 16)) // 256)
        assert choice(10000, 1 << 16, M, 32 * (steps - 192)) and not choice(10000, 1 << 16, M, 32 * (steps - 192) + 1)
        assert choice(1000, 768000, A, 800, n=16384) == (not bf16)                                  # long rows, an x that a unit's cache holds
        assert not bf16 or (choice(1000, 767999, A, 800, n=16384) and choice(1000, 768000, A, 800, n=16385))
    for plan in (s.SPMV_PLAN_SCALAR, s.SPMV_PLAN_VECTOR, s.SPMV_PLAN_BINNED, s.SPMV_PLAN_WINDOWED, s.SPMV_PLAN_TWOPHASE, s.SPMV_PLAN_COLBLOCK, s.SPMV_PLAN_SELL):
        assert not choice(30000, 1 << 20, plan, 20)
    assert rules.gather_snap(A, i64(300), i64(2000)) == 300
    assert rules.gather_snap(M, i64(9000), i64(2048)) == 2048 and rules.gather_snap(M, i64(9000), i64(2049)) == 512


def test_gather_rule_of_the_lines(rules):
    """Lines saved to a compute unit: what stretches of entries touch beyond their chunks, less what the worst chunk is above the mean."""
    import paper_2603_07169_amd as s
    A, M = s.SPMV_PLAN_ADAPTIVE, s.SPMV_PLAN_MERGE

    def pays(m, nnz, plan, bf16, saved, excess=0, mean=100, chunks=256):
        return rules.gather_pays(i64(m), i64(nnz), plan, bf16, 256, i64(chunks), i64(mean + excess), i64(mean * chunks), i64(mean * chunks + 256 * (saved + excess)))

    for excess, chunks in ((0, 256), (700, 256), (700, 1024)):
        at = lambda *case: pays(*case, excess=excess, chunks=chunks)
        assert at(10000, 4 << 20, M, 0, -2000) and not at(10000, 4 << 20, M, 0, -2001)
        assert at(10000, 4 << 20, M, 1, -1250) and not at(10000, 4 << 20, M, 1, -1251)
        assert at(256 * 1600, 4 << 20, A, 0, 400) and not at(256 * 1600, 4 << 20, A, 0, 399)       # a quarter of the rows to a unit
        assert at(256 * 1600, 4 << 20, A, 1, 1100) and not at(256 * 1600, 4 << 20, A, 1, 1099)     # eleven sixteenths
    for plan in (A, M):  # short calls, whatever the lines are
        assert pays(256 * 500, 256 * 5680, plan, 1, -9000) and not pays(256 * 500, 256 * 5680 + 1, plan, 1, -9000)


def test_rule_of_gathered_groups(rules):
    takes = lambda m, groups: rules.gather_groups_choice(i64(m), i64(groups), 256)
    few, many = 3072 * 256, 3072 * 256 + 1
    assert takes(few, 2 * few) and not takes(few, 2 * few - 1)
    assert takes(many, 3 * many) and not takes(many, 3 * many - 1)


NOT_GROUPS = {  # row lengths, first column of every row: each row's columns follow one another
    "diagonal": ([1] * 512, np.arange(512)),
    "rows_of_4": ([4] * 512, 4 * np.arange(512)),
    "rows_of_12": ([12] * 512, 12 * np.arange(512)),
    "rows_of_4_and_12": ([4, 12] * 256, np.arange(512) // 2 * 16 + np.arange(512) % 2 * 4),
    "short_last_row": ([8] * 511 + [5], 8 * np.arange(512)),
    "band": ([16] * 512, np.arange(512)),  # whole groups, at columns that are no multiple of eight
}


@pytest.mark.parametrize("name", list(NOT_GROUPS))
def test_grouped_positions_do_not_make_a_matrix_of_groups(rules, name):
    """What the product on groups of eight asks of the rows (the columns are asked of the device); the positions of all these are grouped."""
    lens, first = NOT_GROUPS[name]
    rp = rowptr_of(lens)
    cols = (np.repeat(first, lens) + np.arange(rp[-1]) - np.repeat(rp[:-1], lens)).astype(np.int32)
    blocks = oracle.row_blocks(rp, 1024, 64)
    _, _, _, lidx = oracle.x_windows(rp, cols, blocks, 1024, 8)
    assert oracle.lidx_grouped(rp, blocks, lidx) and not oracle.csr_groups(len(lens), rp, cols)
    assert rules.rows_of_groups(i64(len(lens)), P(rp)) == (name == "band")


def test_rows_of_groups(rules):
    for lens in ([], [0, 0], [8], [0, 16, 8, 0, 24]):
        assert rules.rows_of_groups(i64(len(lens)), P(rowptr_of(lens)))
    for lens in ([7], [8, 1], [4, 4], [8, 12, 4, 8], [0, 9]):
        assert not rules.rows_of_groups(i64(len(lens)), P(rowptr_of(lens)))
