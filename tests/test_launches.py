"""What is launched, looked at on the host: where kernels read in LDS, how much of it a launch asks for, and which kernel a call
takes, for calls whose results would not show it."""
import os
import subprocess

import pytest

import launch_recorder

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("launches"))


def test_products_of_the_swap_tables_stay_inside_their_tiles(tmp_path):
    """Every tile that a wave of swap_cooc_kernel multiplies lies in the rows that its launch asks LDS for, for all experts and
    groups, also where another cut has fewer groups than the one the launch is sized for."""
    (tmp_path / "walk.cpp").write_text(r"""
#include <cstdio>
#include "hm_cooc.h"
template <int COLS> static int walk(int E, int ng) {
  typedef hm::CoocTiles<COLS> layout;
  const layout t(E, ng);
  int bad = t.rows() != 32 * ((E + 31) / 32 + COLS + (ng + 31) / 32), c = 0, g = 0;
  auto inside = [&](int first, int tiles, int from, int to) { return first >= from && first + 32 * tiles <= to; };
  for (int w = 0; w < hm::kCoocWaves; ++w) {
    if (t.has_c(w)) ++c, bad += !inside(t.c_rows(w), 1, 0, t.s_at()) + !inside(t.c_columns(w), layout::kColumnsOfC, t.s_at(), t.m_at());
    if (t.has_g(w)) ++g, bad += !inside(t.g_rows(w), 1, t.s_at(), t.m_at()) + !inside(t.g_columns(w), layout::kColumnsOfG, t.m_at(), t.rows());
    if (COLS > 1) bad += t.has_c(w) && t.has_g(w);   // these share their sums
  }
  bad += c != (E + 31) / 32 || g != COLS * ((ng + 31) / 32);   // every tile has a wave
  if (bad) std::printf("E %d groups %d columns %d: %d\n", E, ng, COLS, bad);
  return bad;
}
int main() {
  int bad = 0;
  for (int E = 1; E <= 512; ++E)
    for (int ng = 1; ng <= 64; ++ng) bad += hm::cooc_columns(E) == 2 ? walk<2>(E, ng) : walk<1>(E, ng);
  return bad != 0;
}
""")
    exe = str(tmp_path / "walk")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_09591_amd", "csrc"), "-o", exe, str(tmp_path / "walk.cpp")])
    p = subprocess.run([exe], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout[:2000]


def test_selection_asks_for_no_more_lds_than_every_launch_gets(recorder):
    """All hierarchies of the ranks that the call takes, steps that split nothing among them: the counts staged in LDS and the terms of
    64 pairs (four doubles each) beside them stay inside what a kernel has without asking for more, and what fits is staged."""
    result = launch_recorder.run(recorder, r"""
result = []
def chains(G, d, U):
    if len(U) == d:
        yield U
        return
    for u in range(U[-1], G + 1):
        if u % U[-1] == 0 and G % u == 0:
            yield from chains(G, d, U + [u])
for G in (1, 2, 12, 32, 33, 36, 40, 48, 60, 64):
    for d in (1, 2, 3, 4):
        for U in chains(G, d, [1]):
            zi, five = (ctypes.c_void_p * d)(*[at(1).value] * d), (ctypes.c_double * d)(*[0.5] * d)
            rc = L.hm_swap_select(d, (ctypes.c_int32 * d)(*U), G, 64, 8.0, 2.0, zi, at(2), five, 1.0, five, five, 0.1, 0.1, 10.0, at(3), at(4), at(5), at(6),
                                  1 << 30, None)
            result.append([G, U, rc, launched()])
""")
    assert len(result) > 300
    for G, U, rc, launches in result:
        assert rc == 0 and [k["name"] for k in launches] == ["swap_q_kernel<%d>" % (32 if G <= 32 else 64), "swap_argmin_kernel<256>"], (G, U)
        q = launches[0]
        assert q["lds"] + 4 * 64 * 8 <= q["granted"], (G, U, q)
        wanted = [256 * n for n in U[1:] + [G] if n % 4 == 0 and G > 32]
        assert q["lds"] == (sum(wanted) if sum(wanted) + 4 * 64 * 8 <= 65536 else sum(wanted[:3])), (G, U, q)


# A plan of T tokens with a bound of `most` rows per token and, where `rows` is not None, a row count.
_ROWS = r"""
def plan(T, K, most, rows):
    c = B.hm_plan_out()
    c.num_dest, c.row_capacity, c.max_rows_per_token = 32, T * K, most
    c.expected_rows = 0 if rows is None else int(rows * T)
    for i, f in enumerate(("dest_count", "dest_offset", "row_token", "slot_row", "slot_keep", "row_weight", "status")):
        setattr(c, f, at(20 + i).value)
    return ctypes.byref(c)
def kernel(rc):
    assert rc == 0
    one, = launched()
    return one["name"], one["grid"][0]
"""


def test_dispatch_groups_workgroups_by_sizes_alone(recorder):
    """Rows off the line grid: 128 neighbours on one die for rows of 32 bytes or more and up to 80 MB of tokens, 130 MB up to 1,400 bytes a
    row, and at least one whole round of 1,024 workgroups, for each kernel that has the choice and whatever is known of the rows per
    token; whole lines keep the launch order."""
    result = launch_recorder.run(recorder, _ROWS + r"""
result = []
for T, H, off in ((4097, 1030, 0), (38834, 1030, 0), (38835, 1030, 0), (8192, 15, 0), (8192, 17, 0), (92857, 700, 0), (92858, 700, 0), (65000, 701, 0),
                  (65536, 72, 0), (100, 7161, 0), (136, 7161, 0), (137, 7161, 0), (4096, 1024, 16), (4096, 1024, 0), (65536, 100, 0)):
    names = set()
    for most, rows in ((8, None), (0, None), (8, 1.2), (8, 3.0), (8, 5.6), (8, 7.7)):
        x, out = at(1), ctypes.c_void_p(at(2).value + off)
        names.add(kernel(L.hm_dispatch_pack(x, T, 8, H, plan(T, 8, most, rows), out, 8 * T, None)))
    result.append([T, H, off, sorted(names)])   # of kernel and grid
""")
    assert len({n.split("<")[0] for r in result for n, _ in r[3]}) >= 3   # spread_ragged, spread_flat, dispatch_rows
    assert {g >= 1024 for r in result for _, g in r[3]} == {False, True}
    for T, H, off, names in result:
        sizes = (H % 64 != 0 or off != 0) and 2 * H >= 32 and 2 * T * H <= (130e6 if 2 * H <= 1400 else 80e6)
        for name, grid in names:
            assert name.startswith("dispatch_elems") or name.endswith("true>") == (sizes and grid >= 1024), (T, H, off, name, grid)


def test_transpose_reads_eight_rows_for_a_row_count_not_for_a_bound(recorder):
    """Ragged rows: the reads of eight rows in flight for the bf16 transpose of up to eight slots that a row count says are kept nearly all, of
    7 MB or more; four for a plan that was never synchronised, whose bound is eight whatever it holds, and for fp32."""
    result = launch_recorder.run(recorder, _ROWS + r"""
result = []
for T, H in ((16384, 1030), (4097, 1030), (3398, 1030), (3399, 1030), (16384, 2050)):
    for K, most, rows in ((8, 8, None), (8, 0, None), (8, 8, 1.2), (8, 8, 6.9), (8, 8, 7.2), (8, 8, 8), (6, 6, None), (6, 6, 5.8), (5, 5, 4.2), (4, 4, 4), (10, 10, 9.9)):
        for fn, bits in (("hm_combine_transpose_bf16", 16), ("hm_combine_transpose", 32)):
            result.append([T, H, K, rows, bits, kernel(getattr(L, fn)(at(1), T, K, H, plan(T, K, most, rows), at(2), 8 * T, None))[0]])
""")
    for T, H, K, rows, bits, name in result:
        eight = bits == 16 and rows is not None and K <= 8 and rows > max(K - 1, 4.25) and 2 * T * H >= 7e6
        assert name == "spread_ragged_kernel<RowBf16, true, %d, false>" % (8 if eight else 4) if bits == 16 else "RowF32, true, 4" in name, (T, H, K, rows, name)


def test_chunks_of_the_swap_tables_are_summed_by_one_kernel(recorder):
    """Whatever the number of tokens: 16-bit counts of a chunk, up to 16 of them, summed in 32 bits."""
    result = launch_recorder.run(recorder, r"""
result = []
for E in (16, 128, 256):
    for T in (0, 100, 65535, 65536, 522240):
        rc = L.hm_swap_counts(at(1), at(2), T, 8, E, 32, 32, at(3), None, at(4), 1 << 40, None)
        result.append([rc, [k["name"] for k in launched()]])
""")
    for rc, names in result:
        assert rc == 0 and len(names) == 2 and names[1] == "swap_pairs_kernel<unsigned short, 16>", names


def test_counts_take_the_kernel_their_sizes_ask_for(recorder):
    """One kernel of each kind for loads and group counts, and one workgroup only where the owners' table has no room."""
    result = launch_recorder.run(recorder, r"""
result = []
for T, K, E in ((0, 8, 64), (256, 2, 16), (8192, 8, 128), (1024, 64, 4096), (1024, 8, 4097), (600, 8, 8193), (16384, 8, 128), (100001, 1, 256), (30001, 3, 64),
                (70000, 24, 48), (2000000, 1, 4096), (5000, 8, 5000)):
    names = []
    L.hm_expert_load(at(1), at(2), T, K, E, B.hm_topology(4, 8), at(3), at(4), at(5), at(6), None)
    names.append([k["name"] for k in launched()])
    L.hm_group_counts(at(1), at(2), T, K, E, 32, 2, (ctypes.c_int32 * 2)(32, 4), at(3), at(4), None)
    result.append([T, K, E, names + [[k["name"] for k in launched()]]])
""")
    seen = set()
    for T, K, E, both in result:
        for names, what in zip(both, ("load", "group")):
            seen.update(names)
            width = 4 if K >= 4 else 2 if K >= 2 else 1
            alone = T <= 1024 and (E <= 8192 if what == "load" else T * K <= 32768)
            if E > 4096 and alone:
                assert names == ["%s_count_kernel<1024, true>" % what], (T, K, E, names)
            elif E > 4096:
                assert names == ["%s_clear_kernel" % what, "%s_count_kernel<256, false>" % what], (T, K, E, names)
            else:
                assert names in (["%s_owner_kernel<%d, false>" % (what, width)], ["%s_clear_kernel" % what, "%s_owner_kernel<%d, true>" % (what, width)],
                                 ["%s_clear_kernel" % what, "%s_count_kernel<256, false>" % what]), (T, K, E, names)
    assert len(seen) == 2 * (1 + 1 + 1 + 3 + 2), sorted(seen)   # clear, one workgroup, added, spread, whole of two widths


def test_swap_tables_take_the_kernels_their_sizes_ask_for(recorder):
    """Matrix products with partial tables, with added ones, and atomics per slot with their tables in LDS and in memory."""
    result = launch_recorder.run(recorder, r"""
result = []
for E, K, G, T, cuts, way in ((128, 8, 32, 8192, [4, 32], "parts"), (256, 9, 32, 8192, [32], "slots"), (256, 8, 32, 522240, [32], "parts"), (256, 8, 32, 522241, [32], "added"),
                              (257, 8, 32, 8192, [32], "added"), (512, 8, 64, 9001, [8, 64], "added"), (513, 8, 32, 8192, [32], "atomics"), (300, 9, 8, 400, [8], "atomics"),
                              (288, 2, 8, 46004, [1, 8], "atomics"), (300, 1, 32, 300000, [4, 32], "atomics"), (64, 1, 8, 523000, [8], "atomics"),
                              (600, 3, 64, 5000, [16, 32, 64], "memory")):
    Z = (ctypes.c_void_p * len(cuts))(*[at(3 + i).value for i in range(len(cuts))])
    rc = L.hm_swap_counts_multi(at(1), at(2), T, K, E, G, len(cuts), (ctypes.c_int32 * len(cuts))(*cuts), Z, at(10), at(11), 1 << 40, None)
    result.append([E, K, T, way, rc, launched()])
""")
    for E, K, T, way, rc, launches in result:
        cols = 2 if 128 < E <= 256 else 1
        want = {"parts": ["swap_cooc_kernel<%d, true, false>" % cols, "swap_pairs_kernel<unsigned short, 16>"],
                "slots": ["swap_slots_kernel", "swap_cooc_kernel<%d, false, false>" % cols, "swap_pairs_kernel<unsigned short, 16>"],
                "added": ["swap_cooc_kernel<%d, true, true>" % cols, "swap_pairs_kernel<int, 1>"]}.get(way, ["swap_factors_kernel", "swap_build_kernel"])
        assert rc == 0 and [k["name"] for k in launches] == ["swap_clear_kernel"] + want, (E, K, T, way, launches)
        assert all(k["lds"] <= k["granted"] for k in launches), launches
        if way in ("atomics", "memory"):
            assert (launches[1]["lds"] > 0) == (way == "atomics"), launches
